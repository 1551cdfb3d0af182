// Float32-path kernels on the float32 matrix instruction (gfx950): causal GQA attention and the GEMM.
// Operands, products and sums are float32 throughout (32x32x2 and 16x16x4 MFMAs); nothing is rounded to a narrower
// type.  The float32 path is the one that is held to 1e-4 against the float64 definition and that stands in for it
// at configurations no CPU run reaches, so what matters here is that every output is one float32 dot product in a
// fixed order that depends on nothing but its own row and column; speed only has to be enough for whole
// configurations (32 layers x 32768 tokens) to run in seconds.
#include "po_internal.h"

namespace po {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------ attention
// softmax(Q K^T / sqrt(hd)) V with the causal mask, grouped-query heads (Section 4.2 of the paper: attention runs
// over the whole sequence, unchunked).  Workgroup = 128 query rows of one head, wavefront = 32 of them.  Keys go by
// in tiles of 32 staged in LDS (K rows padded by 4 floats, V rows as they are).  Per tile a wavefront forms
// S^T[key][query] = K Q^T with 64 (hd 128) matrix instructions, so that a lane owns ONE query column -- lane l and
// lane l ^ 32 share it, 16 keys each -- and the online softmax needs one exchange with the partner lane per tile;
// the probabilities never leave their registers: register r of S^T is exactly the B operand of step r of
// O^T[hd][query] += V^T P^T when the V fragment of that step is read at the key that register r holds.
// The contraction index of Q K^T is split between the lane halves (half h takes elements [h hd/2, (h+1) hd/2)), so
// that a lane's K fragment is contiguous in LDS (16-byte reads).
// A query's result depends only on its own column of S^T and on the tile grid, which starts at key 0 for every
// workgroup: it is the same bits wherever the row sits in a workgroup and whichever rows are computed beside it
// (tiles wholly above a wavefront's rows are skipped; they would contribute p = 0 and a rescale by 1, exactly).
// o may alias q: a wavefront reads its own 32 query rows before it writes them, and nobody else touches them.
template <int HD>
__global__ void __launch_bounds__(256, HD == 128 ? 1 : 2) attention_f32_mfma_kernel(const float* q, const float* __restrict__ k,
                                                                    const float* __restrict__ v, float* o, int64_t N,
                                                                    int Hq, int Hkv, int64_t blk0) {
    constexpr int KP = HD + 4;        // padded K row: 8 lanes' 16-byte reads fall into different banks
    constexpr int HH = HD / 2;        // contraction elements per lane half
    constexpr int NB = HD / 32;       // 32-row blocks of O^T
    constexpr int V4 = HD / 32;       // float4 per thread and operand of one staged tile (32 rows x HD floats, 256 threads)
    constexpr int RV = HD / 4;        // float4 per row
    __shared__ __align__(16) float Ks[32 * KP];
    __shared__ __align__(16) float Vs[32 * HD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int h = blockIdx.y;
    const int c = h / (Hq / Hkv);
    const int64_t r0 = ((int64_t)(gridDim.x - 1 - blockIdx.x) + blk0) * 128;      // longest rows first
    const int64_t q0 = r0 + wave * 32;          // this wavefront's first query row
    const int64_t t = q0 + col;                 // this lane's query row
    const bool live = t < N;
    const float scale = 1.0f / sqrtf((float)HD);

    float qf[HH];
    {
        const float* qp = q + (t * Hq + h) * HD + half * HH;
#pragma unroll
        for (int i = 0; i < HH / 4; ++i) {
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (live) x = *(const float4*)(qp + 4 * i);
            qf[4 * i] = x.x; qf[4 * i + 1] = x.y; qf[4 * i + 2] = x.z; qf[4 * i + 3] = x.w;
        }
    }
    f32x16 O[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[b][r] = 0.f;
    float m = -INFINITY, l = 0.f;

    const int64_t kv_end = (r0 + 128 < N) ? r0 + 128 : N;
    float4 pk[V4], pv[V4];
    auto fetch = [&](int64_t kv0) {
#pragma unroll
        for (int j = 0; j < V4; ++j) {
            const int idx = tid + 256 * j;
            const int64_t s = kv0 + idx / RV;
            const int c4 = idx % RV;
            pk[j] = pv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s < N) {
                pk[j] = *(const float4*)(k + (s * Hkv + c) * HD + 4 * c4);
                pv[j] = *(const float4*)(v + (s * Hkv + c) * HD + 4 * c4);
            }
        }
    };
    fetch(0);
    for (int64_t kv0 = 0; kv0 < kv_end; kv0 += 32) {
        __syncthreads();                        // everybody is done reading the previous tile
#pragma unroll
        for (int j = 0; j < V4; ++j) {
            const int idx = tid + 256 * j;
            const int row = idx / RV, c4 = idx % RV;
            *(float4*)(Ks + row * KP + 4 * c4) = pk[j];
            *(float4*)(Vs + row * HD + 4 * c4) = pv[j];
        }
        __syncthreads();
        if (kv0 + 32 < kv_end) fetch(kv0 + 32);          // in flight during this tile's arithmetic
        if (kv0 > q0 + 31) continue;                     // wavefront-uniform: every key of the tile is masked for these rows

        f32x16 S;
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = 0.f;
        const float* kr = Ks + col * KP + half * HH;
#pragma unroll
        for (int i = 0; i < HH / 4; ++i) {
            const float4 kk = *(const float4*)(kr + 4 * i);
            S = mfma_f32(kk.x, qf[4 * i], S);
            S = mfma_f32(kk.y, qf[4 * i + 1], S);
            S = mfma_f32(kk.z, qf[4 * i + 2], S);
            S = mfma_f32(kk.w, qf[4 * i + 3], S);
        }
        // register r holds key kv0 + 8 (r / 4) + 4 half + r % 4 of query t
        float p[16];
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t key = kv0 + 8 * (r / 4) + 4 * half + (r % 4);
            p[r] = key > t ? -INFINITY : S[r] * scale;
            tmax = fmaxf(tmax, p[r]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        const float mn = fmaxf(m, tmax);                 // finite: key kv0 <= q0 <= t is never masked
        const float a = expf(m - mn);                    // exp(-inf) = 0 on the first tile
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = expf(p[r] - mn);
            psum += p[r];
        }
        l = l * a + psum;                                // this lane's 16 keys; the partner's are added at the end
        m = mn;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r) O[b][r] *= a;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float vv = Vs[(8 * (r / 4) + 4 * half + (r % 4)) * HD + 32 * b + col];
                O[b] = mfma_f32(vv, p[r], O[b]);
            }
        }
    }
    l += __shfl_xor(l, 32);
    if (!live) return;
    const float inv = 1.0f / l;
    float* op = o + (t * Hq + h) * HD;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(float4*)(op + 32 * b + 8 * g + 4 * half) =
                make_float4(O[b][4 * g] * inv, O[b][4 * g + 1] * inv, O[b][4 * g + 2] * inv, O[b][4 * g + 3] * inv);
}

// q_row0: rows below it need no result (the workgroup that holds it still computes its rows from the 128-row
// boundary on; what it writes below q_row0 nobody reads)
bool launch_attention_f32_mfma(const float* q, const float* k, const float* v, float* o, int64_t N, int Hq, int Hkv, int hd,
                               int64_t q_row0, hipStream_t s) {
    if (N <= 0) return true;
    if (hd != 64 && hd != 128) return false;
    const int64_t blk0 = (q_row0 > 0 && q_row0 < N) ? q_row0 / 128 : 0;
    const dim3 grid((unsigned)((N + 127) / 128 - blk0), (unsigned)Hq);
    if (hd == 128)
        hipLaunchKernelGGL(attention_f32_mfma_kernel<128>, grid, dim3(256), 0, s, q, k, v, o, N, Hq, Hkv, blk0);
    else
        hipLaunchKernelGGL(attention_f32_mfma_kernel<64>, grid, dim3(256), 0, s, q, k, v, o, N, Hq, Hkv, blk0);
    return true;
}

// ------------------------------------------------------------------ GEMM
// C[M,N] = A[M,K] W[N,K]^T (+bias) (+R), all float32, on v_mfma_f32_16x16x4_f32.  Four wavefronts arranged 2 x 2, each a
// patch of T x T tiles of 16 x 16; K in slices of 32 floats, so that a row of an operand slice is one 128-byte line,
// copied global -> LDS directly (buffer_load ... lds, 16-byte segments XOR-swizzled with the row on the global side, as in
// gemm_mfma.hip) into a ring of D slices.  In a slice lane group g = lane / 16 multiplies elements 8 g .. 8 g + 7 of its
// row, one per MFMA.  The fragments of a slice are read while the one before is multiplied; one barrier per slice hands
// slice s + 1 over and frees the position of slice s, into which slice s + D is loaded.
// What bounds it: many rows, the matrix pipe (a bare loop of this instruction does 155 TFLOP/s, the same as 32x32x2); few
// rows, the chain of K / 4 dependent MFMAs per output, which the 32 x 32 tile runs four times faster than one of
// 32x32x2, and the latency of a slice, which the ring depth hides.
// Every output is one running sum over K in one fixed order, whatever M, N and the tile: row results do not depend on
// which other rows a launch computes.  C may alias R (a lane reads the residual it then overwrites).
// Measured (kernel before: 128 x 128 tiles of 32x32x2, slices staged through registers, two barriers each): 1000 rows of
// the 8B shape, down projection 1060 -> 866 us (136 TFLOP/s), gate/up 1990 -> 1726; 256 x 256 outputs of K 256 26 -> 9 us;
// one row of K 14336 1034 -> 84 us.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

#ifdef __HIP_DEVICE_COMPILE__
#define PO_WAIT_BARRIER(n_) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n_) : "memory")
#else
#define PO_WAIT_BARRIER(n_)
#endif

template <int T, int D>
__global__ void __launch_bounds__(256, 2) gemm_f32_mfma_kernel(const float* __restrict__ A, int64_t lda,
                                                               const float* __restrict__ W, int64_t ldw, float* C,
                                                               int64_t ldc, const float* __restrict__ bias, const float* R,
                                                               int64_t ldr, int64_t M, int N, int K) {
    constexpr int BT = 32 * T, UNIT = BT * 128;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, l4 = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)blockIdx.y * BT;
    const int n0 = blockIdx.x * BT;
    const int rows_a = (int)min((int64_t)BT, M - m0), rows_w = min(BT, N - n0);
    // resources: the rows of the tile that exist (others read as zero)
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + m0 * lda), 0, (int)(uint32_t)(rows_a * lda * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (int64_t)n0 * ldw), 0, (int)(uint32_t)(rows_w * ldw * 4), 0x00020000);
    uint32_t voa[4], vow[4];                     // (T entries used: T loads of 8 rows per wavefront and operand)
    const int KT = (K + 31) / 32;
    uint32_t tail = 0;                           // bit i: load i of the last slice lies beyond K for this lane
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int row = (wave * T + i) * 8 + (lane >> 3);
        const int seg = (lane & 7) ^ ((row >> 1) & 7);
        voa[i] = (uint32_t)row * (uint32_t)(lda * 4) + seg * 16;
        vow[i] = (uint32_t)row * (uint32_t)(ldw * 4) + seg * 16;
        if ((KT - 1) * 32 + seg * 4 >= K) tail |= 1u << i;
    }
    // byte offset of slice s_ along K; slices past the end, and columns of the last one past K, lie outside the resources:
    // they read as zero without traffic
#define PO_DMA(s_, pos_, i_)                                                                                          \
    {                                                                                                                  \
        const int so_ = (s_) < KT ? (s_) * 128 : 0x40000000;                                                           \
        const uint32_t past_ = ((s_) == KT - 1 && (tail >> (i_) & 1)) ? 0x40000000u : 0u;                              \
        unsigned char* d_ = smem + (pos_) * 2 * UNIT + (wave * T + (i_)) * 1024;                                       \
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)d_, 16, voa[(i_)] + past_, so_, 0, 0); \
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(d_ + UNIT), 16, vow[(i_)] + past_, so_, 0, 0); \
    }
    int fo[2];                                   // the lane's 8 elements of a row: segments 2 g and 2 g + 1
#pragma unroll
    for (int h = 0; h < 2; ++h) fo[h] = l15 * 128 + (((2 * l4 + h) ^ ((l15 >> 1) & 7)) << 4);
    const int a_base = wm * (T * 16) * 128, w_base = UNIT + wn * (T * 16) * 128;
    f32x4 acc[T][T];                             // [token tile][feature tile]
#pragma unroll
    for (int u = 0; u < T; ++u)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D; ++s)
#pragma unroll
        for (int i = 0; i < T; ++i) PO_DMA(s, s, i)
    PO_WAIT_BARRIER((D - 1) * 2 * T);            // slice 0 has landed
    f32x4 a0[2][T], w0[2][T], a1[2][T], w1[2][T];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < T; ++j) {
            a0[h][j] = *(const f32x4*)(smem + a_base + j * 2048 + fo[h]);
            w0[h][j] = *(const f32x4*)(smem + w_base + j * 2048 + fo[h]);
        }
    // one slice from registers (AC, WC); the next one's fragments and the loads of slice s + D go out in front of it
#define PO_SLICE(AC, WC, AN, WN)                                                                                     \
    {                                                                                                                 \
        PO_WAIT_BARRIER((D - 2) * 2 * T);          /* slice s+1 has landed; all LDS reads of slice s are done */      \
        const int ps1 = ps + 1 >= D ? 0 : ps + 1;                                                                     \
        const unsigned char* u1 = smem + ps1 * 2 * UNIT;                                                              \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                                 \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                                               \
            _Pragma("unroll") for (int u = 0; u < T; ++u)                                                             \
            _Pragma("unroll") for (int t = 0; t < T; ++t)                                                             \
                acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(WC[h][t][e], AC[h][u][e], acc[u][t], 0, 0, 0);       \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
            if (h == 0 && e == 0) {                                                                                   \
                _Pragma("unroll") for (int i = 0; i < T; ++i) PO_DMA(s + D, ps, i)                                    \
            }                                                                                                         \
            if (h == 0 && e > 0 && e < 3) {                                                                           \
                _Pragma("unroll") for (int j = 0; j < T; ++j) {                                                       \
                    if (e == 1) AN[0][j] = *(const f32x4*)(u1 + a_base + j * 2048 + fo[0]);                           \
                    else WN[0][j] = *(const f32x4*)(u1 + w_base + j * 2048 + fo[0]);                                  \
                }                                                                                                     \
            }                                                                                                         \
            if (h == 1 && e < 2) {                                                                                    \
                _Pragma("unroll") for (int j = 0; j < T; ++j) {                                                       \
                    if (e == 0) AN[1][j] = *(const f32x4*)(u1 + a_base + j * 2048 + fo[1]);                           \
                    else WN[1][j] = *(const f32x4*)(u1 + w_base + j * 2048 + fo[1]);                                  \
                }                                                                                                     \
            }                                                                                                         \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
        }                                                                                                             \
        ps = ps1;                                                                                                     \
    }
    int ps = 0;                                  // ring position of slice s
    int s = 0;
    for (; s + 2 <= KT; ++s) {
        PO_SLICE(a0, w0, a1, w1)
        ++s;
        PO_SLICE(a1, w1, a0, w0)
    }
    if (s < KT) PO_SLICE(a0, w0, a1, w1)
#undef PO_SLICE
#undef PO_DMA
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // a lane holds token row l15 of a tile and four consecutive features
    const bool vec = (N % 4 == 0) && (ldc % 4 == 0) && (!R || ldr % 4 == 0);
#pragma unroll
    for (int u = 0; u < T; ++u) {
        const int64_t gm = m0 + wm * (T * 16) + u * 16 + l15;
        if (gm >= M) continue;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int gn = n0 + wn * (T * 16) + t * 16 + 4 * l4;
            if (gn >= N) continue;
            float x[4] = {acc[u][t][0], acc[u][t][1], acc[u][t][2], acc[u][t][3]};
            if (vec) {          // N % 4 == 0 and gn % 4 == 0: the four columns exist
                if (bias) {
                    const float4 b = *(const float4*)(bias + gn);
                    x[0] += b.x; x[1] += b.y; x[2] += b.z; x[3] += b.w;
                }
                if (R) {
                    const float4 r = *(const float4*)(R + gm * ldr + gn);
                    x[0] += r.x; x[1] += r.y; x[2] += r.z; x[3] += r.w;
                }
                *(float4*)(C + gm * ldc + gn) = make_float4(x[0], x[1], x[2], x[3]);
            } else {
                for (int e = 0; e < 4 && gn + e < N; ++e) {
                    float y = x[e];
                    if (bias) y += bias[gn + e];
                    if (R) y += R[gm * ldr + gn + e];
                    C[gm * ldc + gn + e] = y;
                }
            }
        }
    }
}

template <int T, int D>
static void launch_f32_tile(const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc, const float* bias,
                            const float* R, int64_t ldr, int64_t M, int N, int K, hipStream_t s) {
    constexpr int BT = 32 * T, SMEM = D * 2 * BT * 128;
    static_assert(SMEM <= 64 * 1024, "two workgroups per compute unit, and no larger than a launch may ask for unannounced");
    const dim3 grid((unsigned)((N + BT - 1) / BT), (unsigned)((M + BT - 1) / BT));
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<T, D>), grid, dim3(256), SMEM, s, A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K);
}

// false (nothing launched) when the operands do not allow 16-byte loads along K
bool launch_gemm_f32_mfma(const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc, const float* bias,
                          const float* R, int64_t ldr, int64_t M, int N, int K, hipStream_t s) {
    if (M <= 0 || N <= 0) return true;
    if (K <= 0 || K % 4 || lda % 4 || ldw % 4 || ((uintptr_t)A | (uintptr_t)W | (uintptr_t)C | (uintptr_t)bias | (uintptr_t)R) % 16)
        return false;
    if (lda >= (1 << 20) || ldw >= (1 << 20)) return false;      // a tile is addressed with offsets below 2^30 bytes
    // Tile by time: a round of 256 tiles, one per compute unit, costs this many microseconds per K slice of 32 (measured
    // on 256 .. 2048 tiles of each); where all three take one round the small tile has the shorter chain.
    constexpr double us[3] = {1.9, 0.54, 0.2};                     // tiles of 128, 64, 32
    int best = 0;
    double best_us = 0;
    for (int i = 0; i < 3; ++i) {
        const int64_t bt = 128 >> i, tiles = ((M + bt - 1) / bt) * ((N + bt - 1) / bt);
        const double t = us[i] * (double)((tiles + 255) / 256);
        if (i == 0 || t < best_us) { best = i; best_us = t; }
    }
    if (best == 0) launch_f32_tile<4, 2>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, s);
    else if (best == 1) launch_f32_tile<2, 4>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, s);
    else launch_f32_tile<1, 8>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, s);
    return true;
}

}  // namespace po
