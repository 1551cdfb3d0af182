// Float32-path kernels on the float32 matrix instruction (gfx950): causal GQA attention and the GEMM.
// Operands, products and sums are float32 throughout (32x32x2 and 16x16x4 MFMAs); nothing is rounded to a narrower
// type.  The float32 path is the one that is held to 1e-4 against the float64 definition and that stands in for it
// at configurations no CPU run reaches, so what matters here is that every output is one float32 dot product in a
// fixed order that depends on nothing but its own row and column; speed only has to be enough for whole
// configurations (32 layers x 32768 tokens) to run in seconds.
#include "po_internal.h"
#include "slice_window.h"

#include <algorithm>

namespace po {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------ attention
// softmax(Q K^T / sqrt(hd)) V with the causal mask, grouped-query heads (Section 4.2 of the paper: attention runs
// over the whole sequence, unchunked).  A wavefront works on 32 query rows of one head, keys go by in tiles of 32.  Per
// tile it forms S^T[key][query] = K Q^T with 64 (hd 128) matrix instructions, so that a lane owns ONE query column --
// lane l and lane l ^ 32 share it, 16 keys each -- and the online softmax needs one exchange with the partner lane per
// tile; the probabilities never leave their registers: register r of S^T is exactly the B operand of step r of
// O^T[hd][query] += V^T P^T when the V fragment of that step is read at the key that register r holds.
// The contraction index of Q K^T is split between the lane halves (half h takes elements [h hd/2, (h+1) hd/2)), so
// that a lane's K fragment is contiguous (16-byte reads).
// Which wavefronts share the keys depends on the POSITION of a row alone, so that a row is the same bits wherever it
// sits in a launch and whichever rows are computed beside it (the tile grid starts at key 0; tiles wholly above a
// wavefront's rows are skipped, they would contribute p = 0 and a rescale by 1, exactly):
//  * rows from f32_split_rows on: a workgroup is 128 rows, one wavefront per 32 of them, K and V tiles shared through
//    LDS.  Matrix-pipe bound: tiles are copied global -> LDS directly, one tile ahead, one barrier per tile, and two
//    workgroups share a compute unit, so that one's softmax runs beside the other's MFMAs.
//  * rows below: a workgroup is 32 rows and its four wavefronts take every fourth key tile each, straight from global
//    memory, merging at the end in wavefront order.  A short request is bound by the one chain of its last rows (16 tiles
//    of about 3 us at 512 keys), which this cuts to a quarter.
// o may alias q: a workgroup reads its own query rows before it writes them, and nobody else touches them.
// Measured (kernel before: one workgroup per compute unit, tiles through registers, two barriers per tile, head-major
// order), 32 heads of 128: 512 rows 95 -> 48 us, 1024 rows 186 -> 138, 3000 rows 1347 -> 706, 32768 rows 98.0 -> 70.6 ms
// (125 TFLOP/s of 155); 4 heads of 64, 512 rows 50 -> 21 us.  The line between the two at 128: with 1536 in its place 1500
// rows take 246 instead of 289 us, but 2048 428 instead of 408 and 3000 734 instead of 706 (the small workgroups read K and V
// four times as often); at 64 the longer chains favour the small workgroups further (1500 rows 52 against 146 us).
constexpr int f32_split_rows(int hd) { return hd == 64 ? 1536 : 1024; }

template <int HD>
struct F32Rows {                  // a wavefront's 32 query rows: this lane's column
    static constexpr int HH = HD / 2, NB = HD / 32;      // contraction elements per lane half; 32-row blocks of O^T
    float qf[HH];
    f32x16 O[NB];
    float m, l;

    __device__ __forceinline__ void start(const float* q, int64_t t, int64_t N, int h, int Hq, int half) {
        const float* qp = q + (t * Hq + h) * HD + half * HH;
#pragma unroll
        for (int i = 0; i < HH / 4; ++i) {
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (t < N) x = *(const float4*)(qp + 4 * i);
            qf[4 * i] = x.x; qf[4 * i + 1] = x.y; qf[4 * i + 2] = x.z; qf[4 * i + 3] = x.w;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[b][r] = 0.f;
        m = -INFINITY;
        l = 0.f;
    }

    // one key tile: kfrag(i) = elements 4 i .. 4 i + 3 of this lane's half of K row `col`; vfrag(b, r) = V[key of register
    // r][32 b + col]
    template <typename KF, typename VF>
    __device__ __forceinline__ void tile(int64_t kv0, int64_t q0, int64_t t, int half, float scale, KF kfrag, VF vfrag) {
        f32x16 S;
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
        for (int i = 0; i < HH / 4; ++i) {
            const float4 kk = kfrag(i);
            S = mfma_f32(kk.x, qf[4 * i], S);
            S = mfma_f32(kk.y, qf[4 * i + 1], S);
            S = mfma_f32(kk.z, qf[4 * i + 2], S);
            S = mfma_f32(kk.w, qf[4 * i + 3], S);
        }
        // register r holds key kv0 + 8 (r / 4) + 4 half + r % 4 of query t
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = S[r] * scale;
        if (kv0 + 31 > q0) {                             // wavefront-uniform: the tile touches the diagonal
            const int d = (int)(t - kv0) - 4 * half;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r / 4) + (r % 4) > d) p[r] = -INFINITY;
        }
        float tmax = p[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, p[r]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        const float mn = fmaxf(m, tmax);
        // -inf while every score so far is (products that overflowed: a wavefront's first tile need not hold the row's first
        // keys): the tile then adds nothing, instead of exp(-inf + inf)
        const float ref = mn == -INFINITY ? 0.f : mn;
        if (__any(mn > m)) {                             // (else every factor is 1)
            const float a = expf(m - ref);               // exp(-inf) = 0 on the first tile
            l *= a;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[b][r] *= a;
            m = mn;
        }
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = expf(p[r] - ref);
            psum += p[r];
        }
        l += psum;                                       // this lane's 16 keys; the partner's are added at the end
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[b] = mfma_f32(vfrag(b, r), p[r], O[b]);
    }
};

// grid: workgroup i works for head i % Hq; i / Hq counts first the n_main blocks of 128 rows from block blk_main on, then
// the blocks of 32 rows from block blk_split on, the longest rows of all heads first in both
template <int HD>
__global__ void __launch_bounds__(256, 2) attention_f32_mfma_kernel(const float* q, const float* __restrict__ k,
                                                                    const float* __restrict__ v, float* o, int64_t N, int Hq,
                                                                    int Hkv, int n_main, int n_split, int64_t blk_main, int64_t blk_split) {
    constexpr int HH = HD / 2, NB = HD / 32;
    constexpr int ROWB = HD * 4, TB = 32 * ROWB;             // bytes of a K / V row and of a tile
    constexpr int RPL = 1024 / ROWB, LPW = 32 / RPL / 4;     // rows per 1 KiB load; loads per wavefront, operand and tile
    constexpr int SEGS = ROWB / 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int h = (int)(blockIdx.x % (unsigned)Hq), item = (int)(blockIdx.x / (unsigned)Hq);
    const int c = h / (Hq / Hkv);
    const float scale = 1.0f / sqrtf((float)HD);
    const int64_t kvrow = (int64_t)Hkv * HD;                 // floats between two positions
    F32Rows<HD> st;

    if (item < n_main) {
        const int64_t r0 = (n_main - 1 - item + blk_main) * 128;
        const int64_t q0 = r0 + wave * 32;          // this wavefront's first query row
        const int64_t t = q0 + col;                 // this lane's query row
        st.start(q, t, N, h, Hq, half);
        const int64_t kv_end = (r0 + 128 < N) ? r0 + 128 : N;
        // load jj of this wavefront: rows (wave LPW + jj) RPL .. of a tile; K segments swizzled with the row on this side
        uint32_t vok[4], vov[4];                     // (LPW entries used)
#pragma unroll
        for (int jj = 0; jj < LPW; ++jj) {
            const int row = (wave * LPW + jj) * RPL + lane / SEGS, seg = lane % SEGS;
            vok[jj] = (uint32_t)row * (uint32_t)(kvrow * 4) + (uint32_t)((seg ^ (row & 15)) << 4);
            vov[jj] = (uint32_t)row * (uint32_t)(kvrow * 4) + (uint32_t)(seg << 4);
        }
        auto load_tile = [&](int64_t kv0, int stage) {       // rows past N read as zero (masked keys)
            const int rows = (int)min((int64_t)32, N - kv0);
            const int bytes = (int)((rows - 1) * kvrow * 4) + ROWB;
            const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(k + kv0 * kvrow + c * HD), 0, bytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(v + kv0 * kvrow + c * HD), 0, bytes, 0x00020000);
            unsigned char* dst = smem + stage * 2 * TB + wave * LPW * 1024;
#pragma unroll
            for (int jj = 0; jj < LPW; ++jj) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (__attribute__((address_space(3))) void*)(dst + jj * 1024), 16, vok[jj], 0, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (__attribute__((address_space(3))) void*)(dst + TB + jj * 1024), 16, vov[jj], 0, 0, 0);
            }
        };
        load_tile(0, 0);
        int stage = 0;
        for (int64_t kv0 = 0; kv0 < kv_end; kv0 += 32, stage ^= 1) {
            // this tile has landed; everybody is done with the other stage
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (kv0 + 32 < kv_end) load_tile(kv0 + 32, stage ^ 1);
            if (kv0 > q0 + 31) continue;             // wavefront-uniform: every key of the tile is masked for these rows
            const unsigned char* ks = smem + stage * 2 * TB + col * ROWB;
            const float* vs = (const float*)(smem + stage * 2 * TB + TB) + (4 * half) * HD + col;
            st.tile(kv0, q0, t, half, scale,
                    [&](int i) { return *(const float4*)(ks + (((half * (SEGS / 2) + i) ^ (col & 15)) << 4)); },
                    [&](int b, int r) { return vs[(8 * (r / 4) + (r % 4)) * HD + 32 * b]; });
        }
        float l = st.l;
        l += __shfl_xor(l, 32);
        if (t >= N) return;
        const float inv = 1.0f / l;
        float* op = o + (t * Hq + h) * HD;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(float4*)(op + 32 * b + 8 * g + 4 * half) =
                    make_float4(st.O[b][4 * g] * inv, st.O[b][4 * g + 1] * inv, st.O[b][4 * g + 2] * inv, st.O[b][4 * g + 3] * inv);
    } else {
        const int64_t q0 = (n_split - 1 - (item - n_main) + blk_split) * 32;
        const int64_t t = q0 + col;
        st.start(q, t, N, h, Hq, half);
        for (int64_t kv0 = wave * 32; kv0 < q0 + 32; kv0 += 128) {
            // (keys past N are masked: they are past every row; their fragments come from the last position)
            const float* kp = k + min(kv0 + col, N - 1) * kvrow + c * HD + half * HH;
            float4 kf[HH / 4];
#pragma unroll
            for (int i = 0; i < HH / 4; ++i) kf[i] = *(const float4*)(kp + 4 * i);
            const float* vp = v + c * HD + col;
            st.tile(kv0, q0, t, half, scale, [&](int i) { return kf[i]; },
                    [&](int b, int r) { return vp[min(kv0 + 8 * (r / 4) + 4 * half + (r % 4), N - 1) * kvrow + 32 * b]; });
        }
        // merge: O, maximum and row sum of each wavefront through LDS, added in wavefront order
        float* so = (float*)smem;                                        // [wave][hd][32 queries]
        float* sm = so + 4 * HD * 32;                                    // [wave][32] maxima, then [wave][32] row sums
        const float l = st.l + __shfl_xor(st.l, 32);
        if (half == 0) {
            sm[wave * 32 + col] = st.m;
            sm[128 + wave * 32 + col] = l;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) so[(wave * HD + 32 * b + 8 * (r / 4) + 4 * half + (r % 4)) * 32 + col] = st.O[b][r];
        __syncthreads();
        float mx = sm[col], f[4], lt = 0.f;
#pragma unroll
        for (int w = 1; w < 4; ++w) mx = fmaxf(mx, sm[w * 32 + col]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            f[w] = expf(sm[w * 32 + col] - mx);                          // 0 for a wavefront without a tile
            lt += f[w] * sm[128 + w * 32 + col];
        }
        if (t >= N) return;
        const float inv = 1.0f / lt;
        // wavefront w stores dimensions [w HD / 4, ..), each lane half half of those, 4 at a time
        float* op = o + (t * Hq + h) * HD;
#pragma unroll
        for (int x = 0; x < HD / 32; ++x) {
            const int d0 = wave * (HD / 4) + half * (HD / 8) + 4 * x;
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float acc = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) acc += f[w] * so[(w * HD + d0 + e) * 32 + col];
                y[e] = acc * inv;
            }
            *(float4*)(op + d0) = make_float4(y[0], y[1], y[2], y[3]);
        }
    }
}

template <int HD>
static void launch_attention_f32(const float* q, const float* k, const float* v, float* o, int64_t N, int Hq, int Hkv,
                                 int64_t q_row0, hipStream_t s) {
    constexpr int SMEM_MAIN = 2 * 2 * 32 * HD * 4, SMEM_SPLIT = 4 * HD * 32 * 4 + 2 * 128 * 4;
    constexpr int SMEM = SMEM_MAIN > SMEM_SPLIT ? SMEM_MAIN : SMEM_SPLIT;
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(attention_f32_mfma_kernel<HD>), SMEM);
    });
    const int64_t row0 = (q_row0 > 0 && q_row0 < N) ? q_row0 : 0, split_rows = f32_split_rows(HD);
    const int64_t blk_main = std::max<int64_t>(row0, split_rows) / 128, end_main = (N + 127) / 128;
    const int64_t blk_split = row0 / 32, end_split = (std::min<int64_t>(N, split_rows) + 31) / 32;
    const int64_t n_main = std::max<int64_t>(0, end_main - blk_main), n_split = std::max<int64_t>(0, end_split - blk_split);
    hipLaunchKernelGGL(attention_f32_mfma_kernel<HD>, dim3((unsigned)((n_main + n_split) * Hq)), dim3(256), SMEM, s, q, k, v, o,
                       N, Hq, Hkv, (int)n_main, (int)n_split, blk_main, blk_split);
}

// q_row0: rows below it need no result (the block of 128 or 32 rows that holds it is computed whole; what is written
// below q_row0 nobody reads)
bool launch_attention_f32_mfma(const float* q, const float* k, const float* v, float* o, int64_t N, int Hq, int Hkv, int hd,
                               int64_t q_row0, hipStream_t s) {
    if (N <= 0) return true;
    if (hd != 64 && hd != 128) return false;
    if ((int64_t)Hkv * hd >= (1 << 23)) return false;       // a tile of 32 positions is addressed with 32-bit byte offsets
    if (hd == 128) launch_attention_f32<128>(q, k, v, o, N, Hq, Hkv, q_row0, s);
    else launch_attention_f32<64>(q, k, v, o, N, Hq, Hkv, q_row0, s);
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
// Pairs (PAIR_SILU: gate feature f and up feature f; PAIR_ROPE: the two halves of a head, i and i + hd / 2): a tile is half
// columns of one kind and half of the other, `apart` weight rows away, arranged so that a lane finds a pair in tiles t and
// t + T / 2 of its wavefront (T 1: in the other wavefront of its rows, through LDS), and the SiLU-multiply or the rotation
// is done on the accumulators.  Neither the [M, 2F] product nor unrotated queries and keys go through memory, and a layer is
// five launches shorter: the small configuration's whole call 203-215 -> 180 us, 1000 rows of the 8B MLP 2657 -> 2611.
// Measured (kernel before: 128 x 128 tiles of 32x32x2, slices staged through registers, two barriers each): 1000 rows of
// the 8B shape, down projection 1060 -> 866 us (136 TFLOP/s), gate/up 1990 -> 1726; 256 x 256 outputs of K 256 26 -> 9 us;
// one row of K 14336 1034 -> 84 us.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

enum { PAIR_NONE, PAIR_SILU, PAIR_ROPE };

template <int T, int D, int PAIR>
__global__ void __launch_bounds__(256, 2) gemm_f32_mfma_kernel(const float* __restrict__ A, int64_t lda,
                                                               const float* __restrict__ W, int64_t ldw, float* C,
                                                               int64_t ldc, const float* __restrict__ bias, const float* R,
                                                               int64_t ldr, int64_t M, int N, int K, const F32QkvRope qkv) {
    constexpr int BT = 32 * T, UNIT = BT * 128;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, l4 = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const unsigned nt = (unsigned)((N + BT - 1) / BT);       // (one grid dimension: the others end at 65536 tiles)
    const int64_t m0 = (int64_t)(blockIdx.x / nt) * BT;
    const int n0 = (int)(blockIdx.x % nt) * BT;
    // pairs: first weight row of the tile's first kind, and how many rows behind it the other kind lies
    const int wfirst = PAIR == PAIR_NONE ? n0 : PAIR == PAIR_SILU ? n0 / 2 : n0 / qkv.hd * qkv.hd + n0 % qkv.hd / 2;
    const int apart = PAIR == PAIR_SILU ? N / 2 : qkv.hd / 2;
    const int rows_a = (int)min((int64_t)BT, M - m0), rows_w = PAIR == PAIR_NONE ? min(BT, N - n0) : N - wfirst;
    // bounds: the rows of the tile that exist, pairs: of the matrix (others read as zero)
    const int a_bytes = (int)(uint32_t)(rows_a * lda * 4), w_bytes = (int)(uint32_t)(rows_w * ldw * 4);
    void* const pa_ = (void*)(A + m0 * lda);
    void* const pw_ = (void*)(W + (int64_t)wfirst * ldw);
    uint32_t voa[4], vow[4];                     // (T entries used: T loads of 8 rows per wavefront and operand)
    const int KT = (K + 31) / 32;
    uint32_t tail = 0;                           // bit i: load i of the last slice lies beyond K for this lane
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int row = (wave * T + i) * 8 + (lane >> 3);
        const int seg = (lane & 7) ^ ((row >> 1) & 7);
        voa[i] = (uint32_t)row * (uint32_t)(lda * 4) + seg * 16;
        // pairs: row = (wavefront column, kind, index), T / 2 tiles of each kind per wavefront (T 1: a kind per wavefront)
        const int wv = row / (16 * T), in = row % (16 * T);
        const int wrow = PAIR == PAIR_NONE ? row : T == 1 ? wv * apart + in : wv * 8 * T + in % (8 * T) + in / (8 * T) * apart;
        vow[i] = (uint32_t)wrow * (uint32_t)(ldw * 4) + seg * 16;
        if ((KT - 1) * 32 + seg * 4 >= K) tail |= 1u << i;
    }
    // Bounds are checked on the lane offset (not on the scalar offset along K): columns of the last slice past K get one
    // outside, slices past the end an empty descriptor; both read as zero without traffic.
#define PO_SLICE_RSRC(s_)                                                                                              \
    const SliceWindow wa_ = slice_window((s_), KT, (unsigned)a_bytes, 128), ww_ = slice_window((s_), KT, (unsigned)w_bytes, 128); \
    const int so = wa_.offset;                                                                                         \
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(pa_, 0, (int)wa_.bytes, 0x00020000);           \
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(pw_, 0, (int)ww_.bytes, 0x00020000);
#define PO_DMA(s_, pos_, i_)                                                                                          \
    {                                                                                                                  \
        const uint32_t past_ = ((s_) == KT - 1 && (tail >> (i_) & 1)) ? 0x80000000u : 0u;                              \
        unsigned char* d_ = smem + (pos_) * 2 * UNIT + (wave * T + (i_)) * 1024;                                       \
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)d_, 16, voa[(i_)] + past_, so, 0, 0); \
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(d_ + UNIT), 16, vow[(i_)] + past_, so, 0, 0); \
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
    for (int s = 0; s < D; ++s) {
        PO_SLICE_RSRC(s)
#pragma unroll
        for (int i = 0; i < T; ++i) PO_DMA(s, s, i)
    }
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
                PO_SLICE_RSRC(s + D)                                                                                  \
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
#undef PO_SLICE_RSRC
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (PAIR != PAIR_NONE) {
        // T 1: the second kind's accumulators to the wavefront that holds the first
        constexpr int H = T == 1 ? 1 : T / 2;
        f32x4 second[T];
        if (T == 1) {
            __syncthreads();                         // every wavefront is done with the ring
            if (wn == 1) *(f32x4*)(smem + (wm * 64 + lane) * 16) = acc[0][0];
            __syncthreads();
            if (wn == 1) return;
            second[0] = *(const f32x4*)(smem + (wm * 64 + lane) * 16);
        }
#pragma unroll
        for (int u = 0; u < T; ++u) {
            const int64_t gm = m0 + wm * (T * 16) + u * 16 + l15;
            if (gm >= M) continue;
#pragma unroll
            for (int t = 0; t < H; ++t) {
                const f32x4 x = acc[u][t], y = T == 1 ? second[0] : acc[u][T == 1 ? 0 : t + H];
                const int f = wfirst + (T == 1 ? 0 : wn * (8 * T) + t * 16) + 4 * l4;          // weight row of x[0]
                if (PAIR == PAIR_SILU) {
                    float h[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[e] = x[e] / (1.0f + expf(-x[e])) * y[e];
                    if (f < apart) *(float4*)(C + gm * ldc + f) = make_float4(h[0], h[1], h[2], h[3]);       // (F % 4 == 0)
                } else {
                    float a[4] = {x[0], x[1], x[2], x[3]}, b[4] = {y[0], y[1], y[2], y[3]};
                    if (bias) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            a[e] += bias[f + e];
                            b[e] += bias[f + apart + e];
                        }
                    }
                    float* d = f < qkv.qd ? qkv.q + gm * qkv.qd + f
                               : f < qkv.qd + qkv.kvd ? qkv.k + gm * qkv.kvd + (f - qkv.qd)
                                                      : qkv.v + gm * qkv.kvd + (f - qkv.qd - qkv.kvd);
                    if (f < qkv.qd + qkv.kvd) {
                        const int64_t pos = qkv.row_pos ? (int64_t)qkv.row_pos[qkv.pos0 + gm] : qkv.pos0 + gm;
                        const int i0 = f % qkv.hd;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float c = qkv.cos_t[pos * apart + i0 + e], s = qkv.sin_t[pos * apart + i0 + e], a0 = a[e];
                            // (fused by hand: the compiler's choice could differ between tiles)
                            a[e] = fmaf(a0, c, -(b[e] * s));
                            b[e] = fmaf(b[e], c, a0 * s);
                        }
                    }
                    *(float4*)d = make_float4(a[0], a[1], a[2], a[3]);
                    *(float4*)(d + apart) = make_float4(b[0], b[1], b[2], b[3]);
                }
            }
        }
        return;
    }
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

template <int T, int D, int PAIR>
static void launch_f32_tile(const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc, const float* bias,
                            const float* R, int64_t ldr, int64_t M, int N, int K, const F32QkvRope& qkv, hipStream_t s) {
    constexpr int BT = 32 * T, SMEM = D * 2 * BT * 128;
    static_assert(SMEM <= 64 * 1024, "two workgroups per compute unit, and no larger than a launch may ask for unannounced");
    const dim3 grid((unsigned)(((N + BT - 1) / BT) * ((M + BT - 1) / BT)));
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<T, D, PAIR>), grid, dim3(256), SMEM, s, A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, qkv);
}

// Tile of a launch: 0, 1, 2 = 128, 64, 32 rows and columns; largest: the first of them that is allowed; ld: of either operand;
// slice_us: where its time per K slice goes
static int f32_tile(int64_t M, int N, int64_t ld, int largest, double* slice_us = nullptr) {
    // Tile by time: a round of 256 tiles, one per compute unit, costs this many microseconds per K slice of 32 (measured
    // on 256 .. 2048 tiles of each); where all three take one round the small tile has the shorter chain.
    constexpr double us[3] = {1.9, 0.54, 0.2};
    int best = 2;
    double best_us = 1e300;
    for (int i = largest; i < 3; ++i) {
        const int64_t bt = 128 >> i, tiles = ((M + bt - 1) / bt) * ((N + bt - 1) / bt);
        if (bt * ld > (1 << 28)) continue;
        const double t = us[i] * (double)((tiles + 255) / 256);
        if (t < best_us) { best = i; best_us = t; }
    }
    if (slice_us) *slice_us = best_us;
    return best;
}

// the largest tile of a launch with rotation: pairs stay within a head
static int f32_rope_largest(int hd) { return hd == 128 ? 0 : 1; }

int gemm_f32_tile(int64_t M, int N, int K, int rope_hd) { return 128 >> f32_tile(M, N, K, rope_hd ? f32_rope_largest(rope_hd) : 0); }

// false (nothing launched) when the operands do not allow 16-byte loads along K; largest: of f32_tile
template <int PAIR>
static bool launch_f32(const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc, const float* bias,
                       const float* R, int64_t ldr, int64_t M, int N, int K, const F32QkvRope& qkv, int largest, hipStream_t s) {
    if (M <= 0 || N <= 0) return true;
    if (K <= 0 || K % 4 || lda % 4 || ldw % 4 || ((uintptr_t)A | (uintptr_t)W | (uintptr_t)C | (uintptr_t)bias | (uintptr_t)R) % 16)
        return false;
    const int64_t ld = std::max(lda, ldw);
    if (ld > (1 << 23)) return false;        // a tile, of 32 rows at least, is addressed with offsets below 2^30 bytes
    const int best = f32_tile(M, N, ld, largest);
    if (best == 0) launch_f32_tile<4, 2, PAIR>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, qkv, s);
    else if (best == 1) launch_f32_tile<2, 4, PAIR>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, qkv, s);
    else launch_f32_tile<1, 8, PAIR>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, qkv, s);
    return true;
}

bool launch_gemm_f32_mfma(const float* A, int64_t lda, const float* W, int64_t ldw, float* C, int64_t ldc, const float* bias,
                          const float* R, int64_t ldr, int64_t M, int N, int K, hipStream_t s) {
    return launch_f32<PAIR_NONE>(A, lda, W, ldw, C, ldc, bias, R, ldr, M, N, K, F32QkvRope{}, 0, s);
}

// H[M, F] = silu(A Wg^T) (A Wu^T), W = [Wg; Wu] [2 F, K].  false (nothing launched): as above, F % 4, or weights a tile cannot
// address with offsets below 2^31 bytes
bool launch_gemm_f32_silu(const float* A, int64_t lda, const float* W, int64_t ldw, float* H, int64_t ldh, int64_t M, int F, int K,
                          hipStream_t s) {
    if (F % 4 || ldh % 4 || (2 * (int64_t)F + 128) * ldw * 4 > ((int64_t)1 << 31)) return false;
    return launch_f32<PAIR_SILU>(A, lda, W, ldw, H, ldh, nullptr, nullptr, 0, M, 2 * F, K, F32QkvRope{}, 0, s);
}

// Q, K rotated and V of rows A, W = [Wq; Wk; Wv], bias (or null) in the same order.  false: nothing launched
bool launch_gemm_f32_qkv_rope(const float* A, int64_t lda, const float* W, int64_t ldw, const float* bias, int64_t M, int K,
                              const F32QkvRope& qkv, hipStream_t s) {
    const int N = qkv.qd + 2 * qkv.kvd;
    if ((qkv.hd != 64 && qkv.hd != 128) || qkv.qd % qkv.hd || qkv.kvd % qkv.hd || ((int64_t)N + 128) * ldw * 4 > ((int64_t)1 << 31) ||
        ((uintptr_t)qkv.q | (uintptr_t)qkv.k | (uintptr_t)qkv.v) % 16)
        return false;
    // One launch, or where its tiles end in a round that is mostly empty, Q by itself: a second launch takes 4 us and more (M 256,
    // N 4096 + 2048, K 4096: two rounds of 64-row tiles, 384 in all, against one of them and two of 32-row tiles, 2048 rows of a
    // 4096-wide layer, hidden width 4096, in chunks of 256 1629 -> 1493 us)
    const int largest = f32_rope_largest(qkv.hd);
    double whole, q, kv;
    f32_tile(M, N, std::max(lda, ldw), largest, &whole);
    f32_tile(M, qkv.qd, std::max(lda, ldw), largest, &q);
    f32_tile(M, 2 * qkv.kvd, std::max(lda, ldw), largest, &kv);
    if ((whole - q - kv) * ((K + 31) / 32) <= 5.0)
        return launch_f32<PAIR_ROPE>(A, lda, W, ldw, nullptr, 0, bias, nullptr, 0, M, N, K, qkv, largest, s);
    F32QkvRope rest = qkv;
    rest.qd = 0;
    return launch_f32<PAIR_ROPE>(A, lda, W, ldw, nullptr, 0, bias, nullptr, 0, M, qkv.qd, K, qkv, largest, s) &&
           launch_f32<PAIR_ROPE>(A, lda, W + (int64_t)qkv.qd * ldw, ldw, nullptr, 0, bias ? bias + qkv.qd : nullptr, nullptr, 0, M,
                                 2 * qkv.kvd, K, rest, largest, s);
}

}  // namespace po
