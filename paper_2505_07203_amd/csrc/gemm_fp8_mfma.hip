// FP8 (OCP E4M3) MFMA GEMM for the FP8-dynamic variant of the position-wise linear layers (gfx950).
//
//   C[M, N] = (Qa[M, K] * Qw[N, K]^T) * sa[M] * sw[N]      codes one byte each, K-contiguous rows;
//                                                          sa: one scale per token, sw: per output feature
//
// The same design as the bf16 kernel (256 x 256 block, 4 wavefronts x 128 x 128 patch, five-unit LDS
// ring of 32 KiB units filled by buffer_load ... lds, XCD-aware tile order, shared epilogues): a row of a
// unit is again one 128-byte line, which now holds 128 codes, so a slice is 128 k and feeds two k-steps of
// the 32x32x64 MFMA (twice the flops per byte moved, per LDS read and per cycle of the matrix pipe).  A
// fragment is 32 bytes per lane: two 16-byte reads.  The products accumulate in fp32; the scales are
// applied to the accumulators before the (unchanged) epilogue arithmetic.
#include "gemm_common.h"

#include <string.h>

namespace po {

typedef __attribute__((__vector_size__(8 * sizeof(int)))) int i32x8;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

namespace {

using namespace gemm;

constexpr int BKB = 128;                           // bytes (= codes) of K per slice
constexpr int UNIT_BYTES = BM * BKB;               // one operand's slice: 256 rows x 128 bytes = 32 KiB
constexpr int NUNIT = 5;
constexpr int SMEM_BYTES = NUNIT * UNIT_BYTES;

#define PO_HANDOVER() asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory")

template <int EPI>
__global__ void __launch_bounds__(NTHREADS) gemm_fp8_mfma_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // ---- XCD-aware tile assignment
    const int total = p.mt * p.nt;
    const int per_xcd = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int li = xcd * per_xcd + local;
    if (local >= per_xcd || li >= total) return;
    const int group_sz = GROUP_M * p.nt;
    const int g = li / group_sz;
    const int within = li - g * group_sz;
    const int gm_this = min(GROUP_M, p.mt - g * GROUP_M);
    const int tn = within / gm_this;
    const int tm = g * GROUP_M + (within - tn * gm_this);
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, lhi = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;

    // ---- global -> LDS map.  A unit (one operand's 256 rows x 64 k) is 32 one-KiB loads; wavefront w issues
    // loads w*8 .. w*8+7, load q fills rows q*8 .. q*8+7: lane l -> row q*8 + l/8, physical segment l & 7,
    // which holds logical segment (l & 7) ^ ((row >> 1) & 7).  Eight lanes fetch one whole 128-byte line.
    // Each operand is addressed through a buffer resource that starts at the tile's first row and ends with
    // the matrix: the per-lane byte offset never changes, the slice offset is one scalar, and rows of a
    // ragged last tile beyond the matrix read as zero instead of needing a clamp (they are never stored).
    // (split-K launches: workgroup row blockIdx.y works on codes [k0, k0 + K) of both operands)
    const int64_t k0 = (EPI == EPI_PARTIAL) ? (int64_t)blockIdx.y * p.K : 0;
    const uint64_t a_bytes = (uint64_t)(p.M - m0) * (uint64_t)p.lda - (uint64_t)k0, w_bytes = (uint64_t)(p.N - n0) * (uint64_t)p.ldw - (uint64_t)k0;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const unsigned char*)p.A + (int64_t)m0 * p.lda + k0), 0, (int)(uint32_t)(a_bytes > 0xffffffffull ? 0xffffffffull : a_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const unsigned char*)p.W + (int64_t)n0 * p.ldw + k0), 0, (int)(uint32_t)(w_bytes > 0xffffffffull ? 0xffffffffull : w_bytes), 0x00020000);
    uint32_t voa[8], vow[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = wave * 64 + i * 8 + (lane >> 3);
        const int lseg = (lane & 7) ^ ((row >> 1) & 7);
        voa[i] = (uint32_t)row * (uint32_t)p.lda + lseg * 16;
        vow[i] = (uint32_t)row * (uint32_t)p.ldw + lseg * 16;
    }
    const int KT = p.K / BKB;
    // load i_ (0..7) of this wavefront's share of unit u_ (even: activations of slice u_/2, odd: weights)
    // into ring position pos_
#define PO_DMA(u_, pos_, i_)                                                                                  \
    {                                                                                                         \
        const int t_ = min((u_) >> 1, KT - 1);                                                                \
        unsigned char* sa_ = smem + (pos_) * UNIT_BYTES + wave * 8192 + (i_) * 1024;                          \
        __builtin_amdgcn_raw_ptr_buffer_load_lds((u_) & 1 ? rw : ra, (__attribute__((address_space(3))) void*)sa_, 16, \
                                                 (u_) & 1 ? vow[(i_)] : voa[(i_)], t_ * BKB, 0, 0);      \
    }

    f32x16 acc[4][4];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    // fragment read offsets: row l31 of a 32-row tile; k-step kk (64 codes) of its 128 bytes: a lane takes the
    // 32 bytes of logical segments kk*4 + lhi*2 and + 1 (two 16-byte reads); one lane register per k-step,
    // segment, operand and 64 KiB of LDS, the rest of an address is an immediate below 64 KiB
    int a_off[3][2][2], w_off[3][2][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const int fo = l31 * 128 + (((kk * 4 + lhi * 2 + h2) ^ ((l31 >> 1) & 7)) << 4);
#pragma unroll
            for (int hb = 0; hb < 3; ++hb) {
                a_off[hb][kk][h2] = hb * 65536 + wm * 16384 + fo;
                w_off[hb][kk][h2] = hb * 65536 + wn * 16384 + fo;
            }
        }

    // Software pipeline inside the wavefront, as in the bf16 kernel: memory instructions are issued one or
    // two at a time between MFMAs (a 32x32x64 MFMA keeps the pipe busy for 64 cycles).  A slice is two blocks
    // of 16 MFMA, one per k-step of 64 codes; a block also reads the 8 fragments (16 reads) of the next k-step
    // on its first 8 MFMAs and issues 8 loads on the other 8:
    //   block 0 of slice s: fragments of (s, k-step 1); the 8 loads of activation unit s+2
    //   hand-over barrier:  slice s+1 has landed; nobody reads slice s's units any more
    //   block 1 of slice s: fragments of (s+1, k-step 0); the 8 loads of weight unit s+2, into the
    //                       position slice s's activations occupied (unit u lives at u mod 5)
    // At the hand-over the loads issued after those of slice s+1 are the 8 of activation unit s+2.
    i32x8 af0[4], wf0[4], af1[4], wf1[4];
#define PO_FRAG1(AF, WF, pa_, pw_, kk_, j_)                                                          \
    {                                                                                               \
        if ((j_) < 4) {                                                                             \
            const i32x4 lo_ = *(const i32x4*)(smem + a_off[(pa_) >> 1][kk_][0] + ((pa_) & 1) * UNIT_BYTES + ((j_) & 3) * 4096); \
            const i32x4 hi_ = *(const i32x4*)(smem + a_off[(pa_) >> 1][kk_][1] + ((pa_) & 1) * UNIT_BYTES + ((j_) & 3) * 4096); \
            AF[(j_) & 3] = __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7);               \
        } else {                                                                                    \
            const i32x4 lo_ = *(const i32x4*)(smem + w_off[(pw_) >> 1][kk_][0] + ((pw_) & 1) * UNIT_BYTES + ((j_) & 3) * 4096); \
            const i32x4 hi_ = *(const i32x4*)(smem + w_off[(pw_) >> 1][kk_][1] + ((pw_) & 1) * UNIT_BYTES + ((j_) & 3) * 4096); \
            WF[(j_) & 3] = __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7);               \
        }                                                                                           \
    }
    // E4M3 x E4M3 (format selectors 0, 0), block scales fixed at 2^0
#define PO_MFMA1(AF, WF, t_)                                                                        \
    acc[(t_) >> 2][(t_) & 3] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(                     \
        WF[(t_) & 3], AF[(t_) >> 2], acc[(t_) >> 2][(t_) & 3], 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
    // fragment read in slot t (order of first use: MFMA t needs AF[t >> 2] and WF[t & 3]), or -1
#define PO_READ_SLOT(t_) ((t_) == 0 ? 0 : (t_) >= 1 && (t_) <= 4 ? 3 + (t_) : (t_) >= 5 && (t_) <= 7 ? (t_) - 4 : -1)
    // one block: MFMAs on (AFc, WFc); reads k-step kkn_ of the slice at positions (pa_, pw_) into (AFn, WFn);
    // the 8 loads of unit u_ into position up_
#define PO_BLOCK(AFc, WFc, AFn, WFn, pa_, pw_, kkn_, u_, up_)                                         \
    _Pragma("unroll") for (int t = 0; t < 16; ++t) {                                                \
        PO_MFMA1(AFc, WFc, t);                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        if (PO_READ_SLOT(t) >= 0) {                                                                 \
            PO_FRAG1(AFn, WFn, pa_, pw_, kkn_, PO_READ_SLOT(t));                                    \
        } else {                                                                                    \
            PO_DMA(u_, up_, t - 8);                                                                 \
        }                                                                                           \
        __builtin_amdgcn_sched_barrier(0);                                                          \
    }
    // slice s_ whose number is j_ modulo 5 (a literal): its units sit at positions 2j mod 5 and 2j+1 mod 5
#define PO_SLICE(s_, j_)                                                                            \
    {                                                                                               \
        PO_BLOCK(af0, wf0, af1, wf1, (2 * (j_)) % 5, (2 * (j_) + 1) % 5, 1, 2 * (s_) + 4, (2 * (j_) + 4) % 5); \
        PO_HANDOVER();                                                                              \
        PO_BLOCK(af1, wf1, af0, wf0, (2 * (j_) + 2) % 5, (2 * (j_) + 3) % 5, 0, 2 * (s_) + 5, (2 * (j_)) % 5); \
    }
    // in flight when the first slice is awaited: units 0..3 (slices 0 and 1)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) PO_DMA(u, u, i);
    asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");     // slice 0 has landed
#pragma unroll
    for (int j = 0; j < 8; ++j) PO_FRAG1(af0, wf0, 0, 1, 0, j);
    int s = 0;
    for (; s + 5 <= KT; s += 5) {
        PO_SLICE(s, 0);
        PO_SLICE(s + 1, 1);
        PO_SLICE(s + 2, 2);
        PO_SLICE(s + 3, 3);
        PO_SLICE(s + 4, 4);
    }
    if (s < KT) { PO_SLICE(s, 0); ++s; }
    if (s < KT) { PO_SLICE(s, 1); ++s; }
    if (s < KT) { PO_SLICE(s, 2); ++s; }
    if (s < KT) { PO_SLICE(s, 3); ++s; }
#undef PO_SLICE
#undef PO_BLOCK
#undef PO_READ_SLOT
#undef PO_DMA
#undef PO_FRAG1
#undef PO_MFMA1
    // the clamped tail loads have landed and every wavefront has finished reading the ring
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // codes -> values: one scale per token row (this lane's) and one per output feature
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        const float sx = p.sa[min(m0 + wm * 128 + mi * 32 + l31, p.M - 1)];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int col = min(n0 + wn * 128 + ni * 32 + 8 * g4 + 4 * lhi, p.N - 4);
                const float4 sw = *(const float4*)(p.sw + col);
                acc[mi][ni][4 * g4] = acc[mi][ni][4 * g4] * sx * sw.x;
                acc[mi][ni][4 * g4 + 1] = acc[mi][ni][4 * g4 + 1] * sx * sw.y;
                acc[mi][ni][4 * g4 + 2] = acc[mi][ni][4 * g4 + 2] * sx * sw.z;
                acc[mi][ni][4 * g4 + 3] = acc[mi][ni][4 * g4 + 3] * sx * sw.w;
            }
    }
    if (EPI == EPI_PARTIAL) {
        GemmParams q = p;
        q.dst = (bf16_t*)((float*)p.dst + (int64_t)blockIdx.y * p.ldr);     // this split's plane of partial sums
        tile_epilogue<EPI, 4, 4>(q, acc, smem + wave * 8192, m0 + wm * 128, n0 + wn * 128, lane);
    } else {
        tile_epilogue<EPI, 4, 4>(p, acc, smem + wave * 8192, m0 + wm * 128, n0 + wn * 128, lane);
    }
}

// The same GEMM in small block tiles for launches of few 256 x 256 tiles (see the bf16 small kernel for what bounds
// them): 128 columns, four wavefronts 2 x 2, patches of 32 MR rows x 64 columns, a ring of D whole slices (as many as LDS
// holds).  With one workgroup per compute unit a wavefront has 512 registers, enough for the fragments of TWO whole
// slices beside the accumulators: a slice is multiplied from registers while the next one's fragments are read, so by
// the one barrier of a slice nobody needs its LDS position any more and slice s + D is loaded there.  (The same kernel
// on 16x16x128 MFMAs was up to 1.6 x slower: half as much work per fragment read.)  k-steps of 64 in order, as above: the
// same bits.  Measured: down projection (N 4096, K 14336) 471 rows 143 -> 48 us (46 with turns), 2048 rows (256-row tiles) 143 -> 99,
// 2.4 PFLOP/s.
template <int EPI, int MR, int D, bool TURNS>
__global__ void __launch_bounds__(256, 1) gemm_fp8_small_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int BM_ = 64 * MR, BN_ = 128;
    constexpr int AU = BM_ * BKB, WU = BN_ * BKB;          // bytes of a slice of A / W
    constexpr int NA = 2 * MR, NW = 4;                     // global->LDS loads per wavefront and slice
    constexpr int AHEAD = D + 4;                           // how far ahead of the multiplied slice weights are touched

    const int total = p.mt * p.nt;
    const int per_xcd = (total + 7) >> 3;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int li = xcd * per_xcd + local;
    if (local >= per_xcd || li >= total) return;
    constexpr int GM = 1024 / BM_;
    const int group_sz = GM * p.nt;
    const int g = li / group_sz;
    const int within = li - g * group_sz;
    const int gm_this = min(GM, p.mt - g * GM);
    const int tn = within / gm_this;
    const int tm = g * GM + (within - tn * gm_this);
    const int m0 = tm * BM_, n0 = tn * BN_;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, lhi = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int row_base = m0 + wm * (MR * 32), col_base = n0 + wn * 64;

    // the scales of this lane's accumulators: behind the K loop no MFMA would cover their latency
    float sx[MR];
    float4 sw[2][4];
#pragma unroll
    for (int mi = 0; mi < MR; ++mi) sx[mi] = p.sa[min(row_base + mi * 32 + l31, p.M - 1)];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) sw[ni][g4] = *(const float4*)(p.sw + min(col_base + ni * 32 + 8 * g4 + 4 * lhi, p.N - 4));

    // resources: the tile's rows that exist (rows beyond them read as zero), codes from k0 on
    const int64_t k0 = (EPI == EPI_PARTIAL) ? (int64_t)blockIdx.y * p.K : 0;
    const uint32_t a_bytes = (uint32_t)min(BM_, p.M - m0) * (uint32_t)p.lda - (uint32_t)k0;
    const uint32_t w_bytes = (uint32_t)min(BN_, p.N - n0) * (uint32_t)p.ldw - (uint32_t)k0;
    void* const pa_ = (void*)((const unsigned char*)p.A + (int64_t)m0 * p.lda + k0);
    void* const pw_ = (void*)((const unsigned char*)p.W + (int64_t)n0 * p.ldw + k0);
    uint32_t voa[8], vow[4];                               // (voa: NA entries used)
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = (wave * NA + i) * 8 + (lane >> 3);
        voa[i] = (uint32_t)row * (uint32_t)p.lda + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int row = (wave * NW + i) * 8 + (lane >> 3);
        vow[i] = (uint32_t)row * (uint32_t)p.ldw + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const int KT = p.K / BKB;
    // (descriptors empty past the end of K, as in the bf16 small kernel)
#define PO_SLICE_RSRC(s_)                                                                                              \
    const SliceWindow wa_ = slice_window((s_), KT, (unsigned)a_bytes, BKB), ww_ = slice_window((s_), KT, (unsigned)w_bytes, BKB); \
    const int so = wa_.offset;                                                                                         \
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(pa_, 0, (int)wa_.bytes, 0x00020000);           \
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(pw_, 0, (int)ww_.bytes, 0x00020000);
#define PO_DMA_A(pos_, i_)                                                                                               \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                            \
        ra, (__attribute__((address_space(3))) void*)(smem + (pos_) * (AU + WU) + (wave * NA + (i_)) * 1024), 16, voa[(i_)], so, 0, 0);
#define PO_DMA_W(pos_, i_)                                                                                               \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                            \
        rw, (__attribute__((address_space(3))) void*)(smem + (pos_) * (AU + WU) + AU + (wave * NW + (i_)) * 1024), 16,     \
        vow[(i_)], so, 0, 0);
    // a fragment: 32 rows from tile_ on, the 32 bytes of k-step kk_ a lane takes (two 16-byte segments, swizzled)
    int fo[2][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) fo[kk][h2] = l31 * 128 + (((kk * 4 + lhi * 2 + h2) ^ ((l31 >> 1) & 7)) << 4);
#define PO_FRAG(tile_, kk_)                                                                                           \
    __builtin_shufflevector(*(const i32x4*)((tile_) + fo[kk_][0]), *(const i32x4*)((tile_) + fo[kk_][1]), 0, 1, 2, 3, 4, 5, 6, 7)
    // (turns: as in the bf16 small kernel)
    unsigned char* const touched = smem + D * (AU + WU) + wave * 256;
    const uint32_t vot = (uint32_t)(wave * 32 + (lane & 31)) * (uint32_t)p.ldw + (lane >> 5) * BKB;
    int turn = gm_this > 1 ? (tm - g * GM) * 2 : 1 << 30;
#define PO_TOUCH(s_)                                                                                                   \
    if (TURNS) {                                                                                                       \
        if (turn == 0 && (s_) + 1 < KT) {                                                                              \
            const __amdgpu_buffer_rsrc_t rt_ = __builtin_amdgcn_make_buffer_rsrc(pw_, 0, (int)w_bytes, 0x00020000);    \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rt_, (__attribute__((address_space(3))) void*)touched, 4, vot, (s_) * (BKB), 0, 0); \
        }                                                                                                              \
        turn = turn == 0 ? 2 * gm_this - 1 : turn - 1;                                                                 \
    }
    const int a_base = wm * (MR * 32) * 128, w_base = AU + wn * 64 * 128;

    f32x16 acc[MR][2];
#pragma unroll
    for (int mi = 0; mi < MR; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
#pragma unroll
    for (int s = 0; s < D; ++s) {
        PO_SLICE_RSRC(s)
#pragma unroll
        for (int i = 0; i < NA; ++i) PO_DMA_A(s, i)
#pragma unroll
        for (int i = 0; i < NW; ++i) PO_DMA_W(s, i)
    }
    PO_WAIT_BARRIER((D - 1) * (NA + NW));                      // slice 0 has landed
#pragma unroll 1
    for (int s = D; s < AHEAD; ++s) { PO_TOUCH(s) }
    i32x8 A0[2][MR], W0[2][2], A1[2][MR], W1[2][2];            // fragments of a whole slice: [k-step][tile]
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int j = 0; j < 2; ++j) W0[kk][j] = PO_FRAG(smem + w_base + j * 4096, kk);
#pragma unroll
        for (int j = 0; j < MR; ++j) A0[kk][j] = PO_FRAG(smem + a_base + j * 4096, kk);
    }
    // slice s from registers (AC, WC); behind its 4 MR MFMAs the fragment reads of slice s + 1 and the loads of slice
    // s + D into the position of slice s, whose fragments every wavefront holds in registers by the barrier in front
#define PO_SLICE(AC, WC, AN, WN)                                                                                     \
    {                                                                                                                 \
        PO_WAIT_BARRIER((D - 2) * (NA + NW));      /* slice s+1 has landed; all LDS reads of slice s are done */      \
        const int ps1 = ps + 1 >= D ? 0 : ps + 1;                                                                     \
        PO_SLICE_RSRC(s + D)                                                                                          \
        PO_TOUCH(s + AHEAD)                                                                                           \
        const unsigned char* u1 = smem + ps1 * (AU + WU);                                                             \
        _Pragma("unroll") for (int m = 0; m < 4 * MR; ++m) {                                                          \
            const int kk_ = m / (2 * MR), mi_ = (m >> 1) % MR, ni_ = m & 1;                                           \
            acc[mi_][ni_] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(WC[kk_][ni_], AC[kk_][mi_], acc[mi_][ni_], 0, 0, 0, \
                                                                            0x7F7F7F7F, 0, 0x7F7F7F7F);               \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
            constexpr int F_ = 2 * (MR + 2), T_ = F_ + NA + NW;                                                       \
            _Pragma("unroll") for (int x = 0; x < T_; ++x) {                                                          \
                if (x >= m * T_ / (4 * MR) && x < (m + 1) * T_ / (4 * MR)) {                                          \
                    const int fk_ = x / (MR + 2) & 1, fj_ = x % (MR + 2);                                             \
                    if (x < F_ && fj_ < 2) WN[fk_][fj_ & 1] = PO_FRAG(u1 + w_base + fj_ * 4096, fk_);                 \
                    else if (x < F_) AN[fk_][fj_ >= 2 ? fj_ - 2 : 0] = PO_FRAG(u1 + a_base + (fj_ - 2) * 4096, fk_);  \
                    else if (x < F_ + NA) PO_DMA_A(ps, ((x - F_) & 7))                                            \
                    else PO_DMA_W(ps, ((x - F_ - NA) & 3))                                                        \
                    __builtin_amdgcn_sched_barrier(0);                                                                \
                }                                                                                                     \
            }                                                                                                         \
        }                                                                                                             \
        ps = ps1;                                                                                                     \
    }
    int ps = 0;                                  // ring position of slice s
    int s = 0;
    for (; s + 2 <= KT; ++s) {
        PO_SLICE(A0, W0, A1, W1)
        ++s;
        PO_SLICE(A1, W1, A0, W0)
    }
    if (s < KT) PO_SLICE(A0, W0, A1, W1)
#undef PO_SLICE
#undef PO_TOUCH
#undef PO_FRAG
#undef PO_DMA_A
#undef PO_DMA_W
#undef PO_SLICE_RSRC
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // codes -> values
#pragma unroll
    for (int mi = 0; mi < MR; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                acc[mi][ni][4 * g4] = acc[mi][ni][4 * g4] * sx[mi] * sw[ni][g4].x;
                acc[mi][ni][4 * g4 + 1] = acc[mi][ni][4 * g4 + 1] * sx[mi] * sw[ni][g4].y;
                acc[mi][ni][4 * g4 + 2] = acc[mi][ni][4 * g4 + 2] * sx[mi] * sw[ni][g4].z;
                acc[mi][ni][4 * g4 + 3] = acc[mi][ni][4 * g4 + 3] * sx[mi] * sw[ni][g4].w;
            }
    GemmParams q = p;
    if (EPI == EPI_PARTIAL) q.dst = (bf16_t*)((float*)p.dst + (int64_t)blockIdx.y * p.ldr);     // this split's plane
    if (col_base < p.N) tile_epilogue<EPI, MR, 2>(q, acc, smem + wave * 8192, row_base, col_base, lane);
}

// Block tiles of the FP8 launches (see TileForm), fitted to 208 shapes like the bf16 ones; on 255 others, with turns, the pick
// is on average 0.1 % and at most 5 % off the fastest form.  Measured, 256-row tiles against the pick: down projection (N 4096, K 14336) 1
// row 136 -> 41 us, 471 rows 143 -> 46, 1000 rows 141 -> 61, 2048 rows 143 -> 99; gate/up 150 rows 50 -> 34.
constexpr TileForm FORMS[] = {{256, 256, 10.0, 1.02, 1.54}, {64, 128, 3.0, 0.31, 0.41}, {128, 128, 4.6, 0.36, 0.59},
                              {192, 128, 6.3, 0.43, 0.73},  {256, 128, 7.7, 0.55, 0.90}};
constexpr TileForms TILES = {FORMS, sizeof(FORMS) / sizeof(FORMS[0]), BKB, 1};


template <int EPI>
void launch_256(const GemmParams& p, hipStream_t s, int splits) {
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(gemm_fp8_mfma_kernel<EPI>), SMEM_BYTES);
    });
    const int per_xcd = (p.mt * p.nt + 7) / 8;
    hipLaunchKernelGGL(gemm_fp8_mfma_kernel<EPI>, dim3((unsigned)(per_xcd * 8), (unsigned)splits), dim3(NTHREADS), SMEM_BYTES, s, p);
}

template <int EPI, int MR, int D, bool TURNS>
void launch_small_t(const GemmParams& p, hipStream_t s, int splits) {
    constexpr int SMEM = D * (64 * MR + 128) * BKB + (TURNS ? 1024 : 0);       // the ring; where touches go
    static_assert(SMEM <= 160 * 1024 && SMEM >= 4 * 8192, "LDS of a compute unit; staging of four wavefronts");
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(gemm_fp8_small_kernel<EPI, MR, D, TURNS>), SMEM);
    });
    const int per_xcd = (p.mt * p.nt + 7) / 8;
    hipLaunchKernelGGL((gemm_fp8_small_kernel<EPI, MR, D, TURNS>), dim3((unsigned)(per_xcd * 8), (unsigned)splits), dim3(256), SMEM,
                       s, p);
}

// Turns (see takes_turns of the bf16 kernels), for a launch of M rows in tiles of 64 mr rows, K per split.  Measured like those,
// on 355 launches, weights from HBM, time with turns against without: 64 rows per tile from five row tiles on, the last a quarter
// full, -13 to 0 %, but -4 to +8 with fewer than 40 slices, which end before a lead of ten pays; two to four row tiles -9 to +26;
// 128 rows with the last tile two fifths full -21 to 0, emptier -6 to +7; 192 rows, whose ring would be a slice shorter with turns,
// -10 to +4 with the last tile two thirds full, emptier -1 to +16, never taken; 256 rows -1 to +11, never.  K splits are no
// different (128 rows where taken -9 and -7).  Weights in the memory-side cache: 64 rows +10 to +30 where taken, 128 rows -5 to +10.
bool takes_turns(int mr, int64_t M, int K) {
    const int64_t rows = 64 * mr, mt = (M + rows - 1) / rows, last = M - (mt - 1) * rows;
    if (mr == 1) return mt >= 5 && 4 * last >= rows && K >= 40 * BKB;
    return mr == 2 && mt >= 3 && 5 * last >= 2 * rows;
}

// DT: ring depth with turns (a ring that fills the LDS leaves no room for where touches go)
template <int EPI, int MR, int D, int DT>
void launch_small(GemmParams p, hipStream_t s, int splits) {
    p.mt = (p.M + 64 * MR - 1) / (64 * MR);
    p.nt = (p.N + 127) / 128;
    if (MR <= 2 && !p.w_cached && takes_turns(MR, p.M, p.K)) launch_small_t<EPI, MR, MR <= 2 ? DT : D, MR <= 2>(p, s, splits);
    else launch_small_t<EPI, MR, D, false>(p, s, splits);
}

template <int EPI>
void launch_form(int form, const GemmParams& p, hipStream_t s, int splits = 1) {
    switch (form) {
        case 1: launch_small<EPI, 1, 6, 6>(p, s, splits); break;
        case 2: launch_small<EPI, 2, 5, 4>(p, s, splits); break;
        case 3: launch_small<EPI, 3, 4, 4>(p, s, splits); break;
        case 4: launch_small<EPI, 4, 3, 3>(p, s, splits); break;
        default: launch_256<EPI>(p, s, splits); break;
    }
}

template <int EPI>
void launch_t(const GemmParams& p, hipStream_t s) { launch_form<EPI>(pick_form(TILES, p, 1), p, s); }

GemmParams base_params(const unsigned char* A, int64_t lda, const float* sa, const unsigned char* W, int64_t ldw,
                       const float* sw, int64_t M, int N, int K) {
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A = (const bf16_t*)A; p.W = (const bf16_t*)W; p.lda = lda; p.ldw = ldw;      // byte pointers, byte pitches
    p.sa = sa; p.sw = sw;
    p.q_scale = 1.0f;
    p.M = (int)M; p.N = N; p.K = K;
    p.mt = (int)((M + BM - 1) / BM);
    p.nt = (N + BN - 1) / BN;
    return p;
}

}  // namespace

// K must be a multiple of 128 (whole slices), N of 64 (the epilogues work on 64-column patches).
bool gemm_fp8_supported(int N, int K) { return K > 0 && K % 128 == 0 && N > 0 && N % 64 == 0; }

int gemm_fp8_tile(int64_t M, int N, int K, int splits, int* rows, int* cols, bool w_cached, bool* turns) {
    GemmParams p = base_params(nullptr, K, nullptr, nullptr, K, nullptr, M, N, K);
    if (splits == 0) splits = plan_splits(TILES, p, SIZE_MAX, false);
    p.K = K / splits;
    const TileForm& t = FORMS[pick_form(TILES, p, splits)];
    *rows = t.bm;
    *cols = t.bn;
    *turns = t.bn == 128 && !w_cached && takes_turns(t.bm / 64, M, p.K);
    return splits;
}

void launch_gemm_fp8(int epi, const unsigned char* A, int64_t lda, const float* sa, const unsigned char* W, int64_t ldw,
                     const float* sw, bf16_t* C, int64_t ldc, const bf16_t* bias, const bf16_t* R, int64_t ldr, int64_t M,
                     int N, int K, hipStream_t s, bool w_cached) {
    if (M <= 0 || N <= 0) return;
    GemmParams p = base_params(A, lda, sa, W, ldw, sw, M, N, K);
    p.w_cached = w_cached;
    p.bias = bias; p.R = R; p.ldr = ldr; p.dst = C; p.ld = ldc;
    switch (epi) {
        case EPI_STORE: launch_t<EPI_STORE>(p, s); break;
        case EPI_RESIDUAL: launch_t<EPI_RESIDUAL>(p, s); break;
        case EPI_SILU_MUL: launch_t<EPI_SILU_MUL>(p, s); break;
        default: break;
    }
}

// The split-K forms (few rows): partial sums already carry the row and column scales, so the reduce kernels
// of the bf16 GEMM finish them.  epi: EPI_RESIDUAL (C = sum + R) or EPI_SILU_MUL (C = H [M, N / 2]).
int launch_gemm_fp8_splitk(int epi, const unsigned char* A, int64_t lda, const float* sa, const unsigned char* W,
                           int64_t ldw, const float* sw, bf16_t* C, int64_t ldc, const bf16_t* R, int64_t ldr, int64_t M,
                           int N, int K, float* part, size_t part_bytes, hipStream_t s, bool w_cached) {
    if (M <= 0 || !gemm_fp8_supported(N, K) || (epi != EPI_RESIDUAL && epi != EPI_SILU_MUL)) return 0;
    if (epi == EPI_RESIDUAL && ((N & 7) || (ldc & 7) || (ldr & 7))) return 0;
    GemmParams p = base_params(A, lda, sa, W, ldw, sw, M, N, K);
    p.w_cached = w_cached;
    const int splits = plan_splits(TILES, p, part_bytes, false);
    if (splits < 2) return 0;
    p.K = K / splits;
    p.dst = (bf16_t*)part;
    p.ld = N;
    p.ldr = M * (int64_t)N;
    launch_form<EPI_PARTIAL>(pick_form(TILES, p, splits), p, s, splits);
    if (epi == EPI_RESIDUAL) launch_splitk_reduce_residual(part, splits, R, ldr, C, ldc, M, N, s);
    else launch_splitk_reduce_silu(part, splits, C, ldc, M, N, s);
    return splits;
}

int launch_gemm_fp8_qkv_rope_splitk(const unsigned char* A, int64_t lda, const float* sa, const unsigned char* Wqkv,
                                    int64_t ldw, const float* sw, const bf16_t* bias, bf16_t* Q, bf16_t* Kd, bf16_t* Vt,
                                    int64_t ldv, const float* rope_cos, const float* rope_sin, int64_t pos0,
                                    const int32_t* row_pos, int64_t M, int qd, int kvd, int hd, int K, float q_scale,
                                    float* part, size_t part_bytes, hipStream_t s, bool w_cached) {
    const int N = qd + 2 * kvd;
    if (M <= 0 || !gemm_fp8_supported(N, K) || (qd & 63) || (kvd & 63) || (hd & 63)) return 0;
    GemmParams p = base_params(A, lda, sa, Wqkv, ldw, sw, M, N, K);
    p.w_cached = w_cached;
    const int splits = plan_splits(TILES, p, part_bytes, false);
    if (splits < 2) return 0;
    p.K = K / splits;
    p.dst = (bf16_t*)part;
    p.ld = N;
    p.ldr = M * (int64_t)N;
    launch_form<EPI_PARTIAL>(pick_form(TILES, p, splits), p, s, splits);
    GemmParams r = base_params(A, lda, sa, Wqkv, ldw, sw, M, N, K);
    r.bias = bias; r.dst = Q; r.dst_k = Kd; r.dst_vt = Vt; r.ldv = ldv;
    r.rope_cos = rope_cos; r.rope_sin = rope_sin; r.pos0 = pos0; r.row_pos = row_pos;
    r.qd = qd; r.kvd = kvd; r.hd = hd; r.q_scale = q_scale;
    launch_splitk_reduce_qkv(part, splits, r, s);
    return splits;
}

void launch_gemm_fp8_qkv_rope(const unsigned char* A, int64_t lda, const float* sa, const unsigned char* Wqkv, int64_t ldw,
                              const float* sw, const bf16_t* bias, bf16_t* Q, bf16_t* Kd, bf16_t* Vt, int64_t ldv,
                              const float* rope_cos, const float* rope_sin, int64_t pos0, const int32_t* row_pos,
                              int64_t M, int qd, int kvd, int hd, int K, float q_scale, hipStream_t s, bool w_cached) {
    if (M <= 0) return;
    GemmParams p = base_params(A, lda, sa, Wqkv, ldw, sw, M, qd + 2 * kvd, K);
    p.w_cached = w_cached;
    p.q_scale = q_scale;
    p.bias = bias; p.dst = Q; p.dst_k = Kd; p.dst_vt = Vt; p.ldv = ldv;
    p.rope_cos = rope_cos; p.rope_sin = rope_sin; p.pos0 = pos0; p.row_pos = row_pos;
    p.qd = qd; p.kvd = kvd; p.hd = hd;
    launch_t<EPI_QKV_ROPE>(p, s);
}

}  // namespace po
