// bf16 MFMA GEMM for the position-wise linear layers (gfx950 / CDNA4).
//
//   C[M, N] = A[M, K] * W[N, K]^T        A: activations (token-major), W: weights in the
//                                        checkpoint layout [out, in]; both K-contiguous.
//
// What bounds it: the board's power limit.  These GEMMs keep the matrix pipe busy 64-72 % of their cycles (counters), and
// the clock the board grants (1.6-1.9 GHz of a nominal 2.4) falls with every joule spent per flop, so the design
// minimises energy per flop, not instruction slots:
//  * v_mfma_f32_16x16x32_bf16.  A bare loop of it on random operands sustains 2.1-2.2 PFLOP/s on this board, against
//    1.9 for 32x32x16 (both power-limited, with one wavefront per SIMD as with two).  The workgroup is eight
//    wavefronts, two per SIMD, arranged 2 x 4 over a 256 x 256 block tile: each owns a 128-row x 64-column patch of
//    8 x 4 tiles (128 fp32 accumulators per lane) and reads 12 fragments per 32 MFMAs.  The second wavefront of a
//    SIMD is there for the waits, not for the issue rate: it multiplies while the first waits for a fragment or at
//    the hand-over barrier, and it halves the time of the epilogue.  (A four-wavefront form with 128 x 128 patches,
//    16 fragment reads per 64 MFMAs, was built on the same ring and gives the same bits: 2-18 % slower.)  Memory
//    instructions simply sit one behind each MFMA.
//  * K is consumed in slices of 64, so that a row of an operand slice is one whole 128-byte cache line: eight
//    lanes of a load fetch one line.  Operand slices go straight from global memory into LDS (buffer_load ... lds,
//    16 bytes per lane, no staging registers; copies of this kernel that stage them through registers, with the
//    ds_writes early or late in the slice, clock 5 % higher but keep the matrix pipe 9-11 points less busy: vector
//    memory returns and LDS writes take issue slots that MFMAs of neither wavefront of the SIMD can use).  One operand's slice is a 32 KiB unit; LDS (160 KiB) is a
//    ring of five units filled in the order A0 W0 A1 W1 ...: two are being multiplied while up to three are in
//    flight.  These loads are the largest single item of the energy bill (a timing-only copy without them runs
//    15-18 % faster, one without the LDS fragment reads 7 %); their bytes per flop are fixed by the 256 x 256 tile,
//    the largest whose accumulators fit the register file.
//  * A slice is four phases of 16 MFMAs (k-step 0 rows 0-63, k-step 0 rows 64-127, k-step 1 rows 0-63, k-step 1
//    rows 64-127).  Fragments are read a whole phase ahead of their MFMAs into the A / W register set that is idle,
//    so at the hand-over barrier, which sits BEHIND PHASE 2, every LDS read of the slice is done: phase 3 multiplies
//    from registers while it reads the first fragments of the next slice, which the barrier has just handed over,
//    and the loads that overwrite this slice's two units are issued right behind the barrier.  No wavefront starts
//    a slice by waiting for LDS (worth 3-4 % over a barrier at the slice's end).
//  * LDS layout: 128-byte rows (64 bf16), the eight 16-byte segments of a row XOR-swizzled with (row >> 1) & 7, so
//    that a fragment read (16 lanes = 16 consecutive rows, same logical segment; two rows share the 256 bytes the
//    banks span) touches 16 distinct 16-byte bank groups.  The DMA writes a wavefront's 64 x 16 bytes contiguously,
//    so the swizzle is applied on the global side: lane l of a load fetches logical segment (l & 7) ^ swizzle(row).
//  * Workgroups are dispatched round-robin over the 8 XCDs (each with a private L2), so the block id is first
//    split into (XCD, local index) and every XCD walks a contiguous range of output tiles in groups of 4 M-tiles x
//    consecutive N-tiles: the 32 tiles resident on one XCD share 4 activation panels and 8 weight panels through
//    that XCD's L2.
//  * The MFMA is issued as (W fragment) x (A fragment)^T: in an accumulator tile a lane holds ONE token row and
//    four consecutive output features, so the epilogue arithmetic (bias, residual add in fp32, SiLU-multiply of
//    gate/up pairs, rotary embedding of Q/K pairs) works on whole lanes; the position-wise results then pass through
//    LDS so that they leave as whole row segments (see tile_epilogue16).
//
// A row's K reduction order (one fp32 accumulator per output runs over K in steps of 32) is fixed by the kernel and
// independent of how M is tiled or chunked, which is what makes the chunk-by-chunk evaluation of Section 4.2
// bit-exact.
#include "gemm_common.h"

#include <string.h>

#include <algorithm>

namespace po {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

namespace {

using namespace gemm;

constexpr int BK = 64;
constexpr int UNIT_BYTES = BM * BK * 2;            // one operand's slice: 256 rows x 128 bytes = 32 KiB
constexpr int NUNIT = 5;                           // ring of five units: the whole 160 KiB of LDS
constexpr int SMEM_BYTES = NUNIT * UNIT_BYTES;
constexpr int NT_BF16 = 512;                       // eight wavefronts

// MU = 16-row groups per wavefront patch: 8 (the form described above) or 6 (192-row block tile, phases of 12 MFMAs, the A
// unit three quarters full): the bits are the same, and 3/4 of a tile's time in 3/4 of its rows lets a launch whose 256-row
// tiles end in a nearly empty round come out with less of it.
template <int EPI, int MU>
__global__ void __launch_bounds__(NT_BF16) gemm_bf16_mfma_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int BM_ = 32 * MU, MH = MU / 2;      // block tile rows; 16-row groups per phase
    constexpr int NA = MU / 2;                     // global->LDS loads per wavefront for an A unit (W: 4)

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
    const int m0 = tm * BM_, n0 = tn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, l4 = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;

    const int64_t k0 = (EPI == EPI_PARTIAL) ? (int64_t)blockIdx.y * p.K : 0;
    const uint64_t a_bytes = (uint64_t)(p.M - m0) * (uint64_t)p.lda * 2 - (uint64_t)k0 * 2,
                   w_bytes = (uint64_t)(p.N - n0) * (uint64_t)p.ldw * 2 - (uint64_t)k0 * 2;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.A + (int64_t)m0 * p.lda + k0), 0, (int)(uint32_t)(a_bytes > 0xffffffffull ? 0xffffffffull : a_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.W + (int64_t)n0 * p.ldw + k0), 0, (int)(uint32_t)(w_bytes > 0xffffffffull ? 0xffffffffull : w_bytes), 0x00020000);
    uint32_t voa[4], vow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                // (voa: NA entries used)
        const int row = (wave * 4 + i) * 8 + (lane >> 3), rowa = (wave * NA + i) * 8 + (lane >> 3);
        vow[i] = (uint32_t)row * (uint32_t)(p.ldw * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
        voa[i] = (uint32_t)rowa * (uint32_t)(p.lda * 2) + (((lane & 7) ^ ((rowa >> 1) & 7)) << 4);
    }
    const int KT = p.K / BK;
    // load i_ (0..3) of this wavefront's share of the A (is_w_ = 0) or W unit of slice slice_, into ring
    // position pos_
#define PO_DMA(is_w_, slice_, pos_, i_)                                                                              \
    {                                                                                                                  \
        unsigned char* d_ = smem + (pos_) * UNIT_BYTES + (wave * ((is_w_) ? 4 : NA) + (i_)) * 1024;                    \
        __builtin_amdgcn_raw_ptr_buffer_load_lds((is_w_) ? rw : ra, (__attribute__((address_space(3))) void*)d_, 16,   \
                                                 (is_w_) ? vow[(i_)] : voa[(i_)],                    \
                                                 min((slice_), KT - 1) * (BK * 2), 0, 0);                              \
    }
    int f_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) f_off[ks] = l15 * 128 + (((ks * 4 + l4) ^ ((l15 >> 1) & 7)) << 4);
    const int a_base = wm * (MU * 16) * 128, w_base = wn * 64 * 128;

    f32x4 acc[MU][4];
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // prologue: A0 W0 A1 W1 in flight (A2 follows in slice 0); slice 0's first fragments
#pragma unroll
    for (int u4 = 0; u4 < 4; ++u4)
#pragma unroll
        for (int i = 0; i < ((u4 & 1) ? 4 : NA); ++i) PO_DMA(u4 & 1, u4 >> 1, u4, i)
    if (MU == 8) asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");      // slice 0 has landed
    else asm volatile("s_waitcnt vmcnt(7)\n\ts_barrier" ::: "memory");
    bf16x8 A0[4], A1[4], W0[4], W1[4];           // (A: MH entries used)
#pragma unroll
    for (int j = 0; j < 4; ++j) W0[j] = *(const bf16x8*)(smem + UNIT_BYTES + w_base + j * 2048 + f_off[0]);
#pragma unroll
    for (int j = 0; j < MH; ++j) A0[j] = *(const bf16x8*)(smem + a_base + j * 2048 + f_off[0]);
    // One phase: 4 MH MFMAs, rows 16 MH uh_ .. of the patch (A fragments AC, W fragments WC); behind MFMA m the
    // memory instruction number m of the phase, if it has one:
    //   RA_: read the MH A fragments (rows 16 MH rah_ .., k-step rak_) of the unit at ua_ into AN
    //   RW_: read the four W fragments (k-step rwk_) of the unit at uw_ into WN (behind the A reads)
    //   DMA_: the NA or 4 global->LDS loads of (dw_ ? W : A) unit of slice ds_ into position dp_ (behind the reads)
#define PO_PHASE(AC, WC, uh_, RA_, AN, ua_, rah_, rak_, RW_, WN, uw_, rwk_, DMA_, dw_, ds_, dp_)                    \
    _Pragma("unroll") for (int m = 0; m < 4 * MH; ++m) {                                                                \
        const int u_ = (uh_) * MH + (m >> 2), t_ = m & 3;                                                             \
        acc[u_][t_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(WC[t_], AC[m >> 2], acc[u_][t_], 0, 0, 0);              \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
        const int nra_ = (RA_) ? MH : 0, nrw_ = (RW_) ? 4 : 0;                                                         \
        if (m < nra_) {                                                                                               \
            AN[m & 3] = *(const bf16x8*)((ua_) + ((rah_) * MH + (m & 3)) * 2048 + f_off[rak_]);     \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
        } else if (m < nra_ + nrw_) {                                                                                 \
            WN[(m - nra_) & 3] = *(const bf16x8*)((uw_) + ((m - nra_) & 3) * 2048 + f_off[rwk_]);  \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
        } else if ((DMA_) && m < nra_ + nrw_ + ((dw_) ? 4 : NA)) {                                                  \
            PO_DMA(dw_, ds_, dp_, (m - nra_ - nrw_) & 3)                                         \
            __builtin_amdgcn_sched_barrier(0);                                                                        \
        }                                                                                                             \
    }
    int pa = 0;                                  // ring position of slice s's A unit; its W unit at pa + 1
    for (int s = 0; s < KT; ++s) {
        const int pw = pa + 1 >= NUNIT ? pa + 1 - NUNIT : pa + 1;
        const int pa1 = pa + 2 >= NUNIT ? pa + 2 - NUNIT : pa + 2;    // A(s+1)
        const int pw1 = pa + 3 >= NUNIT ? pa + 3 - NUNIT : pa + 3;    // W(s+1)
        const unsigned char* ua = smem + pa * UNIT_BYTES + a_base;
        const unsigned char* uw = smem + pw * UNIT_BYTES + w_base;
        const unsigned char* ua1 = smem + pa1 * UNIT_BYTES + a_base;
        const unsigned char* uw1 = smem + pw1 * UNIT_BYTES + w_base;
        // phase 0: k-step 0, rows 0-63 | reads A(k0, rows 64-127) and W(k1)
        PO_PHASE(A0, W0, 0, 1, A1, ua, 1, 0, 1, W1, uw, 1, 0, 0, 0, 0)
        // phase 1: k-step 0, rows 64-127 | reads A(k1, rows 0-63); loads A(s+2) into the position W(s-1) left
        PO_PHASE(A1, W0, 1, 1, A0, ua, 0, 1, 0, W1, uw, 1, 1, 0, s + 2, (pa + 4 >= NUNIT ? pa + 4 - NUNIT : pa + 4))
        // phase 2: k-step 1, rows 0-63 | reads A(k1, rows 64-127)
        PO_PHASE(A0, W1, 0, 1, A1, ua, 1, 1, 0, W0, uw, 0, 0, 0, 0, 0)
        // hand-over: slice s+1 has landed (all but the NA youngest loads), every LDS read of slice s is done
        if (MU == 8) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // phase 3: k-step 1, rows 64-127 | reads W(k0) and A(k0, rows 0-63) of slice s+1; loads W(s+2) into A(s)'s position
        PO_PHASE(A1, W1, 1, 1, A0, ua1, 0, 0, 1, W0, uw1, 0, 1, 1, s + 2, pa)
        pa = pa1;
    }
#undef PO_PHASE
#undef PO_DMA
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    if (EPI == EPI_PARTIAL) {
        GemmParams q = p;
        q.dst = (bf16_t*)((float*)p.dst + (int64_t)blockIdx.y * p.ldr);
        tile_epilogue16<EPI, MU>(q, acc, smem + wave * 4096, m0 + wm * (MU * 16), n0 + wn * 64, lane);
    } else {
        tile_epilogue16<EPI, MU>(p, acc, smem + wave * 4096, m0 + wm * (MU * 16), n0 + wn * 64, lane);
    }
}

// The same GEMM in small block tiles, for launches whose 256-column tiles would leave compute units idle (requests of up
// to about 2000 rows, the last layer's single row, split-K launches).  What bounds those launches is the way of an operand
// slice into LDS, not the matrix pipe: a 256-row tile of the kernel above takes 1.05 us per slice in a launch of 16 tiles,
// and the same 128 x 128 tile 0.8 us with two slices in flight and 0.41 with four.  So a tile has 128 columns, four
// wavefronts (2 x 2 patches of 16 MU rows x 64 columns) and as many slices in flight as the LDS of a whole compute unit holds
// (D = 7 at 32 rows .. 2 at 256; two workgroups per compute unit with half the depth each were 1.9 x slower at one round
// of tiles and no faster at two).  A and W have rings of their own, D + 1 and D slices: A(s + D) is loaded during phase 0
// of slice s into what A(s - 1) left, W(s + D) behind the hand-over barrier into W(s)'s place.  A slice is two phases,
// one per k-step of 32, with the next k-step's fragments read behind this one's MFMAs; swizzle, tile order and epilogues
// are those of the kernel above, and so are the bits (one fp32 accumulator per output, K in steps of 32, in order).
// Weights on their way from HBM.  A wavefront's loads return in order, so a slice whose weight rows come from HBM paces
// everything behind it: one round of 32-row tiles (N 128 or 4096, K 4096 .. 14336, 32 or 64 rows) streams its weights at 39-47
// GB/s per compute unit from HBM and at 62-76 from the memory-side cache.  The row tiles of a group sit on one
// XCD and multiply with the same weights; without help all of them wait for the same lines.  So they take turns: every 2 R
// slices one of R row tiles touches the weights of two slices a few slices ahead of the ring (one dword per line and lane,
// into LDS that nobody reads), waits for HBM that once, and all others find them in L2.  (Every tile touching its share of
// every slice helps nobody: then each of them waits for HBM every slice.)
// A touch out of turn is skipped by a branch (as an instruction with nothing to load it cost every slice 2-6 %).  Weights
// in the memory-side cache need no turns (see takes_turns).
// Measured: down projection (N 4096, K 14336) at 300 rows 97 -> 80 us with the turns, 471 rows 92 -> 79 (225 on 256-row
// tiles), 1000 rows 133 -> 117; O projection at 300 rows 30 -> 26, QKV at 1000 rows 67 -> 57.  Not kept, with and
// without turns: one ring and one barrier per slice, whole slices of fragments in registers (no faster up to 192 rows), all
// loads of a slice behind the hand-over (2-8 % slower); turns in the 256 x 256 kernel (2-3 % slower).
template <int EPI, int MU, int D, bool TURNS>
__global__ void __launch_bounds__(256, 2) gemm_bf16_small_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int BM_ = 32 * MU, BN_ = 128;
    constexpr int AU = BM_ * 128, WU = BN_ * 128;          // bytes of a slice of A / W
    constexpr int NA = MU, NW = 4;                         // global->LDS loads per wavefront and slice
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
    const int l15 = lane & 15, l4 = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;

    // resources: the tile's rows that exist (rows beyond them read as zero), columns from k0 on
    const int64_t k0 = (EPI == EPI_PARTIAL) ? (int64_t)blockIdx.y * p.K : 0;
    const uint32_t a_bytes = (uint32_t)min(BM_, p.M - m0) * (uint32_t)(p.lda * 2) - (uint32_t)(k0 * 2);
    const uint32_t w_bytes = (uint32_t)min(BN_, p.N - n0) * (uint32_t)(p.ldw * 2) - (uint32_t)(k0 * 2);
    void* const pa_ = (void*)(p.A + (int64_t)m0 * p.lda + k0);
    void* const pw_ = (void*)(p.W + (int64_t)n0 * p.ldw + k0);
    uint32_t voa[8], vow[4];                               // (voa: NA entries used)
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = (wave * NA + i) * 8 + (lane >> 3);
        voa[i] = (uint32_t)row * (uint32_t)(p.lda * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int row = (wave * NW + i) * 8 + (lane >> 3);
        vow[i] = (uint32_t)row * (uint32_t)(p.ldw * 2) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const int KT = p.K / BK;
    // Loads of slice s_ go through descriptors that are empty past the end of K: they read as zero without traffic, by
    // the lane offset (bounds are checked on that, not on the scalar offset along K).
#define PO_SLICE_RSRC(s_)                                                                                              \
    const SliceWindow wa_ = slice_window((s_), KT, (unsigned)a_bytes, BK * 2), ww_ = slice_window((s_), KT, (unsigned)w_bytes, BK * 2); \
    const int so = wa_.offset;                                                                                         \
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(pa_, 0, (int)wa_.bytes, 0x00020000);           \
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(pw_, 0, (int)ww_.bytes, 0x00020000);
#define PO_DMA_A(pos_, i_)                                                                                               \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                            \
        ra, (__attribute__((address_space(3))) void*)(smem + (pos_) * AU + (wave * NA + (i_)) * 1024), 16, voa[(i_)], so, 0, 0);
#define PO_DMA_W(pos_, i_)                                                                                               \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                            \
        rw, (__attribute__((address_space(3))) void*)(smem + (D + 1) * AU + (pos_) * WU + (wave * NW + (i_)) * 1024), 16,  \
        vow[(i_)], so, 0, 0);
    int f_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) f_off[ks] = l15 * 128 + (((ks * 4 + l4) ^ ((l15 >> 1) & 7)) << 4);
    // this wavefront's 32 weight rows of slices s_ and s_ + 1, one dword per line, when it is this row tile's turn.  (A load
    // of 64 lines keeps the address unit busy for 64 cycles even where it is masked off, hence the branch.  The hand-over's
    // count of younger loads leaves a touch out: it then waits for one load more, of the slice after.)
    unsigned char* const touched = smem + (D + 1) * AU + D * WU + wave * 256;
    const uint32_t vot = (uint32_t)(wave * 32 + (lane & 31)) * (uint32_t)(p.ldw * 2) + (lane >> 5) * 128;
    int turn = gm_this > 1 ? (tm - g * GM) * 2 : 1 << 30;
#define PO_TOUCH(s_)                                                                                                   \
    if (TURNS) {                                                                                                       \
        if (turn == 0 && (s_) + 1 < KT) {                                                                              \
            const __amdgpu_buffer_rsrc_t rt_ = __builtin_amdgcn_make_buffer_rsrc(pw_, 0, (int)w_bytes, 0x00020000);    \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rt_, (__attribute__((address_space(3))) void*)touched, 4, vot, (s_) * (BK * 2), 0, 0); \
        }                                                                                                              \
        turn = turn == 0 ? 2 * gm_this - 1 : turn - 1;                                                                 \
    }
    const int a_base = wm * (MU * 16) * 128, w_base = (D + 1) * AU + wn * 64 * 128;

    f32x4 acc[MU][4];
#pragma unroll
    for (int u = 0; u < MU; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};

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
    bf16x8 A0[MU], A1[MU], W0[4], W1[4];
#pragma unroll
    for (int j = 0; j < MU; ++j) A0[j] = *(const bf16x8*)(smem + a_base + j * 2048 + f_off[0]);
#pragma unroll
    for (int j = 0; j < 4; ++j) W0[j] = *(const bf16x8*)(smem + w_base + j * 2048 + f_off[0]);

    // One phase: the 4 MU MFMAs of one k-step; spread behind them the MU + 4 fragment reads of the next k-step (A unit
    // at ua_, W unit at uw_, k-step kn_) and then ND_ global->LDS loads
#define PO_PHASE(AC, WC, AN, WN, ua_, uw_, kn_, ND_, LOAD_)                                                            \
    _Pragma("unroll") for (int m = 0; m < 4 * MU; ++m) {                                                               \
        acc[m >> 2][m & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(WC[m & 3], AC[m >> 2], acc[m >> 2][m & 3], 0, 0, 0); \
        __builtin_amdgcn_sched_barrier(0);                                                                             \
        constexpr int T_ = MU + 4 + (ND_);                                                                             \
        _Pragma("unroll") for (int x = 0; x < T_; ++x) {                                                               \
            if (x >= m * T_ / (4 * MU) && x < (m + 1) * T_ / (4 * MU)) {                                               \
                if (x < MU) AN[x < MU ? x : 0] = *(const bf16x8*)((ua_) + x * 2048 + f_off[kn_]);                      \
                else if (x < MU + 4) WN[(x - MU) & 3] = *(const bf16x8*)((uw_) + (x - MU) * 2048 + f_off[kn_]);        \
                else { LOAD_(x - MU - 4) }                                                                             \
                __builtin_amdgcn_sched_barrier(0);                                                                     \
            }                                                                                                          \
        }                                                                                                              \
    }
    int pa = 0, pw = 0;                          // ring positions of slice s: A in D + 1 positions, W in D
    for (int s = 0; s < KT; ++s) {
        const int pa1 = pa + 1 > D ? 0 : pa + 1, pw1 = pw + 1 >= D ? 0 : pw + 1;
        const int pa_free = pa == 0 ? D : pa - 1;              // position of A(s - 1)
        PO_SLICE_RSRC(s + D)
        PO_TOUCH(s + AHEAD)
        const unsigned char* ua = smem + pa * AU + a_base;
        const unsigned char* uw = smem + pw * WU + w_base;
        const unsigned char* ua1 = smem + pa1 * AU + a_base;
        const unsigned char* uw1 = smem + pw1 * WU + w_base;
        // phase 0: k-step 0 | reads k-step 1; loads A(s + D) into the position A(s - 1) left
#define PO_LA(i_) PO_DMA_A(pa_free, ((i_) < NA ? (i_) : 0))
        PO_PHASE(A0, W0, A1, W1, ua, uw, 1, NA, PO_LA)
        // hand-over: slice s+1 has landed (everything but slices s+2 .. s+D-1 and A(s+D)); all LDS reads of slice s are done
        PO_WAIT_BARRIER((D - 2) * (NA + NW) + NA);
        // phase 1: k-step 1 | reads k-step 0 of slice s+1; loads W(s + D) into W(s)'s position
#define PO_LW(i_) PO_DMA_W(pw, ((i_) < NW ? (i_) : 0))
        PO_PHASE(A1, W1, A0, W0, ua1, uw1, 0, NW, PO_LW)
        pa = pa1;
        pw = pw1;
    }
#undef PO_LA
#undef PO_TOUCH
#undef PO_LW
#undef PO_PHASE
#undef PO_DMA_A
#undef PO_DMA_W
#undef PO_SLICE_RSRC
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (EPI == EPI_PARTIAL) {
        GemmParams q = p;
        q.dst = (bf16_t*)((float*)p.dst + (int64_t)blockIdx.y * p.ldr);
        tile_epilogue16<EPI, MU>(q, acc, smem + wave * 4096, m0 + wm * (MU * 16), n0 + wn * 64, lane);
    } else {
        tile_epilogue16<EPI, MU>(p, acc, smem + wave * 4096, m0 + wm * (MU * 16), n0 + wn * 64, lane);
    }
}

// The 32 x 128 tile of a launch of at most 16 rows (the last layer's single row above all), worked on in strips of 16
// columns (16 gate and the 16 up columns behind them, a rotary pair of 16: two strips of W rows) by a wavefront of its own.
// What bounds it: the weights' way from HBM, and a compute unit streams 128 rows of them at 39-47 GB/s (see above): with 4096
// columns in 32 tiles that is 1.5 TB/s.  Strips put a wavefront on every compute unit (256 for 4096 columns, 896 pairs for
// 28672), and 5.3-6 TB/s is what they stream.  One wavefront needs no barrier; K goes by in blocks of 256, so that a visit to
// a row is 512 bytes, straight into a ring of D blocks in LDS.  (16-byte segments XOR-swizzled with the row on the global
// side: the 16 rows of a fragment read lie 512 bytes apart.)  One accumulator per output, K in steps of 32, in order: the bits
// of every other tile.  Measured at one row: down projection (N 4096, K 14336) 76 -> 24 us, O projection 23 -> 8.4, QKV 24 ->
// 11; the 32B shape's (N 5120, K 27648) 140 -> 57, 31 -> 13, 32 -> 15; at 16 rows 83 -> 25, 25 -> 9, 26 -> 13.
// NA: loads of two activation rows per block (rows past the last one loaded hold anything: they meet no other row's sums).
template <int EPI, int NA, int D>
__global__ void __launch_bounds__(64, 2) gemm_bf16_strip_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int NS = (EPI == EPI_SILU_MUL || EPI == EPI_QKV_ROPE) ? 2 : 1;
    constexpr int BKS = 256, ROWB = BKS * 2;               // K per block; bytes of a row of it
    constexpr int BLOCK = (16 * NS + 2 * NA) * ROWB, NL = 8 * NS + NA;
    const int lane = threadIdx.x, l15 = lane & 15, l4 = lane >> 4;
    // first column of the strip(s): 16 t of a 64-column patch, its pair 32 behind
    const int c0 = NS == 2 ? (blockIdx.x >> 1) * 64 + (blockIdx.x & 1) * 16 : blockIdx.x * 16;

    // Offsets of the lane in a load of two rows; a descriptor per block, from its first column to the end of the last row
    const uint32_t lda2 = (uint32_t)(p.lda * 2), ldw2 = (uint32_t)(p.ldw * 2);
    const int row2 = lane >> 5, seg = lane & 31;           // row of the pair, physical segment
    uint32_t voa[8], vow[8];                               // (voa: NA entries used)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 2 * i + row2;
        voa[i] = (uint32_t)row * lda2 + (uint32_t)((seg ^ row) << 4);
        vow[i] = (uint32_t)row * ldw2 + (uint32_t)((seg ^ row) << 4);
    }
    const uint32_t a_bytes = (uint32_t)(p.M - 1) * lda2 + (uint32_t)p.K * 2, w_bytes = 15u * ldw2 + (uint32_t)p.K * 2;
    const unsigned char* const wbase = (const unsigned char*)(p.W + (int64_t)c0 * p.ldw);
    const int NB = (p.K + BKS - 1) / BKS;
#define PO_LOAD_BLOCK(b_, pos_)                                                                                        \
    {                                                                                                                  \
        const uint32_t o_ = (b_) < NB ? (uint32_t)(b_) * ROWB : 0u;                                                    \
        const __amdgpu_buffer_rsrc_t ra_ = __builtin_amdgcn_make_buffer_rsrc((void*)((const unsigned char*)p.A + o_), 0, (int)((b_) < NB ? a_bytes - o_ : 0u), 0x00020000); \
        unsigned char* const d_ = smem + (pos_) * BLOCK;                                                               \
        _Pragma("unroll") for (int t = 0; t < NS; ++t) {                                                               \
            const __amdgpu_buffer_rsrc_t rw_ = __builtin_amdgcn_make_buffer_rsrc((void*)(wbase + (int64_t)(32 * t) * ldw2 + o_), 0, (int)((b_) < NB ? w_bytes - o_ : 0u), 0x00020000); \
            _Pragma("unroll") for (int i = 0; i < 8; ++i)                                                              \
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rw_, (__attribute__((address_space(3))) void*)(d_ + (t * 8 + i) * 1024), 16, vow[i], 0, 0, 0); \
        }                                                                                                              \
        _Pragma("unroll") for (int i = 0; i < NA; ++i)                                                                 \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra_, (__attribute__((address_space(3))) void*)(d_ + (NS * 8 + i) * 1024), 16, voa[i], 0, 0, 0); \
    }
    static_assert((D - 1) * NL < 64, "what the counter of loads holds");
    f32x4 acc[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < D; ++b) PO_LOAD_BLOCK(b, b)
    const int arow = l15 < 2 * NA ? l15 : 0;               // (a lane without an activation row multiplies row 0 again)
#define PO_W(ks_, t_) (*(const bf16x8*)(u + (t_) * 8192 + l15 * ROWB + ((((ks_) * 4 + l4) ^ l15) << 4)))
#define PO_A(ks_) (*(const bf16x8*)(u + NS * 8192 + arow * ROWB + ((((ks_) * 4 + l4) ^ arow) << 4)))
    int pos = 0, b = 0;
    for (; b < p.K / BKS; ++b) {
        PO_WAIT_LOADS((D - 1) * NL);                       // block b has landed
        const unsigned char* u = smem + pos * BLOCK;
        bf16x8 wf[8][NS], af[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
            for (int t = 0; t < NS; ++t) wf[ks][t] = PO_W(ks, t);
            af[ks] = PO_A(ks);
        }
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
#pragma unroll
            for (int t = 0; t < NS; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][t], af[ks], acc[t], 0, 0, 0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // (every fragment is in registers: the position is free)
        PO_LOAD_BLOCK(b + D, pos)
        pos = pos + 1 == D ? 0 : pos + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (b < NB) {                                          // the last block has fewer than 8 k-steps of K
        const unsigned char* u = smem + pos * BLOCK;
        for (int ks = 0; ks < (p.K - b * BKS) >> 5; ++ks)
#pragma unroll
            for (int t = 0; t < NS; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(PO_W(ks, t), PO_A(ks), acc[t], 0, 0, 0);
    }
#undef PO_A
#undef PO_W
#undef PO_LOAD_BLOCK

    // a lane holds token row l15 and features 4 l4 .. + 3 of a strip
    if (l15 >= p.M) return;
    const int row = l15, col = c0 + 4 * l4;
    if (EPI == EPI_SILU_MUL) {
        const f32x4 &g = acc[0], &up = acc[NS - 1];
        *(uint2*)(p.dst + (int64_t)row * p.ld + (c0 >> 6) * 32 + (c0 & 63) + 4 * l4) =
            pack4(silu_f(g[0]) * up[0], silu_f(g[1]) * up[1], silu_f(g[2]) * up[2], silu_f(g[3]) * up[3]);
    } else if (EPI == EPI_QKV_ROPE) {
        float a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = acc[0][e];
            b[e] = acc[NS - 1][e];
            if (p.bias) {
                a[e] += bf2f(p.bias[col + e]);
                b[e] += bf2f(p.bias[col + 32 + e]);
            }
        }
        if (c0 < p.qd + p.kvd) {
            const bool is_q = c0 < p.qd;
            const float qs = is_q ? p.q_scale : 1.0f;
            const int half = p.hd >> 1, c = is_q ? c0 : c0 - p.qd;
            const int head = c / p.hd, in = c - head * p.hd;
            const int i0 = (in >> 6) * 32 + (in & 63) + 4 * l4;               // rotary index of register 0
            const int64_t pos_ = p.row_pos ? (int64_t)p.row_pos[p.pos0 + row] : p.pos0 + row;
            bf16_t* drow = (is_q ? p.dst + (int64_t)row * p.qd : p.dst_k + (int64_t)row * p.kvd) + head * p.hd;
            const float4 cs = *(const float4*)(p.rope_cos + pos_ * half + i0), sn = *(const float4*)(p.rope_sin + pos_ * half + i0);
            const float cv[4] = {cs.x, cs.y, cs.z, cs.w}, sv[4] = {sn.x, sn.y, sn.z, sn.w};
            float lo[4], hi[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {                  // (roundings as in tile_epilogue16)
                lo[e] = fmaf(a[e], cv[e], -(b[e] * sv[e])) * qs;
                hi[e] = fmaf(a[e], sv[e], b[e] * cv[e]) * qs;
            }
            *(uint2*)(drow + i0) = pack4(lo[0], lo[1], lo[2], lo[3]);
            *(uint2*)(drow + half + i0) = pack4(hi[0], hi[1], hi[2], hi[3]);
        } else {
            bf16_t* dcol = p.dst_vt + p.pos0 + row + (int64_t)(col - p.qd - p.kvd) * p.ldv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dcol[(int64_t)e * p.ldv] = f2bf(a[e]);
                dcol[(int64_t)(e + 32) * p.ldv] = f2bf(b[e]);
            }
        }
    } else {
        float v[4] = {acc[0][0], acc[0][1], acc[0][2], acc[0][3]};
        const bf16_t* add = EPI == EPI_RESIDUAL ? p.R + (int64_t)row * p.ldr + col : p.bias ? p.bias + col : nullptr;
        if (add) {
            const uint2 r = *(const uint2*)add;
            v[0] += __uint_as_float(r.x << 16); v[1] += __uint_as_float(r.x & 0xffff0000u);
            v[2] += __uint_as_float(r.y << 16); v[3] += __uint_as_float(r.y & 0xffff0000u);
        }
        *(uint2*)(p.dst + (int64_t)row * p.ld + col) = pack4(v[0], v[1], v[2], v[3]);
    }
}

// C[row][col .. col+7] = bf16(sum over splits of part[s][row][col ..] + R[row][col ..]); one thread per 8 features.
__global__ void __launch_bounds__(256) splitk_reduce_residual_kernel(const float* __restrict__ part, int64_t plane,
                                                                     int splits, const bf16_t* R, int64_t ldr,
                                                                     bf16_t* C, int64_t ldc, int M, int N) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int n8 = N >> 3;
    if (i >= (int64_t)M * n8) return;
    const int row = (int)(i / n8), col = (int)(i - (int64_t)row * n8) * 8;
    const float* pp = part + (int64_t)row * N + col;
    float4 a = *(const float4*)pp, b = *(const float4*)(pp + 4);
    for (int sidx = 1; sidx < splits; ++sidx) {
        const float4 x = *(const float4*)(pp + sidx * plane), y = *(const float4*)(pp + sidx * plane + 4);
        a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
        b.x += y.x; b.y += y.y; b.z += y.z; b.w += y.w;
    }
    const uint4 r = *(const uint4*)(R + (int64_t)row * ldr + col);
    uint4 o;
    o.x = (uint32_t)f2bf(a.x + __uint_as_float(r.x << 16)) | ((uint32_t)f2bf(a.y + __uint_as_float(r.x & 0xffff0000u)) << 16);
    o.y = (uint32_t)f2bf(a.z + __uint_as_float(r.y << 16)) | ((uint32_t)f2bf(a.w + __uint_as_float(r.y & 0xffff0000u)) << 16);
    o.z = (uint32_t)f2bf(b.x + __uint_as_float(r.z << 16)) | ((uint32_t)f2bf(b.y + __uint_as_float(r.z & 0xffff0000u)) << 16);
    o.w = (uint32_t)f2bf(b.z + __uint_as_float(r.w << 16)) | ((uint32_t)f2bf(b.w + __uint_as_float(r.w & 0xffff0000u)) << 16);
    *(uint4*)(C + (int64_t)row * ldc + col) = o;
}

// QKV after a split-K GEMM: one workgroup = one 64-column patch x 8 token rows.  Sums the splits' partials,
// then does what the fused QKV epilogue does with an accumulator patch: + bias, rotary embedding of the
// pair (column j, column j + 32) of a Q / K patch, V stored transposed.  Thread mapping: Q / K patches
// column-fastest (row stores are contiguous), V patches row-fastest (V^T columns are contiguous).
__global__ void __launch_bounds__(256) splitk_reduce_qkv_kernel(const float* __restrict__ part, int64_t plane, int splits,
                                                                const GemmParams p) {
    const int cb = blockIdx.x * 64;
    const bool is_v = cb >= p.qd + p.kvd;
    const int j = is_v ? (int)(threadIdx.x >> 3) : (int)(threadIdx.x & 31);
    const int row = blockIdx.y * 8 + (is_v ? (int)(threadIdx.x & 7) : (int)(threadIdx.x >> 5));
    if (row >= p.M) return;
    const float* pp = part + (int64_t)row * p.N + cb + j;
    float a = pp[0], b = pp[32];
    for (int sidx = 1; sidx < splits; ++sidx) {
        a += pp[sidx * plane];
        b += pp[sidx * plane + 32];
    }
    if (p.bias) {
        a += bf2f(p.bias[cb + j]);
        b += bf2f(p.bias[cb + 32 + j]);
    }
    if (!is_v) {
        const bool is_q = cb < p.qd;
        const int c = is_q ? cb : cb - p.qd;
        const int head = c / p.hd;
        const int half = p.hd >> 1;
        const int i0 = (((c - head * p.hd) >> 6) << 5) + j;                  // rotary index
        const int64_t pos = p.row_pos ? (int64_t)p.row_pos[p.pos0 + row] : p.pos0 + row;
        const float cs = p.rope_cos[pos * half + i0], sn = p.rope_sin[pos * half + i0];
        bf16_t* drow = (is_q ? p.dst + (int64_t)row * p.qd : p.dst_k + (int64_t)row * p.kvd) + head * p.hd + i0;
        const float qs = is_q ? p.q_scale : 1.0f;
        drow[0] = f2bf((a * cs - b * sn) * qs);
        drow[half] = f2bf((b * cs + a * sn) * qs);
    } else {
        const int f = cb - p.qd - p.kvd + j;
        bf16_t* dcol = p.dst_vt + p.pos0 + row;
        dcol[(int64_t)f * p.ldv] = f2bf(a);
        dcol[(int64_t)(f + 32) * p.ldv] = f2bf(b);
    }
}

// Gate/up after a split-K GEMM: H[row][cb/2 + j] = silu(sum gate column cb + j) * (sum up column cb + 32 + j),
// the interleaving of the fused SiLU-multiply epilogue; one thread per output feature.
__global__ void __launch_bounds__(256) splitk_reduce_silu_kernel(const float* __restrict__ part, int64_t plane, int splits,
                                                                 bf16_t* H, int64_t ldh, int M, int N) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int nf = N >> 1;
    if (i >= (int64_t)M * nf) return;
    const int row = (int)(i / nf), f = (int)(i - (int64_t)row * nf);
    const float* pp = part + (int64_t)row * N + ((f >> 5) << 6) + (f & 31);
    float g = pp[0], u = pp[32];
    for (int sidx = 1; sidx < splits; ++sidx) {
        g += pp[sidx * plane];
        u += pp[sidx * plane + 32];
    }
    H[(int64_t)row * ldh + f] = f2bf(silu_f(g) * u);
}

// Block tiles of the bf16 launches (see TileForm), fitted without turns to 232 shapes: N, K of the 8B and 32B projections, 1 ..
// 8192 rows, weights from HBM.  On 254 other launches (ten pairs of N and K, 20 .. 4096 rows), with turns as takes_turns has
// them, the pick is on average 0.1 % and at most 5 % off the fastest form.  Measured, 256-row tiles against the pick: down
// projection (N 4096, K 14336) 70 rows 244 -> 78 us, 471 rows 247 -> 80, 1000 rows 245 -> 115; O projection (4096 x 4096) 471 rows
// 72 -> 27, 845 rows 74 -> 36; from about 2000 rows (gate/up:
// 200) on the 256 x 256 tile, which moves half the bytes per flop, or the 192 x 256 one where that ends in a fuller
// round: QKV of the 32B shape (N 7168) at 3072 rows 220 -> 195 us, O projection at 5000 rows 176 -> 148, the 8B shape's
// QKV at 3500 rows 174 -> 148.
constexpr TileForm FORMS[] = {{256, 256, 5.9, 0.99, 1.41}, {32, 128, 3.1, 0.29, 0.31}, {64, 128, 2.3, 0.34, 0.40},
                              {96, 128, 2.8, 0.35, 0.47},  {128, 128, 2.7, 0.41, 0.55}, {160, 128, 3.6, 0.46, 0.63},
                              {192, 128, 3.6, 0.49, 0.70}, {256, 128, 1.0, 0.83, 0.97}, {192, 256, 3.3, 0.89, 1.15}};
constexpr TileForms TILES = {FORMS, sizeof(FORMS) / sizeof(FORMS[0]), BK, 2};
constexpr int STRIPS = sizeof(FORMS) / sizeof(FORMS[0]);       // not by time, see takes_strips

template <int EPI, int MU>
void launch_big(GemmParams p, hipStream_t s, int splits) {
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(gemm_bf16_mfma_kernel<EPI, MU>), SMEM_BYTES);
    });
    p.mt = (p.M + 32 * MU - 1) / (32 * MU);
    const int per_xcd = (p.mt * p.nt + 7) / 8;
    hipLaunchKernelGGL((gemm_bf16_mfma_kernel<EPI, MU>), dim3((unsigned)(per_xcd * 8), (unsigned)splits), dim3(NT_BF16),
                       SMEM_BYTES, s, p);
}

template <int EPI, int MU, int D, bool TURNS>
void launch_small_t(const GemmParams& p, hipStream_t s, int splits) {
    constexpr int SMEM = ((D + 1) * 32 * MU + D * 128) * 128 + 1024;           // the rings; where touches go
    static_assert(SMEM <= 160 * 1024 && SMEM >= 4 * 4096, "LDS of a compute unit; staging of four wavefronts");
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(gemm_bf16_small_kernel<EPI, MU, D, TURNS>), SMEM);
    });
    const int per_xcd = (p.mt * p.nt + 7) / 8;
    hipLaunchKernelGGL((gemm_bf16_small_kernel<EPI, MU, D, TURNS>), dim3((unsigned)(per_xcd * 8), (unsigned)splits), dim3(256),
                       SMEM, s, p);
}

// Turns, for a launch of M rows in tiles of 32 mu rows.  They pay where row tiles wait for weights from HBM, and how many do is a
// matter of the last row tile's rows: a workgroup that is nearly empty, short of activations to load, runs ahead of the others
// and fetches their weights for them (down projection of the 8B shape in 128-row tiles, us without / with turns: last tile 3 %
// full 110 / 118, 81 % full 134 / 115).  With two row tiles the one that is not on turn has nothing left to wait for.
// Measured on 393 launches, weights from HBM, eleven pairs of N and K between 2048 and 28672, 33 .. 2000 rows, time with turns
// against without:
//   up to 64 rows per tile: five row tiles and more -23 to 0 %, three or four with the last half full -15 to -4, emptier -9 to
//     +13, two +1 to +19;
//   96 rows: last tile half full or more -17 to +2, emptier -7 to +9;
//   128 rows: half full or more -14 to +2, emptier -3 to +13;
//   160 rows: three quarters full -13 to +4, emptier -4 to +12;  192 rows: -4 to +9, never taken;
//   256 rows, with the shallowest ring: -13 to 0 whatever the rows.
// (The +2 and +4 are launches of exactly 256 tiles.)  K splits, by the row tiles they have, are no different: two row tiles +3
// to +17 %, 256-row tiles -3 to -8.  Weights that sit in the memory-side cache come fast enough for all, and there turns cost 2
// to 25 %: a model that stays in it takes none (w_cached); an operator by itself does not know and goes by weights from HBM.
bool takes_turns(int mu, int64_t M) {
    const int64_t rows = 32 * mu, mt = (M + rows - 1) / rows, last = M - (mt - 1) * rows;
    const bool half = 2 * last >= rows;
    if (mu == 8) return mt > 2 || (mt == 2 && half);
    if (mu == 6 || mt < 3) return false;
    if (mu == 5) return 4 * last >= 3 * rows;
    return half || (mu <= 2 && mt >= 5);
}

template <int EPI, int MU, int D>
void launch_small(GemmParams p, hipStream_t s, int splits) {
    p.mt = (p.M + 32 * MU - 1) / (32 * MU);
    p.nt = (p.N + 127) / 128;
    if (MU != 6 && !p.w_cached && takes_turns(MU, p.M)) launch_small_t<EPI, MU, D, MU != 6>(p, s, splits);
    else launch_small_t<EPI, MU, D, false>(p, s, splits);
}

constexpr bool strip_pairs(int epi) { return epi == EPI_SILU_MUL || epi == EPI_QKV_ROPE; }

// Launches of up to 16 rows go in strips instead of 32 x 128 or 64 x 128 tiles, also where other tiles would be faster than those.
// Measured, weights from HBM, 1 .. 16 rows, us strips / the faster of the two tiles (silu: pairs of strips): up to 8192 columns
// 3.7 / 4.4 (N 4096, K 256), 8.5 / 22 (4096 x 4096), 15 / 26 (8192 x 4096), 47 / 89 (8192 x 14336), silu 20 / 26 (8192 x 4096).
// A compute unit holds three strips or pairs of up to two rows at once (their rings' LDS), two of more rows; past one round of
// them, 8192 columns and pairs of 16384, or 12288 with up to two rows, short K loses up to 0.8 us (12288 x 256 5.6 / 5.1, 16384 x
// 1024 10.7 / 10.2) and K 4096 wins 2-17 % (10240 24 / 29, 16384 28 / 34).  Pairs at the far end lose in between (16384 columns,
// K 2048 15.7 / 17.0, 4096 34.4 / 32.1, 14336 92 / 111; 14336 x 4096 27.5 / 30).  Wider launches (gate/up of the 8B shape, 224 tiles) stream their weights at 4.9
// TB/s as they are, 4.5 in strips.  (Weights from the memory-side cache, K 4096: pairs 9 / 16 at 4096 columns, 18 / 16 at 8192, 34 / 21
// at 16384; K 1024 wins there as well.)
bool takes_strips(const GemmParams& p, bool pairs) {
    if (p.M > 16 || p.N > 16384 || p.lda >= (1 << 20) || p.ldw >= (1 << 20)) return false;       // (offsets of 16 rows below 2^26 bytes)
    if (pairs) return p.N <= 14336 || p.K <= 2048 || p.K >= 8192;
    return p.N <= (p.M <= 2 ? 12288 : 8192) || p.K >= 4096;
}

// In few-rows mode the other choice is K splits.  Up to 16 rows, us strips / splits, weights from HBM: 3072 to 8192 columns always
// strips (4096 x 4096 8.6 / 12.6, 4096 x 14336 24 / 28, 8192 x 27648 76 / 91); fewer leave compute units without a strip (2048 x
// 4096 7.8 / 10.3, 2048 x 14336 20.2 / 20.1, 512 x 14336 18 / 16, 2048 x 27648 33 / 28), and more are a second round that ends with most
// of them idle (10240 x 4096 24 / 24, 12288 x 14336 82 / 64, 16384 x 14336 97 / 81).
bool takes_strips_in_few_rows_mode(const GemmParams& p, bool pairs) {
    return takes_strips(p, pairs) && (p.N <= 2048 ? p.K <= 8192 : p.N <= 8192 || p.K <= 4096);
}

template <int EPI, int NA>
void launch_strips(const GemmParams& p, hipStream_t s) {
    constexpr int NS = strip_pairs(EPI) ? 2 : 1, D = NS == 2 ? 3 : NA == 1 ? 5 : 4;
    constexpr int SMEM = D * (16 * NS + 2 * NA) * 512;
    static_assert(SMEM <= 80 * 1024, "two workgroups on a compute unit at least");
    static OncePerDevice lds;
    lds.run(current_device(), [] {
        allow_dynamic_lds((const void*)(gemm_bf16_strip_kernel<EPI, NA, D>), SMEM);
    });
    hipLaunchKernelGGL((gemm_bf16_strip_kernel<EPI, NA, D>), dim3((unsigned)(p.N / (16 * NS))), dim3(64), SMEM, s, p);
}

template <int EPI>
void launch_form(int form, const GemmParams& p, hipStream_t s, int splits = 1) {
    if (EPI != EPI_PARTIAL && form == STRIPS) {
        constexpr int E = EPI == EPI_PARTIAL ? EPI_STORE : EPI;
        if (p.M <= 2) launch_strips<E, 1>(p, s);
        else launch_strips<E, 8>(p, s);
        return;
    }
    switch (form) {
        case 1: launch_small<EPI, 1, 7>(p, s, splits); break;
        case 2: launch_small<EPI, 2, 6>(p, s, splits); break;
        case 3: launch_small<EPI, 3, 5>(p, s, splits); break;
        case 4: launch_small<EPI, 4, 4>(p, s, splits); break;
        case 5: launch_small<EPI, 5, 3>(p, s, splits); break;
        case 6: launch_small<EPI, 6, 3>(p, s, splits); break;
        case 7: launch_small<EPI, 8, 2>(p, s, splits); break;
        case 8: launch_big<EPI, 6>(p, s, splits); break;
        default: launch_big<EPI, 8>(p, s, splits); break;
    }
}

int whole_form(const GemmParams& p, bool pairs) { return takes_strips(p, pairs) ? STRIPS : pick_form(TILES, p, 1); }

template <int EPI>
void launch_t(const GemmParams& p, hipStream_t s) { launch_form<EPI>(whole_form(p, strip_pairs(EPI)), p, s); }

GemmParams base_params(const bf16_t* A, int64_t lda, const bf16_t* W, int64_t ldw, int64_t M, int N, int K) {
    GemmParams p;
    memset(&p, 0, sizeof(p));
    p.A = A; p.W = W; p.lda = lda; p.ldw = ldw;
    p.M = (int)M; p.N = N; p.K = K;
    p.q_scale = 1.0f;
    p.mt = (int)((M + BM - 1) / BM);
    p.nt = (N + BN - 1) / BN;
    return p;
}

}  // namespace

// K must be a multiple of 64 (whole slices), N of 64 (the epilogues work on 64-column patches).
bool gemm_mfma_supported(int N, int K) { return K > 0 && K % 64 == 0 && N > 0 && N % 64 == 0; }

int gemm_mfma_tile(int64_t M, int N, int K, int splits, int* rows, int* cols, bool w_cached, bool* turns) {
    GemmParams p = base_params(nullptr, K, nullptr, K, M, N, K);
    if (splits == 0) splits = plan_splits(TILES, p, SIZE_MAX, false);
    p.K = K / splits;
    const int form = splits == 1 ? whole_form(p, false) : pick_form(TILES, p, splits);
    const bool strips = form == STRIPS;
    *rows = strips ? 16 : FORMS[form].bm;
    *cols = strips ? 16 : FORMS[form].bn;
    *turns = *cols == 128 && !w_cached && takes_turns(*rows / 32, M);
    return splits;
}

double gemm_mfma_launch_cost(int64_t M, int N) { return (double)((form_tiles(FORMS[0], M, N) + 255) / 256); }

void launch_gemm_mfma(int epi, const bf16_t* A, int64_t lda, const bf16_t* W, int64_t ldw, bf16_t* C, int64_t ldc,
                      const bf16_t* bias, const bf16_t* R, int64_t ldr, int64_t M, int N, int K, hipStream_t s, bool w_cached) {
    if (M <= 0 || N <= 0) return;
    GemmParams p = base_params(A, lda, W, ldw, M, N, K);
    p.w_cached = w_cached;
    p.bias = bias; p.R = R; p.ldr = ldr; p.dst = C; p.ld = ldc;
    switch (epi) {
        case EPI_STORE: launch_t<EPI_STORE>(p, s); break;
        case EPI_RESIDUAL: launch_t<EPI_RESIDUAL>(p, s); break;
        case EPI_SILU_MUL: launch_t<EPI_SILU_MUL>(p, s); break;
        default: break;
    }
}

namespace gemm {

int64_t form_tiles(const TileForm& t, int64_t M, int N) { return ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

// whole_k: the launch's K over all splits
static double form_us(const TileForms& f, int form, int64_t M, int N, int whole_k, int splits) {
    const TileForm& t = f.form[form];
    const int64_t tiles = form_tiles(t, M, N) * splits, rounds = (tiles + 255) / 256;
    const double fill = (double)(tiles - (rounds - 1) * 256) / 256;
    const double us = t.us + (double)(whole_k / f.slice) / splits * ((double)(rounds - 1) * t.hi + t.lo + (t.hi - t.lo) * fill);
    return form == 0 ? 0.95 * us : us;           // a predicted gain below the fit's error does not leave the 256 x 256 tile
}

int pick_form(const TileForms& f, const GemmParams& p, int splits) {
    int best = 0;
    // (the small forms address a tile with offsets below 2^30 bytes)
    if (p.lda >= (1 << 20) || p.ldw >= (1 << 20)) return best;
    for (int i = 1; i < f.n; ++i)
        if (form_us(f, i, p.M, p.N, p.K * splits, splits) < form_us(f, best, p.M, p.N, p.K * splits, splits)) best = i;
    return best;
}

// Modelled time: the tiles' as in pick_form but at least the weights' at the 4.6 TB/s these launches reach, plus, split, a
// second launch (3 us) and the partial sums written and read at 6 TB/s (fitted to 40 bf16 shapes, 1 .. 1000 rows: on
// average 3.6 % off the fastest of all forms and splits).  Measured at 150 rows of the 8B shape, 256-row tiles with their
// splits -> now: O 24 -> 17 us, down 49 -> 36, QKV 28 -> 22, gate/up 75 -> 60 (unsplit).  Launches of up to 64 tiles
// always split where they can: nearly the whole chip is idle without.  (For bf16 launches that take strips few-rows mode does not
// ask here.)
int plan_splits(const TileForms& f, const GemmParams& p, size_t part_bytes, bool must) {
    const int kt = p.K / f.slice;
    auto allowed = [&](int splits) {
        return kt % splits == 0 && kt / splits >= 2 && (size_t)splits * (size_t)p.M * (size_t)p.N * sizeof(float) <= part_bytes;
    };
    if (form_tiles(f.form[0], p.M, p.N) * 2 > 256 || !allowed(2)) return 1;
    auto us = [&](int splits) {
        GemmParams q = p;
        q.K = p.K / splits;
        const double t = std::max(form_us(f, pick_form(f, q, splits), p.M, p.N, p.K, splits),
                                  (double)f.weight_bytes * p.N * p.K / 4.6e6);
        return splits == 1 ? t : t + 3.0 + 8.0 * splits * p.M * p.N / 6e6;
    };
    must = must || form_tiles(f.form[pick_form(f, p, 1)], p.M, p.N) <= 64;
    int best = must ? 2 : 1;
    for (int splits = 2 * best; splits <= 8; splits *= 2)
        if (allowed(splits) && us(splits) < us(best)) best = splits;
    return best;
}

void launch_splitk_reduce_residual(const float* part, int splits, const bf16_t* R, int64_t ldr, bf16_t* C, int64_t ldc,
                                   int64_t M, int N, hipStream_t s) {
    const int64_t n = M * (int64_t)(N >> 3);
    hipLaunchKernelGGL(splitk_reduce_residual_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part,
                       M * (int64_t)N, splits, R, ldr, C, ldc, (int)M, N);
}

void launch_splitk_reduce_silu(const float* part, int splits, bf16_t* H, int64_t ldh, int64_t M, int N, hipStream_t s) {
    const int64_t n = M * (int64_t)(N >> 1);
    hipLaunchKernelGGL(splitk_reduce_silu_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part, M * (int64_t)N,
                       splits, H, ldh, (int)M, N);
}

void launch_splitk_reduce_qkv(const float* part, int splits, const GemmParams& r, hipStream_t s) {
    hipLaunchKernelGGL(splitk_reduce_qkv_kernel, dim3((unsigned)(r.N / 64), (unsigned)((r.M + 7) / 8)), dim3(256), 0, s, part,
                       (int64_t)r.M * r.N, splits, r);
}

}  // namespace gemm

int launch_gemm_qkv_rope_splitk(const bf16_t* A, int64_t lda, const bf16_t* Wqkv, int64_t ldw, const bf16_t* bias,
                                bf16_t* Q, bf16_t* Kd, bf16_t* Vt, int64_t ldv, const float* rope_cos,
                                const float* rope_sin, int64_t pos0, const int32_t* row_pos, int64_t M, int qd, int kvd,
                                int hd, int K, float q_scale, float* part, size_t part_bytes, hipStream_t s, bool w_cached) {
    const int N = qd + 2 * kvd;
    if (M <= 0 || !gemm_mfma_supported(N, K) || (qd & 63) || (kvd & 63) || (hd & 63)) return 0;
    GemmParams p = base_params(A, lda, Wqkv, ldw, M, N, K);
    p.w_cached = w_cached;
    if (takes_strips_in_few_rows_mode(p, true)) return 0;
    const int splits = plan_splits(TILES, p, part_bytes, false);
    if (splits < 2) return 0;
    p.K = K / splits;
    p.dst = (bf16_t*)part;
    p.ld = N;
    p.ldr = M * (int64_t)N;
    launch_form<EPI_PARTIAL>(pick_form(TILES, p, splits), p, s, splits);
    GemmParams r = base_params(A, lda, Wqkv, ldw, M, N, K);
    r.bias = bias; r.dst = Q; r.dst_k = Kd; r.dst_vt = Vt; r.ldv = ldv;
    r.rope_cos = rope_cos; r.rope_sin = rope_sin; r.pos0 = pos0; r.row_pos = row_pos;
    r.qd = qd; r.kvd = kvd; r.hd = hd; r.q_scale = q_scale;
    launch_splitk_reduce_qkv(part, splits, r, s);
    return splits;
}

int launch_gemm_mfma_splitk_silu(const bf16_t* A, int64_t lda, const bf16_t* W, int64_t ldw, bf16_t* H, int64_t ldh,
                                 int64_t M, int N, int K, float* part, size_t part_bytes, hipStream_t s, bool w_cached) {
    if (M <= 0 || !gemm_mfma_supported(N, K)) return 0;
    GemmParams p = base_params(A, lda, W, ldw, M, N, K);
    p.w_cached = w_cached;
    if (takes_strips_in_few_rows_mode(p, true)) return 0;
    const int splits = plan_splits(TILES, p, part_bytes, false);
    if (splits < 2) return 0;
    p.K = K / splits;
    p.dst = (bf16_t*)part;
    p.ld = N;
    p.ldr = M * (int64_t)N;
    launch_form<EPI_PARTIAL>(pick_form(TILES, p, splits), p, s, splits);
    launch_splitk_reduce_silu(part, splits, H, ldh, M, N, s);
    return splits;
}

int launch_gemm_mfma_splitk_residual(const bf16_t* A, int64_t lda, const bf16_t* W, int64_t ldw, bf16_t* C,
                                     int64_t ldc, const bf16_t* R, int64_t ldr, int64_t M, int N, int K,
                                     float* part, size_t part_bytes, bool must, hipStream_t s, bool w_cached) {
    if (M <= 0 || N <= 0 || !gemm_mfma_supported(N, K) || (N & 7) || (ldc & 7) || (ldr & 7)) return 0;
    GemmParams p = base_params(A, lda, W, ldw, M, N, K);
    p.w_cached = w_cached;
    if (!must && takes_strips_in_few_rows_mode(p, false)) return 0;
    const int splits = plan_splits(TILES, p, part_bytes, must);
    if (splits < 2) return 0;
    p.K = K / splits;
    p.dst = (bf16_t*)part;
    p.ld = N;
    p.ldr = M * (int64_t)N;              // floats between two splits' planes
    launch_form<EPI_PARTIAL>(pick_form(TILES, p, splits), p, s, splits);
    launch_splitk_reduce_residual(part, splits, R, ldr, C, ldc, M, N, s);
    return splits;
}

void launch_gemm_qkv_rope(const bf16_t* A, int64_t lda, const bf16_t* Wqkv, int64_t ldw, const bf16_t* bias,
                          bf16_t* Q, bf16_t* Kd, bf16_t* Vt, int64_t ldv, const float* rope_cos,
                          const float* rope_sin, int64_t pos0, const int32_t* row_pos, int64_t M, int qd, int kvd,
                          int hd, int K, float q_scale, hipStream_t s, bool w_cached) {
    if (M <= 0) return;
    GemmParams p = base_params(A, lda, Wqkv, ldw, M, qd + 2 * kvd, K);
    p.w_cached = w_cached;
    p.q_scale = q_scale;
    p.bias = bias; p.dst = Q; p.dst_k = Kd; p.dst_vt = Vt; p.ldv = ldv;
    p.rope_cos = rope_cos; p.rope_sin = rope_sin; p.pos0 = pos0; p.row_pos = row_pos;
    p.qd = qd; p.kvd = kvd; p.hd = hd;
    launch_t<EPI_QKV_ROPE>(p, s);
}

}  // namespace po
