// Shared by the GEMMs that copy slices along K into a ring in LDS: what a copy may read, and how a slice is handed over
// (the first is plain C++, host and device).
#pragma once

namespace po {

// A tile is copied into LDS through a buffer descriptor of `bytes` bytes from the tile's first element, at (lane offset +
// scalar offset); lanes beyond the descriptor read as zero without traffic.  The bounds check is made on the LANE offset
// only: by contract the scalar offset is added behind it.  So a slice past the end of K must not be expressed by a
// scalar offset outside the tile; it gets an empty descriptor instead.
struct SliceWindow {
    unsigned bytes;      // of the descriptor
    int offset;          // scalar offset of the slice
};

constexpr SliceWindow slice_window(int s, int n_slices, unsigned tile_bytes, int slice_bytes) {
    return s < n_slices ? SliceWindow{tile_bytes, s * slice_bytes} : SliceWindow{0u, 0};
}

}  // namespace po

// all but the n_ youngest global->LDS loads and every LDS read done, then the workgroup barrier (n_ a constant
// expression of template parameters, which the host pass would not take as an asm operand)
#ifdef __HIP_DEVICE_COMPILE__
#define PO_WAIT_BARRIER(n_) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n_) : "memory")
// the wait alone, for a workgroup of one wavefront
#define PO_WAIT_LOADS(n_) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n_) : "memory")
#else
#define PO_WAIT_BARRIER(n_)
#define PO_WAIT_LOADS(n_)
#endif
