// gemm_tile.hpp -- device helpers shared by the direct-to-LDS GEMM kernels.
#pragma once

#include "common.hpp"

namespace gp {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef __attribute__((address_space(3))) void* LdsPtr;

// Buffer resource over `bytes` bytes at p; raw buffer accesses beyond it read
// 0 and drop writes, which implements the tile-edge masking without branches.
constexpr uint32_t OOB = 0x80000000u;
__device__ __forceinline__ Rsrc make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// LDS tiles hold ROWS rows of BK elements (128 bytes) with no padding; the
// 16-byte chunk c of row r is stored at chunk c ^ swz(r).  swz varies over
// any 8 consecutive rows (conflict-free fragment reads, where 8 lanes read 8
// consecutive rows) and over rows 8 apart (conflict-free transposing stores,
// where 8 lanes write rows 8 apart).
__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// All waves of the workgroup meet once every LDS read of this wave has
// returned.  No memory fence: a fence would also wait for every outstanding
// direct-to-LDS load of the wave (vmcnt(0)) and so drain the prefetch ring;
// the loads a k-tile needs are waited for explicitly (wait_vmcnt) before.
// The memory clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wave index as a wave-uniform (scalar) value, so LDS base addresses derived
// from it stay in SGPRs (M0 of the direct loads).
__device__ __forceinline__ int uniform_wave_id(int tid) { return __builtin_amdgcn_readfirstlane(tid >> 6); }

// Consecutive workgroup ids go round-robin to the 8 XCDs: regrouped into one
// contiguous run of ids per XCD (bid < G, the grid).
__device__ __forceinline__ int xcd_order(int bid, int G) {
    const int G8 = G & ~7;
    return bid < G8 ? (bid & 7) * (G8 >> 3) + (bid >> 3) : bid;
}
// Output tile `id` of a problem: tiles are numbered in bands of H tile rows,
// column by column within a band, so that the tiles one XCD runs at once form
// a compact block and its L2 serves each A row panel and B column panel to
// several of them.
__device__ __forceinline__ void band_tile(int id, int tiles_m, int tiles_n, int H, int& tm, int& tn) {
    const int band = id / (H * tiles_n), in_band = id - band * H * tiles_n;
    const int bh = min(H, tiles_m - band * H);
    tm = band * H + in_band % bh;
    tn = in_band / bh;
}

} // namespace
} // namespace gp
