// Grid barriers of the multi-block kernels: the flags, their ordinals, and when
// a block's flag says that it has arrived.
//
// A job's work area ends with one flag per block.  A solve is two launches with
// barriers, the reduction and the divide and conquer, after one launch without
// (k_sytrd_reg, k_svd_jacobi), which clears the flags: the reduction then
// counts its barriers from 1, the divide and conquer from GRID_ORD_DC + 1, so
// within a solve the ordinals only grow and nothing of an earlier solve is
// left to compare with.  Which blocks a launch joins follows the live order,
// so a flag kept from solve to solve may be left as it is over any number of
// them (with ordinals that went on from launch to launch in 32 bits, a flag
// that 32768 launches had passed by counted as arrived).
#pragma once

namespace tt {

constexpr int SYNC_MAXP = 64;              // blocks one barrier may join
constexpr unsigned GRID_ORD_REDUCE = 0;    // the reduction's ordinals: this + 1, ..
constexpr unsigned GRID_ORD_DC = 1u << 16; // the divide and conquer's; the reduction passes at most 1024

// Thread tid of nt clears the flags (at the start of a solve), by stores past the
// caches, as the barriers write and read them.
__host__ __device__ inline void grid_clear(unsigned* flag, int tid, int nt) {
  for (int q = tid; q < SYNC_MAXP; q += nt)
    __hip_atomic_store(flag + q, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__host__ __device__ inline bool grid_arrived(unsigned flag, unsigned ordinal) { return flag >= ordinal; }

}  // namespace tt
