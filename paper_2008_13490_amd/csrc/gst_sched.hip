// Grouped schedules of word lists without shared prefixes.
//
// Random words apply a different gate in every chain, and a matrix-vector step
// that reads its gate from LDS is bound by those reads (2 KB per two-qubit
// step, 32 KB per three-qubit step).  The chains are independent of each
// other, so they need not run in lockstep: a tile of up to 16 chains advances,
// at every schedule entry, up to four chains whose next gate is the same, as
// one product of that gate (held in registers) with a block of four states.
// The schedule depends on the words alone.  It is built once per request by
// this kernel, forward in time; run from its last entry to its first it is a
// schedule of the reverse sweep.
//
// Entries come in rounds of two that advance different chains, so that a
// round's products are independent.  Each entry takes the gate that most
// remaining chains wait for, and of its chains the four with the most steps
// left.  On random words over five gates a tile of 16 chains fills 98 % of its
// columns, over six gates 94 % (12 chains: 86 and 80 %, 8: 64 and 59 %; with the
// four lowest chains instead of the longest ones, and one entry a round, 82 %
// instead of 99: the others fall behind and finish alone).
//
// One wave per tile, lane c = chain c (gst_sched_tile.h).  The words are staged in LDS a window
// of steps at a time.  An entry takes about 60 vector and 60 scalar
// instructions whatever the tile; the longest tile bounds the launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"
#include "gst_sched_tile.h"

namespace gst {
namespace {

// The lanes of the kernel's wave.
struct WaveLanes {
  __device__ __forceinline__ int lane() const { return threadIdx.x; }
  __device__ __forceinline__ unsigned long long ballot(bool v) const { return __ballot(v); }
  __device__ __forceinline__ int first(int v) const { return __builtin_amdgcn_readfirstlane(v); }
  __device__ __forceinline__ int64_t from(int64_t v, int lane) const { return uniform64(__shfl(v, lane)); }
  __device__ __forceinline__ int from(int v, int lane) const { return uniform(__shfl(v, lane)); }
  // the value D lanes further round the row of sixteen
  template <int D>
  __device__ __forceinline__ uint32_t round(uint32_t v) const {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + D, 0xF, 0xF, false);  // row_ror:D
  }
  __device__ __forceinline__ void sync() const { __syncthreads(); }
};

struct Words {
  uint8_t w[SCHED_CHAINS][SCHED_WINDOW];
  __device__ __forceinline__ uint8_t get(int c, int t) const { return w[c][t]; }
  __device__ __forceinline__ void put(int c, int t, uint8_t k) { w[c][t] = k; }
};

__global__ __launch_bounds__(64) void sched_kernel(const SchedBuild a) {
  __shared__ Words words;
  sched_tile(a, (int64_t)blockIdx.x, words, WaveLanes());
}

}  // namespace

hipError_t launch_sched(const SchedBuild& a, int64_t n_tiles, hipStream_t stream) {
  if (n_tiles <= 0) return hipSuccess;
  if (a.tile_seqs < 1 || a.tile_seqs > SCHED_CHAINS || a.K < 1 || a.K > 8 || n_tiles > 0x7fffffff)
    return hipErrorInvalidValue;
  gst_launch(sched_kernel, dim3((unsigned)n_tiles), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace gst
