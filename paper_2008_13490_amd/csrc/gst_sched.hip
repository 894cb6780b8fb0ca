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
// One wave per tile, lane c = chain c.  The words are staged in LDS a window
// of steps at a time.  An entry takes about 60 vector and 60 scalar
// instructions whatever the tile; the longest tile bounds the launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"

namespace gst {
namespace {

constexpr int SCHED_WINDOW = 512;  // steps of every word staged at a time

// Adds to `rank` whether the chain D lanes further round the row waits for the
// same gate (bits 28..31 of the key) with a larger key.
template <int D>
__device__ __forceinline__ void rank_against(uint32_t key, int& rank) {
  const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x120 + D, 0xF, 0xF, false);  // row_ror:D
  rank += (other - key - 1u) < (1u << 28) - 1u && (other >> 28) == (key >> 28) ? 1 : 0;
}

__global__ __launch_bounds__(64) void sched_kernel(const SchedBuild a) {
  __shared__ uint8_t words[SCHED_CHAINS][SCHED_WINDOW];
  const int lane = threadIdx.x, c = lane & 15;
  const int64_t tile = blockIdx.x;
  const int64_t q0 = tile * a.tile_seqs;
  const int n = (int)(q0 + a.tile_seqs < a.S ? a.tile_seqs : a.S - q0);
  int64_t beg = 0;
  int len = 0;
  if (c < n) {
    const int64_t seq = a.order[q0 + c];
    beg = a.off[seq];
    len = (int)(a.off[seq + 1] - beg);
  }
  const int longest = __builtin_amdgcn_readfirstlane(len);  // the order is by length, descending
  uint32_t* out = a.entries ? a.entries + a.tile_ptr[tile] : nullptr;
  int64_t e = 0;
  int pos = 0;
  for (int w0 = 0; w0 < longest; w0 += SCHED_WINDOW) {
    __syncthreads();
    for (int x = 0; x < n; ++x) {
      const int64_t b = (int64_t)uniform64(__shfl(beg, x)) + w0;
      const int m = min(uniform(__shfl(len, x)) - w0, SCHED_WINDOW);
      for (int t = lane; t < m; t += 64) words[x][t] = a.gates[b + t];
    }
    __syncthreads();
    const int stop = min(len, w0 + SCHED_WINDOW);
    int g = pos < stop ? (int)words[c][pos - w0] : 15;
    for (;;) {
      const bool on = pos < stop && lane < 16;
      if (!__ballot(on)) break;
      // rank among the chains with the same gate: most steps left first
      const uint32_t key = ((uint32_t)g << 28) | ((uint32_t)min(len - pos, (1 << 24) - 1) << 4) | (uint32_t)(15 - c);
      int rank = 0;
      rank_against<1>(key, rank);
      rank_against<2>(key, rank);
      rank_against<3>(key, rank);
      rank_against<4>(key, rank);
      rank_against<5>(key, rank);
      rank_against<6>(key, rank);
      rank_against<7>(key, rank);
      rank_against<8>(key, rank);
      rank_against<9>(key, rank);
      rank_against<10>(key, rank);
      rank_against<11>(key, rank);
      rank_against<12>(key, rank);
      rank_against<13>(key, rank);
      rank_against<14>(key, rank);
      rank_against<15>(key, rank);
      // a round's two entries: twice the gate that most chains wait for
      bool left = on, taken = false;
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        int best = 0, most = 0;
        for (int k = 0; k < a.K; ++k) {
          const int m = __popcll(__ballot(left && g == k));
          best = m > most ? k : best;
          most = m > most ? m : most;
        }
        const bool take = left && g == best && rank < SCHED_COLS;
        uint32_t entry = (uint32_t)best << 24;
#pragma unroll
        for (int r = 0; r < SCHED_COLS; ++r) {
          const unsigned long long m = __ballot(take && rank == r);
          const unsigned long long odd = __ballot(take && rank == r && (pos & 1));
          const uint32_t id = m ? (uint32_t)(__ffsll((long long)m) - 1) : (uint32_t)SCHED_CHAINS;
          entry |= (id * 2u + (odd ? 1u : 0u)) << (6 * r);
        }
        if (out && lane == 0) out[e] = entry;
        ++e;
        if (left && g == best) rank -= SCHED_COLS;  // the gate's next four, if it is taken twice
        left = left && !take;
        taken = taken || take;
      }
      if (taken) {
        ++pos;
        g = pos < stop ? (int)words[c][pos - w0] : 15;
      }
    }
  }
  // the reverse sweeps run whole groups of entries
  const uint32_t none = SCHED_NONE;
  for (; e % SCHED_ALIGN; ++e)
    if (out && lane == 0) out[e] = none;
  if (!out && lane == 0) a.tile_n[tile] = e;
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
