// Kernels for one- and two-qubit gate sets (D = 4 or 16).
//
// Thesis Sec. 6.3.1: p[s][m] = e_m^T G[s_L] ... G[s_1] rho, the multinomial
// log-likelihood of the counts and its gradient (chain rule of the product).
//
// Layout on the chip
//   * A team of 16 lanes (one DPP row) owns one chain; lane i holds component
//     i of the current state (rows i >= D are zero padding for one qubit).
//     A wave runs four chains, a workgroup of four waves sixteen.
//   * The gate set lives in LDS twice: G (rows) for the forward product and
//     G^T (rows = columns of G) for the adjoint, rows padded to 18 doubles so
//     that the 16-byte reads of a team hit distinct banks.
//   * One step of a forward chain is, in lane i, 16 fused multiply-adds
//     acc = fma(G[k][i][j], f[j], acc), j ascending from acc = 0, with f[j]
//     broadcast from lane j of the row by DPP row_newbcast inside
//     v_fmac_f64.  This is the order of the plain definition of the product,
//     so states and probabilities are bit-identical to a sequential loop.
//   * Reverse sweeps run b <- G^T b; the pairs (b_t, f_{t-1}) of four steps of a
//     wave's four chains are staged in LDS and added to their gates' tiles by
//     FP64 MFMA 16x16x4, four pairs each (gst_seq.h).
//   * Each workgroup writes one slab of partial results; a last kernel adds
//     the slabs in ascending order (deterministic).
//
// Kernels
//   leaf_kernel      one sequence per team: forward chain, readout, objective,
//                    seeds, reverse sweep (segments recomputed from
//                    checkpoints in HBM), dG
//   reduce_kernel    sums the slabs
// (the kernels of the shared-prefix plan are in gst_plan_kernels.hip)
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"
#include "gst_seq.h"

namespace gst {
namespace {

// ---------------------------------------------------------------------------
// leaf kernel: one sequence of (off, gates) per 16-lane team
// ---------------------------------------------------------------------------
template <int D, int KT, bool PRE>
__global__ __launch_bounds__(256, seq_waves(PRE)) void leaf_kernel(const LeafLaunch a) {
  extern __shared__ double lds_raw[];
  const int K = a.K, M = a.M;
  const Lds s = carve(lds_raw, K);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, team = lane >> 4;
  stage_gateset<D>(s, a.G, a.E, a.rho, K, M);

  const int64_t gteam = ((int64_t)blockIdx.x * WAVES + wave) * TPW + team;
  const auto* g_off = as_global(a.off);
  const auto* g_gates = as_global(a.gates);
  const SeqArgs q{K,
                  M,
                  a.mode,
                  a.want_grad != 0,
                  as_global(pad_index(a)),
                  as_global(a.counts),
                  as_global(a.W),
                  as_global(a.probs),
                  a.ckpt ? a.ckpt + gteam * a.ckpt_per_team : nullptr};
  SeqSums<KT> sum;
  sum.clear();
  Pairs* st = wave_pairs(lds_raw, K, wave);

  const int64_t n_groups = (a.n_items + TPW - 1) / TPW;
  const int64_t n_waves = (int64_t)gridDim.x * WAVES;
  for (int64_t grp = (int64_t)blockIdx.x * WAVES + wave; grp < n_groups; grp += n_waves) {
    const int64_t seq = grp * TPW + team;
    const bool has = seq < a.n_items;
    const int64_t beg = has ? g_off[seq] : 0;
    const int L = has ? (int)(g_off[seq + 1] - beg) : 0;
    seq_group<D, KT, PRE>(q, s, st, has, seq, g_gates + beg, L, sum);
  }

  if (sum.bad) atomicAdd(a.status + 0, (unsigned long long)sum.bad);
  if (sum.nonpos) atomicAdd(a.status + 1, (unsigned long long)sum.nonpos);
  if (!q.grad && a.mode != MODE_LOGLIK) return;
  write_slab<D, KT>(lds_raw + lds_main_bytes(K) / 8, sum, M, K, a.slab + (int64_t)blockIdx.x * slab_width(D, M, K));
}

// Slab sums in two deterministic stages (bodies in gst_device.h).
__global__ __launch_bounds__(256) void reduce_stage1(const double* __restrict__ slab, int n_slabs, int64_t P,
                                                     int per, double* __restrict__ part) {
  slab_sum_stage1(slab, n_slabs, P, per, part, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void reduce_stage2(const double* __restrict__ part, int n_part, int64_t P,
                                                     double* objective, double* grad,
                                                     const double* __restrict__ extra_rho, int D) {
  slab_sum_stage2(part, n_part, P, objective, grad, extra_rho, D, blockIdx.x);
}

}  // namespace

int leaf_ckpt_interval(int) { return C; }
int leaf_teams_per_block(int) { return WAVES * TPW; }
int max_gates_for(int D) { return D <= 16 ? KMAX : (D == 64 ? 5 : 0); }  // D = 64: a wave's operands of all gates in registers

int leaf_blocks_for(int D, int64_t n_items) {
  (void)D;
  const int64_t per_block = WAVES * TPW;
  int64_t b = (n_items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > 2048) b = 2048;
  return (int)b;
}

hipError_t launch_leaf(const LeafLaunch& a, int n_blocks, hipStream_t stream) {
  const size_t bytes = seq_lds_bytes(a.K);
  if (a.K < 1 || a.K > KMAX) return hipErrorInvalidValue;
  if (a.D == 16 && a.K <= 6 && !a.few)
    gst_launch(leaf_kernel<16, 6, false>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 16 && a.K <= 6)
    gst_launch(leaf_kernel<16, 6, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 16)
    gst_launch(leaf_kernel<16, KMAX, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 4 && a.K <= 4)
    gst_launch(leaf_kernel<4, 4, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 4)
    gst_launch(leaf_kernel<4, KMAX, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

int reduce_parts(int n_slabs) {
  int g = (n_slabs + 15) / 16;
  return g < 1 ? 1 : (g > 64 ? 64 : g);
}

hipError_t launch_reduce(const double* slab, int n_slabs, int64_t P, double* objective, double* grad,
                         const double* extra_rho, int D, double* part, hipStream_t stream) {
  const int G = reduce_parts(n_slabs);
  const int per = (n_slabs + G - 1) / G;
  gst_launch(reduce_stage1, dim3((unsigned)((P + 63) / 64), G), dim3(256), 0, stream, slab, n_slabs, P, per,
                     part);
  gst_launch(reduce_stage2, dim3((unsigned)((P + 63) / 64)), dim3(256), 0, stream, part, G, P, objective, grad,
                     extra_rho, D);
  return hipGetLastError();
}

}  // namespace gst
