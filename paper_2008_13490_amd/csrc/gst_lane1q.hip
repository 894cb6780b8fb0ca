// One-qubit gate sets (D = 4) with one chain per lane.
//
// A one-qubit state has four components, too few to spread over a 16-lane
// DPP row without idle lanes; here every lane owns a whole chain (its four
// components in registers), a wave runs 64 sequences at once and takes
// tiles of 64 consecutive sequences of a request's length-sorted order from
// the work queue.
//
//   * Forward step, per lane: f'_i = fma(G[k][i][3], f_3, fma(.., fma(G[k][i][0],
//     f_0, 0))), columns ascending from zero as in the plain definition, so
//     states and probabilities are bit-identical to a sequential loop.  The
//     gate rows come from the wave's copy of the gate set in LDS, a gate every
//     18 doubles (lanes that apply the same gate read the same address, those
//     of different gates other banks), and are loaded a step ahead in the forward pass.
//   * Checkpoints every 8 steps in HBM (coalesced across the wave); the
//     reverse sweep recomputes a segment from its checkpoint into the wave's
//     LDS, applies b <- G^T b and accumulates dG_k += b f^T in per-lane
//     registers, gate by gate, for the lanes that apply it.
//   * Segments in which no word ends take their gate indices as one 8-byte load
//     per lane, two segments ahead; those that all 64 words run through (the
//     lengths of a tile are sorted) select no step.
//   * At the end of a tile the wave adds its 64 lanes in a fixed butterfly
//     order and writes the tile's row of partial sums (the slab layout of the
//     other kernels), so a request's result does not depend on which wave ran
//     which tile, nor on the other requests of a batch.
//
// What bounds it.  A list of 30,000 words is 469 waves, half a wave per SIMD, so
// a step's latency counts: about 105 vector instructions (48 multiply-adds for
// the three passes, 48 for the gradient, whose lanes are masked gate by gate)
// and the LDS reads of three gates.  30,000 words of 256 steps: three gates 245 ->
// 161 us, four gates 267 -> 172 us, against a kernel whose gates lay 16 doubles
// apart (all on the same banks) and whose indices came byte by byte.  Loading the
// reverse step's gate a step ahead too needs registers that spill at four gates
// (296 us) and gains nothing at three (167 us).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"

namespace gst {
namespace {

constexpr int CL = 8;               // steps per reverse segment (checkpoint interval)
constexpr int GST1 = 18;            // stride of a gate (doubles)
constexpr int HEAD = 1 + 4 + 16;    // a tile's sums of objective, rho and effects
constexpr int SLOT = 4 * GST1 + 16 + 4 + HEAD + 1;  // doubles of LDS per wave: G[4], E[4][4], rho[4], the head sums
constexpr int STASH = CL * 64 * 4;  // a segment's states: [step][half][lane][2]

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int sh = 32; sh >= 1; sh >>= 1) v += __shfl_xor(v, sh);
  return v;
}

// The 16 entries of a gate, rows in pairs of columns.
struct Gate {
  double2 a[8];
};
__device__ __forceinline__ Gate load_gate(const double* g) {
  const double2* r = reinterpret_cast<const double2*>(g);
  Gate x;
#pragma unroll
  for (int e = 0; e < 8; ++e) x.a[e] = r[e];
  return x;
}

// f' = G f with the plain column order.
__device__ __forceinline__ void apply(const Gate& g, double (&f)[4]) {
  double x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    x[i] = fma(g.a[2 * i + 1].y, f[3], fma(g.a[2 * i + 1].x, f[2], fma(g.a[2 * i].y, f[1], fma(g.a[2 * i].x, f[0], 0.0))));
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = x[i];
}

// b' = G^T b.
__device__ __forceinline__ void apply_t(const Gate& g, double (&b)[4]) {
  const double y0 = fma(g.a[6].x, b[3], fma(g.a[4].x, b[2], fma(g.a[2].x, b[1], g.a[0].x * b[0])));
  const double y1 = fma(g.a[6].y, b[3], fma(g.a[4].y, b[2], fma(g.a[2].y, b[1], g.a[0].y * b[0])));
  const double y2 = fma(g.a[7].x, b[3], fma(g.a[5].x, b[2], fma(g.a[3].x, b[1], g.a[1].x * b[0])));
  const double y3 = fma(g.a[7].y, b[3], fma(g.a[5].y, b[2], fma(g.a[3].y, b[1], g.a[1].y * b[0])));
  b[0] = y0;
  b[1] = y1;
  b[2] = y2;
  b[3] = y3;
}

// dG += b f^T in place: with fused multiply-adds of the compiler's choice the
// accumulators of the lanes that skip a gate are copied (300 spilled registers).
__device__ __forceinline__ void add_outer(double (&dG)[16], const double (&b)[4], const double (&f)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    asm volatile(
        "v_fmac_f64 %0, %4, %5\n\t"
        "v_fmac_f64 %1, %4, %6\n\t"
        "v_fmac_f64 %2, %4, %7\n\t"
        "v_fmac_f64 %3, %4, %8"
        : "+v"(dG[4 * i]), "+v"(dG[4 * i + 1]), "+v"(dG[4 * i + 2]), "+v"(dG[4 * i + 3])
        : "v"(b[i]), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]));
}

// Gate indices of steps [t, t + 8) of a word packed into 64 bits (byte x =
// step t + x; steps at or past L read as NONE).  `full` (uniform): every lane's
// word runs through them.  `base` always exists.  Byte by byte only where some word
// ends within them: lanes whose words have ended, or that have none, leave the others
// their one load (a list of one word of 100 gates, probabilities: the launch 10.2 ->
// 8.3 us).
typedef const __attribute__((address_space(1))) uint8_t* gbytes;
constexpr int NONE = 4;  // no gate: a step past the end of the word (its row address stays in the wave's LDS)
__device__ __forceinline__ uint64_t load_pack(gbytes word, int t, int L, gbytes base, bool full) {
  uint64_t k = 0;
  if (full) {
    __builtin_memcpy(&k, word + t, 8);
    return k;
  }
  k = NONE * 0x0101010101010101ull;
  if (t + CL <= L) __builtin_memcpy(&k, word + t, 8);
  if (!__ballot(t < L && t + CL > L)) return k;
  k = 0;
#pragma unroll
  for (int x = 0; x < CL; ++x) {
    const bool in = t + x < L;
    const uint64_t v = *(in ? word + t + x : base);
    k |= (in ? v : (uint64_t)NONE) << (8 * x);
  }
  return k;
}

// The gate of step x of a packed segment.
__device__ __forceinline__ int gate_of(uint64_t k, int x) {
  const uint32_t h = x < 4 ? (uint32_t)k : (uint32_t)(k >> 32);
  return (int)((h >> (8 * (x & 3))) & 0xFFu);
}

template <int K>
__global__ __launch_bounds__(256, 2) void lane1q_kernel(const BatchLaunch a) {
  extern __shared__ double lds1[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double* Gw = lds1 + wave * SLOT;
  double* Ew = Gw + 4 * GST1;
  double* rw = Ew + 16;
  double* head = rw + 4;
  double2* fsl = reinterpret_cast<double2*>(lds1 + 4 * SLOT + (size_t)wave * STASH) + lane;
  const int64_t gwave = (int64_t)blockIdx.x * 4 + wave;
  double* ck = a.ckpt + gwave * a.ckpt_per_team + lane * 4;
  int staged = -1;
  unsigned nonpos = 0;
  for (;;) {
    int tile = 0;
    if (lane == 0) tile = (int)atomicAdd(a.queue, 1u);
    tile = __builtin_amdgcn_readfirstlane(tile);
    if (tile >= a.n_tiles) break;
    const BatchTile* tp = a.tiles + tile;
    const int req = uniform(tp->req);
    const int64_t q0 = uniform64(tp->q0), q1 = uniform64(tp->q1);
    const BatchReq* rp = a.reqs ? a.reqs + req : &a.one;
    const int M = uniform(rp->M), mode = uniform(rp->mode);
    if (req != staged) {
      wave_sync();
      if (lane < K * 16) Gw[(lane >> 4) * GST1 + (lane & 15)] = rp->G[lane];
      if (lane < 16) Ew[lane] = lane < M * 4 ? rp->E[lane] : 0.0;
      if (lane < 4) rw[lane] = rp->rho[lane];
      staged = req;
      wave_sync();
    }
    const auto* g_off = as_global(uniform_ptr(rp->off));
    const auto* g_order = as_global(uniform_ptr(rp->order));
    const auto* g_gates = as_global(uniform_ptr(rp->gates));
    const auto* g_counts = as_global(uniform_ptr(rp->counts));
    const auto* g_W = as_global(uniform_ptr(rp->W));
    auto* g_probs = as_global(uniform_ptr(rp->probs));
    const bool grad = uniform(rp->want_grad) != 0;
    unsigned tile_nonpos = 0;
    // (the head sums are added up in LDS, 64 sequences at a time: the registers are the gradient's)
    wave_sync();
    if (lane < HEAD) head[lane] = 0.0;
    wave_sync();
    auto add_head = [&](int x, double v) {
      v = wsum(v);
      if (lane == 0) head[x] += v;
    };
    double dG[K][16];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int e = 0; e < 16; ++e) dG[k][e] = 0.0;
    for (int64_t qb = q0; qb < q1; qb += 64) {
      const int64_t q = qb + lane;
      const bool has = q < q1;
      const int64_t seq = has ? g_order[q] : 0;
      const int64_t beg = has ? g_off[seq] : 0;
      const int L = has ? (int)(g_off[seq + 1] - beg) : 0;
      int Lw = L, Lmin = L;
#pragma unroll
      for (int sh = 32; sh >= 1; sh >>= 1) {
        Lw = max(Lw, __shfl_xor(Lw, sh));
        Lmin = min(Lmin, __shfl_xor(Lmin, sh));
      }
      Lw = uniform(Lw);
      Lmin = uniform(Lmin);
      const gbytes word = g_gates + beg;
      // (the indices were checked when the request was created)
      auto pack = [&](int t) { return load_pack(word, t, L, g_gates, t + CL <= Lmin); };
      auto gate = [&](uint64_t k, int x) { return load_gate(Gw + gate_of(k, x) * GST1); };
      double f[4] = {rw[0], rw[1], rw[2], rw[3]};
      // ---- forward, a segment of eight steps at a time; its gate indices
      // are loaded two segments ahead, its rows a step ahead ----
      uint64_t k0 = pack(0), k1 = pack(CL);
      for (int t0 = 0; t0 < Lw; t0 += CL) {
        const uint64_t kc = k0;
        k0 = k1;
        k1 = pack(t0 + 2 * CL);
        if (grad && t0 < L) reinterpret_cast<double4*>(ck + (int64_t)(t0 / CL) * 256)[0] = double4{f[0], f[1], f[2], f[3]};
        Gate ga = gate(kc, 0), gb;
        if (t0 + CL <= Lmin) {
#pragma unroll
          for (int x = 0; x < CL; x += 2) {
            gb = gate(kc, x + 1);
            apply(ga, f);
            if (x + 2 < CL) ga = gate(kc, x + 2);
            apply(gb, f);
          }
        } else {
#pragma unroll
          for (int x = 0; x < CL; ++x) {
            if (x + 1 < CL) gb = gate(kc, x + 1);
            if (t0 + x < L) apply(ga, f);
            ga = gb;
          }
        }
      }
      // ---- readout, objective, seeds ----
      double obj = 0.0;
      double dp[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if (m < M) {
          const double* e = Ew + m * 4;
          const double p = fma(e[3], f[3], fma(e[2], f[2], fma(e[1], f[1], fma(e[0], f[0], 0.0))));
          if (has) {
            const int64_t o = seq * M + m;
            if (g_probs) g_probs[o] = p;
            if (mode == MODE_LOGLIK) {
              const int32_t N = g_counts[o];
              if (N > 0) {
                if (p <= 0.0) {
                  ++tile_nonpos;
                  obj = INFINITY;  // -N log p with p <= 0; no term is ever -inf
                } else {
                  obj -= (double)N * log(p);
                  dp[m] = -(double)N / p;
                }
              }
            } else if (mode == MODE_VJP) {
              dp[m] = g_W[o];
            }
          }
        }
      }
      if (mode == MODE_LOGLIK) add_head(0, obj);
      if (!grad) continue;
      double b[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if (m < M) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            add_head(5 + m * 4 + j, dp[m] * f[j]);
            b[j] = fma(Ew[m * 4 + j], dp[m], b[j]);
          }
        }
      }
      // ---- reverse sweep, one segment at a time: recompute its states from
      // the checkpoint into LDS, then walk it backwards.  Gate indices are
      // loaded two segments ahead, checkpoints one ----
      const int nsegw = (Lw + CL - 1) / CL, nseg = (L + CL - 1) / CL;
      auto state = [&](int c) {
        return reinterpret_cast<const double4*>(ck + (int64_t)(c >= 0 && c < nseg ? c : 0) * 256)[0];
      };
      k0 = nsegw > 0 ? pack((nsegw - 1) * CL) : 0ull;
      k1 = nsegw > 1 ? pack((nsegw - 2) * CL) : 0ull;
      double4 s0 = nsegw > 0 ? state(nsegw - 1) : double4{0.0, 0.0, 0.0, 0.0};
      for (int c = nsegw - 1; c >= 0; --c) {
        const int base = c * CL;
        const bool full = base + CL <= Lmin;
        const uint64_t kc = k0;
        k0 = k1;
        if (c >= 2) k1 = pack((c - 2) * CL);
        double s[4] = {s0.x, s0.y, s0.z, s0.w};
        s0 = state(c - 1);
        Gate ga = gate(kc, 0), gb;
#pragma unroll
        for (int x = 0; x < CL; ++x) {
          if (x + 1 < CL) gb = gate(kc, x + 1);
          fsl[(2 * x) * 64] = double2{s[0], s[1]};
          fsl[(2 * x + 1) * 64] = double2{s[2], s[3]};
          if (x + 1 < CL) {
            apply(ga, s);
            ga = gb;
          }
        }
        // One body for full and ragged segments: with two the compiler keeps the
        // accumulators twice.
#pragma unroll
        for (int x = CL - 1; x >= 0; --x) {
          ga = gate(kc, x);
          const double2 fl = fsl[(2 * x) * 64], fh = fsl[(2 * x + 1) * 64];
          const double fx[4] = {fl.x, fl.y, fh.x, fh.y};
          const int k = gate_of(kc, x);
          // dG_k += b fx^T for the gate of this step, gate by gate
#pragma unroll
          for (int kk = 0; kk < K; ++kk)
            if (k == kk) add_outer(dG[kk], b, fx);
          double nb[4] = {b[0], b[1], b[2], b[3]};
          apply_t(ga, nb);
#pragma unroll
          for (int j = 0; j < 4; ++j) b[j] = full || k != NONE ? nb[j] : b[j];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) add_head(1 + j, has ? b[j] : 0.0);
    }
    {
      const double tn = wsum((double)tile_nonpos);
      if (lane == 0 && tn > 0) atomicAdd(a.req_nonpos + (a.reqs ? req : 0), (unsigned long long)tn);
      nonpos += tile_nonpos;
    }
    if (!grad && mode != MODE_LOGLIK) continue;
    // ---- the tile's partial sums: [objective | rho (4) | E (M*4) | G (K*16)] ----
    double* out = rp->slab + (int64_t)tp->local * slab_width(4, M, K);
    wave_sync();
    if (lane < 5 + 4 * M) out[lane] = head[lane];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const double sm = wsum(dG[k][e]);
        if (lane == 0) out[5 + M * 4 + k * 16 + e] = sm;
      }
  }
  const double np = wsum((double)nonpos);  // per-lane counts
  if (lane == 0 && np > 0) atomicAdd(a.status + 1, (unsigned long long)np);
}

}  // namespace

// Per-lane kernel for one-qubit requests with K <= 4 (registers of dG).
bool lane1q_supported(int K) { return K >= 1 && K <= 4; }

size_t lane1q_lds() { return ((size_t)4 * SLOT + (size_t)4 * STASH) * sizeof(double); }

int lane1q_ckpt_per_wave(int64_t max_len) { return (int)(((max_len + CL - 1) / CL + 1) * 256); }

int lane1q_blocks_per_cu(int K) {
  int n = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (K) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lane1q_kernel<1>, 256, lane1q_lds()); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lane1q_kernel<2>, 256, lane1q_lds()); break;
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lane1q_kernel<3>, 256, lane1q_lds()); break;
    case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, lane1q_kernel<4>, 256, lane1q_lds()); break;
    default: break;
  }
  return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_lane1q(const BatchLaunch& a, int K, int n_blocks, hipStream_t stream) {
  switch (K) {
    case 1: gst_launch(lane1q_kernel<1>, dim3(n_blocks), dim3(256), lane1q_lds(), stream, a); break;
    case 2: gst_launch(lane1q_kernel<2>, dim3(n_blocks), dim3(256), lane1q_lds(), stream, a); break;
    case 3: gst_launch(lane1q_kernel<3>, dim3(n_blocks), dim3(256), lane1q_lds(), stream, a); break;
    case 4: gst_launch(lane1q_kernel<4>, dim3(n_blocks), dim3(256), lane1q_lds(), stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gst
