// The per-sequence evaluation of the 16-lane-team kernels: four sequences per
// wave, one per DPP row, lane i of a row holding component i of its state.
// Included by the plain sequence kernel and the persistent tile kernel.
//
// What bounds it.  A vector instruction and an FP64 MFMA never overlap on a SIMD
// (measured: a wave of 16x16x4 MFMAs and a wave of 32-bit integer operations
// take the sum of their times), so a step costs its vector instructions, about
// 4.4 cycles each, plus its MFMAs, 64 cycles each; and its rows cost LDS time,
// 4 cycles per 16-byte read of a wave.  The three passes over a word (forward,
// recomputation of a segment, reverse) are 48 multiply-adds and 23 such reads
// per step of four chains; the rest is kept small:
//   * a step's row address is one addition: the gates' byte offsets are
//     multiplied once per chunk and broadcast inside the addition;
//   * where all four words of a group still run (their lengths are sorted) no
//     step selects between the old and the new state;
//   * the gate gradient collects four (adjoint, state) pairs of one gate per
//     MFMA from four steps of the four chains, staged in LDS; the places are
//     found with scalar instructions, a vector instruction only unpacks them.
//     (One MFMA per step and gate present, the other chains' rows zeroed, needs
//     no staging but 3.1 MFMAs a step instead of 1.4, and was no faster.)
// Staging four steps instead of eight leaves room for three waves per SIMD
// instead of two.  On 24 requests with 37 M two-qubit steps the tile kernel went
// from 51 to 37 cycles of a CU per step: the LDS is busy for 75 % of that, the
// SIMDs for 69 %.
#pragma once
#include "gst_device.h"

namespace gst {
namespace {

// Waves per SIMD.  A launch that fills the chip with three runs each step's row
// loads when they are needed and leaves the waiting to the other waves; one of
// fewer loads every row a step ahead (PRE), which takes 64 more registers and leaves
// room for two.  Both do the same operations in the same order.  Where the line
// lies, in us without and with loading ahead:
//   tile kernel, words of up to 256 gates: 4,000 words 145, 129; 8,192 (two tiles per CU)
//     158, 146; 10,000 168, 149; 12,000 (2.9) 177, 152; 16,000 189, 199; 30,000 285, 321.
//     Its workgroups are persistent: loading ahead is the faster one up to three tiles
//     per CU, although only two run at once.
//   plain kernel, up to 64 gates: 2,000 words 43, 40; 8,192 (two workgroups per CU) 55.4,
//     54.6; 8,300 65, 75; 12,000 70, 88.  A third workgroup would wait for a whole one.
constexpr int seq_waves(bool pre) { return pre ? 2 : 3; }

// A wave's partial sums.  Tile element (r, c) of dE (outcome r) and dG is in
// lane 16 (r & 3) + c, register r >> 2.
template <int KT>
struct SeqSums {
  double obj, drho;
  d4 dE;
  d4 dG[KT];
  unsigned bad, nonpos;
  __device__ __forceinline__ void clear() {
    obj = 0.0;
    drho = 0.0;
    dE = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < KT; ++k) dG[k] = d4{0.0, 0.0, 0.0, 0.0};
    bad = 0;
    nonpos = 0;
  }
};

typedef const __attribute__((address_space(1))) uint8_t* gbytes;
typedef const __attribute__((address_space(1))) int32_t* gcounts;
typedef const __attribute__((address_space(1))) double* gdoubles;

// What the four sequences of a group are evaluated with.
struct SeqArgs {
  int K, M, mode;
  bool grad;
  gbytes base;         // a byte that always exists, read in place of indices past the end of a word
  gcounts counts;
  gdoubles W;
  __attribute__((address_space(1))) double* probs;  // or null
  double* ck;          // this team's checkpoints
};

// The pairs staged for the gate gradient: half a segment's steps of the wave's
// four chains (pair 4R + row), and a pair of zeros.
constexpr int HALF = C / 2, PAIRS = HALF * TPW;
struct Pairs {
  double b[PAIRS + 1][16];
  double f[PAIRS + 1][16];
};
// LDS: the gate set, and behind it the waves' pairs, at the end of a tile the
// sums of its waves (the gate set stays for the next tile).
__host__ __device__ inline size_t seq_lds_bytes(int K) {
  const size_t a = WAVES * sizeof(Pairs), b = lds_red_bytes(K);
  return lds_main_bytes(K) + (a > b ? a : b);
}
__device__ __forceinline__ Pairs* wave_pairs(double* lds_raw, int K, int wave) {
  Pairs* p = reinterpret_cast<Pairs*>(lds_raw + lds_main_bytes(K) / 8) + wave;
  const int lane = threadIdx.x & 63;
  if (lane < 16) {
    p->b[PAIRS][lane] = 0.0;
    p->f[PAIRS][lane] = 0.0;
  }
  return p;
}

// dG_k += sum of b f^T over the staged pairs with gate k, four per MFMA 16x16x4
// (A[i][z] = b_z[i], B[z][j] = f_z[j]); lane e < PAIRS holds pair e's gate.
template <int KT>
__device__ __forceinline__ void add_pairs(const Pairs& st, int gate, int K, d4 (&dG)[KT]) {
  const int lane = threadIdx.x & 63, i = lane & 15, shift = 8 * (lane >> 4);
#pragma unroll
  for (int x = 0; x < KT; ++x)
    if (x < K) {
      unsigned m = (unsigned)__ballot(gate == x);
      while (m) {
        unsigned at = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          at |= (unsigned)__builtin_ctz(m | 1u << PAIRS) << (8 * z);
          m &= m - 1;
        }
        const int e = (int)((at >> shift) & 0xFFu);
        dG[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(st.b[e][i], st.f[e][i], dG[x], 0, 0, 0);
      }
    }
}

// Lane i's row (of the gates or of their transposes, `base` at row i of the
// first) of the gate whose byte offset lane R of the DPP row holds.
template <int D, int R>
__device__ __forceinline__ RowD<D> step_row(const double* base, int koff) {
  return load_row_d<D>(reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + bcast_i32<R>(koff)));
}

// One sequence per row: `seq` (its row of the counts, weights and
// probabilities) with the word `word` of length L; `has` false: no sequence.
template <int D, int KT, bool PRE>
__device__ __forceinline__ void seq_group(const SeqArgs& a, const Lds& s, Pairs* st, bool has, int64_t seq,
                                          gbytes word, int L, SeqSums<KT>& sum) {
  const int lane = threadIdx.x & 63, i = lane & 15, team = lane >> 4;
  const int K = a.K, M = a.M;
  const int Lw = wave_max4(L), Lmin = -wave_max4(-L);
  constexpr int KB = GATE_STRIDE * 8;  // bytes of a gate in LDS
  const double* grow0 = s.Gs + i * ROW;
  const double* gtrow0 = s.GTs + i * ROW;
  double f = s.rho[i];
  // ---- forward chain, a checkpoint every C steps.  Gate indices are loaded
  // one chunk of 16 steps ahead; the loads are unconditional (past the end of
  // the word they read a byte that always exists) so that the compiler can
  // wait for the previous load alone ----
  int kv_next = *(i < L ? word + i : a.base);
  kv_next = i < L ? kv_next : 0;
  for (int t0 = 0; t0 < Lw; t0 += 16) {
    int kv = kv_next;
    const bool in = t0 + 16 + i < L;
    kv_next = *(in ? word + t0 + 16 + i : a.base);
    kv_next = in ? kv_next : 0;
    if (t0 + i < L && kv >= K) {
      ++sum.bad;
      kv = 0;
    }
    const int koff = kv * KB;
    RowD<D> ra, rb;
    if (PRE) ra = step_row<D, 0>(grow0, koff);
    if (t0 + 16 <= Lmin) {
#define GST_FWD_STEP(R, ROW_)                                        \
  {                                                                  \
    if (a.grad && ((R) % C) == 0) a.ck[((t0 + R) / C) * 16 + i] = f;   \
    f = dot_row(f, ROW_);                                              \
  }
#define GST_FWD_TWO(R)                                                           \
  if (PRE) rb = step_row<D, R + 1>(grow0, koff); else ra = step_row<D, R>(grow0, koff); \
  GST_FWD_STEP(R, ra)                                                            \
  if (PRE && R < 14) ra = step_row<D, (R + 2) & 15>(grow0, koff);                   \
  if (!PRE) rb = step_row<D, R + 1>(grow0, koff);                                   \
  GST_FWD_STEP(R + 1, rb)
      GST_FWD_TWO(0) GST_FWD_TWO(2) GST_FWD_TWO(4) GST_FWD_TWO(6)
      GST_FWD_TWO(8) GST_FWD_TWO(10) GST_FWD_TWO(12) GST_FWD_TWO(14)
#undef GST_FWD_STEP
      continue;
    }
#define GST_FWD_STEP(R, ROW_)                                            \
  {                                                                      \
    const int t = t0 + R;                                                \
    if (a.grad && ((R) % C) == 0 && t < L) a.ck[(t / C) * 16 + i] = f;     \
    const double fn = dot_row(f, ROW_);                                    \
    f = t < L ? fn : f;                                                  \
  }
    for (;;) {
      GST_FWD_TWO(0)
      if (t0 + 2 >= Lw) break;
      GST_FWD_TWO(2)
      if (t0 + 4 >= Lw) break;
      GST_FWD_TWO(4)
      if (t0 + 6 >= Lw) break;
      GST_FWD_TWO(6)
      if (t0 + 8 >= Lw) break;
      GST_FWD_TWO(8)
      if (t0 + 10 >= Lw) break;
      GST_FWD_TWO(10)
      if (t0 + 12 >= Lw) break;
      GST_FWD_TWO(12)
      if (t0 + 14 >= Lw) break;
      GST_FWD_TWO(14)
      break;
    }
#undef GST_FWD_TWO
#undef GST_FWD_STEP
  }

  // ---- readout: lane m < M of a row holds p_m ----
  const double p = dot16_bcast(f, reinterpret_cast<const double2*>(s.Es + i * ROW));
  double dp = 0.0;
  if (has && i < M) {
    const int64_t o = seq * M + i;
    if (a.probs) a.probs[o] = p;
    if (a.mode == MODE_LOGLIK) {
      const int32_t N = a.counts[o];
      if (N > 0) {
        if (p <= 0.0) {
          ++sum.nonpos;
          sum.obj = INFINITY;  // -N log p with p <= 0; no term is ever -inf
        } else {
          sum.obj -= (double)N * log(p);
          dp = -(double)N / p;
        }
      }
    } else if (a.mode == MODE_VJP) {
      dp = a.W[o];
    }
  }
  if (!a.grad) return;

  // ---- dE[m] += dp_m f over the rows; seed b = sum_m dp_m e_m ----
  sum.dE = __builtin_amdgcn_mfma_f64_16x16x4f64(dp, f, sum.dE, 0, 0, 0);
  double b = dot16_bcast(dp, reinterpret_cast<const double2*>(s.ETs + i * ROW));

  // ---- reverse sweep, one segment of C steps at a time: its states from the
  // checkpoint, then back.  A segment's gate indices and checkpoint are loaded
  // one segment ahead ----
  const int nseg = (L + C - 1) / C;
  const int nsegw = wave_max4(nseg);
  int kv_nx;
  bool kv_in;
  double ck_nx;
  {
    const int c = nsegw - 1;
    const bool seg = c >= 0 && c < nseg;
    kv_in = seg && i < C && c * C + i < L;
    kv_nx = *(kv_in ? word + c * C + i : a.base);
    ck_nx = *(seg ? a.ck + c * 16 + i : a.ck);
  }
  // lane e < PAIRS: the lane that holds the gate of pair e (row e & 3, step e >> 2) of the first half
  const int pair_src = lane < PAIRS ? 16 * (lane & 3) + (lane >> 2) : C;
  for (int c = nsegw - 1; c >= 0; --c) {
    const bool act = c < nseg;
    const int base = c * C;
    int kv = kv_in ? kv_nx : 0;
    if (kv >= K) kv = 0;  // counted in the forward sweep
    const int koff = kv * KB;
    const int gate = kv_in ? kv : 0xFF;  // the gate, or none (lanes i >= C: none)
    double fs[C];
    fs[0] = act ? ck_nx : 0.0;
    {
      const bool seg = c >= 1 && c - 1 < nseg;
      kv_in = seg && i < C && (c - 1) * C + i < L;
      kv_nx = *(kv_in ? word + (c - 1) * C + i : a.base);
      ck_nx = *(seg ? a.ck + (c - 1) * 16 + i : a.ck);
    }
    RowD<D> ra, rb;
    if (PRE) ra = step_row<D, 0>(grow0, koff);
#define GST_REC_TWO(R)                                                           \
  if (PRE) rb = step_row<D, R + 1>(grow0, koff); else ra = step_row<D, R>(grow0, koff); \
  fs[R + 1] = dot_row(fs[R], ra);                                                  \
  if (PRE) ra = step_row<D, R + 2>(grow0, koff); else rb = step_row<D, R + 1>(grow0, koff); \
  fs[R + 2] = dot_row(fs[R + 1], rb);
    GST_REC_TWO(0) GST_REC_TWO(2) GST_REC_TWO(4)
#undef GST_REC_TWO
    if (PRE) rb = step_row<D, 7>(gtrow0, koff); else ra = step_row<D, 6>(grow0, koff);
    fs[7] = dot_row(fs[6], ra);
    const bool full = base + C <= Lmin;
#define GST_BWD(R, ROW_)                                     \
  {                                                          \
    st->b[((R) % HALF) * TPW + team][i] = b;                   \
    st->f[((R) % HALF) * TPW + team][i] = fs[R];               \
    const double bn = dot_row(b, ROW_);                        \
    if (full)                                                \
      b = bn;                                                \
    else                                                     \
      b = act && base + R < L ? bn : b;                      \
  }
#define GST_BWD_TWO(R)                                                              \
  if (PRE) ra = step_row<D, R - 1>(gtrow0, koff); else rb = step_row<D, R>(gtrow0, koff);  \
  GST_BWD(R, rb)                                                                    \
  if (PRE && R > 1) rb = step_row<D, (R - 2) & 15>(gtrow0, koff);                      \
  if (!PRE) ra = step_row<D, R - 1>(gtrow0, koff);                                     \
  GST_BWD(R - 1, ra)
#define GST_PAIRS(H)                                                      \
  {                                                                       \
    wave_sync();                                                          \
    add_pairs<KT>(*st, __shfl(gate, pair_src + H * HALF), K, sum.dG);     \
    wave_sync();                                                          \
  }
    GST_BWD_TWO(7) GST_BWD_TWO(5)
    GST_PAIRS(1)
    GST_BWD_TWO(3) GST_BWD_TWO(1)
    GST_PAIRS(0)
#undef GST_PAIRS
#undef GST_BWD_TWO
#undef GST_BWD
  }
  if (has) sum.drho += b;
}

// Adds the waves' sums in their order (in `red`, the waves' pairs) and writes the
// slab row [objective | drho (D) | dE (M*D) | dG (K*D*D)].
template <int D, int KT>
__device__ void write_slab(double* red, SeqSums<KT>& sum, int M, int K, double* slab) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double o = sum.obj, dr = sum.drho;
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) o += __shfl_xor(o, sh);
  dr += __shfl_xor(dr, 16);
  dr += __shfl_xor(dr, 32);
  for (int w = 0; w < WAVES; ++w) {
    __syncthreads();  // the pairs have been read; the previous wave's sums are in place
    if (wave != w) continue;
    const bool first = w == 0;
    if (lane == 0) red[0] = first ? o : red[0] + o;
    if (lane < 16) red[1 + lane] = first ? dr : red[1 + lane] + dr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int at = (4 * v + (lane >> 4)) * 16 + (lane & 15);
      red[17 + at] = first ? sum.dE[v] : red[17 + at] + sum.dE[v];
    }
#pragma unroll
    for (int k = 0; k < KT; ++k)
      if (k < K) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int at = 273 + k * 256 + (4 * v + (lane >> 4)) * 16 + (lane & 15);
          red[at] = first ? sum.dG[k][v] : red[at] + sum.dG[k][v];
        }
      }
  }
  __syncthreads();
  const int64_t P = slab_width(D, M, K);
  for (int x = tid; x < P; x += blockDim.x) {
    int src;
    if (x < 1 + D) {
      src = x;
    } else if (x < 1 + D + M * D) {
      const int y = x - 1 - D;
      src = 17 + (y / D) * 16 + (y % D);
    } else {
      const int y = x - 1 - D - M * D;
      const int k = y / (D * D), r = (y / D) % D, c = y % D;
      src = 273 + k * 256 + r * 16 + c;
    }
    slab[x] = red[src];
  }
}

}  // namespace
}  // namespace gst
