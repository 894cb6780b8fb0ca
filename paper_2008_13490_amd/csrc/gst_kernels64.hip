// Kernels for three-qubit gate sets (D = 64).
//
// Thesis Sec. 6.3.1: p[s][m] = e_m^T G[s_L] ... G[s_1] rho, the multinomial
// log-likelihood of the counts and its gradient.
//
// Two evaluations share the kernels below: lists with shared prefixes as a
// grouped-chain plan (gst_plan64.h), other lists as grouped schedules
// (gst_sched.hip).  Both hold the gates in registers as operands of the FP64
// matrix cores and step a block of states at a time, 16 columns with one word
// in the plan's tiles, 4 columns that happen to need the same gate in the
// schedules' tiles.  An FP64 MFMA adds its four products one after another in
// ascending order, so every state is the chain of fused multiply-adds
// acc = fma(G[i][j], f[j], acc), j = 0 .. 63 from acc = 0, of the plain
// definition, and probabilities are bit-identical to a sequential loop.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"
#include "gst_plan64.h"

namespace gst {
namespace {

constexpr int N64 = 64;
constexpr int GATE64 = N64 * N64;  // doubles per gate in LDS

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) v += __shfl_xor(v, sh);
  return v;
}

// Workgroup barrier for the LDS exchange of a step: waits for this wave's LDS
// operations only, so the global stores of the step and the operand loads of
// the next step stay in flight across it (a full __syncthreads() would wait for
// them as well).  The memory clobber keeps the compiler from moving LDS
// accesses across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------
// Lists without shared prefixes: grouped schedules (gst_sched.hip).
//
// A tile of up to 16 chains is a workgroup's; an entry steps up to four chains
// by one gate: 64 x 64 times 64 x 4, wave w computing rows 16w .. 16w + 15 with
// sixteen v_mfma_f64_4x4x4 (four blocks of four rows by the same four columns;
// 16 cycles each, 22 in a dependent chain, the rate of the 16x16x4 form).  A
// wave keeps its operands of all K <= 5 gates in registers (160 VGPRs), so the
// gates cost no bandwidth; with each step's 32 KB gate read from LDS, one
// chain per wave, those reads bound a chain-step at 256 cycles per CU.  The
// states live in LDS, double-buffered by the parity of the chain's step, so a
// round of two entries (of different chains) needs one barrier.
//
// Both kernels run eight waves, two per SIMD.  Forward: four waves per entry of
// the round, so the two products fill each other's latencies (302 -> 170 us
// below, against one entry after the other on two workgroups of four waves per
// CU; 164 since the gates' rows come through LDS); the states before each entry are recorded one after the other, so that a
// chain-step takes 512 bytes whatever its entry holds.
// Reverse: four waves step the adjoints of both entries, at a raised priority,
// and the other four load the recorded states two rounds ahead and add
// dG += b f^T, one 16x16x4 MFMA per 16 x 16 tile and entry, in accumulators for
// all gates (160 registers), so the adjoints are never stored and the states
// are read once.  (One role per wave: the transposed gates' operands and the
// accumulators together spill, 461 instead of 253 us.)  A tile belongs to a
// fixed workgroup, so the sums do not depend on scheduling.
//
// 8,000 words of up to 128 gates (510,378 steps), per evaluation with the
// gradient: 4.86 -> 0.43 ms, against a chain per wave with the gates in LDS,
// stored adjoints, and a GEMM over the stored pairs.  A round takes about 0.5 us
// forward and 0.9 us reverse; the LDS reads of a round (each wave reads all
// four states, repeated for its four row blocks) take half of that, the
// products the other half.
// ---------------------------------------------------------------------------

// A state in LDS: component 4s + k at k * SKS + s, so that a lane reads its
// sixteen operands of row k with eight 16-byte reads.
constexpr int SKS = 18;            // stride of the four component classes (doubles)
constexpr int SST = 4 * SKS + 2;   // stride of a state
constexpr int SLOTS = 2 * (SCHED_CHAINS + 1);
__device__ __forceinline__ int state_at(int j) { return (j & 3) * SKS + (j >> 2); }

// Operands of G (or, TR, of its transpose) for the 4x4x4 MFMA: lane 16k + 4b + i
// holds rows 16w + 4b + i, columns 4s + k, s = 0 .. 15.  Columns of G^T are read from
// memory as they are; rows of G through LDS, since one load of sixteen rows takes
// sixteen cache lines (that alone was 12 us of the launch, for a list of one word of
// 16 gates as for one of 8,000: 20 -> 9 and 174 -> 163 us).
constexpr int GST = N64 + 2;  // stride (doubles) of a staged gate's rows
template <bool TR>
struct SchedGates {
  double g[5][16];
  __device__ __forceinline__ void load_columns(const double* G, int K, int w, int l) {
    static_assert(TR, "the transposed gates");
    const auto* p = as_global(G);
#pragma unroll
    for (int x = 0; x < 5; ++x)
      if (x < K) {
#pragma unroll
        for (int s = 0; s < 16; ++s) g[x][s] = p[x * GATE64 + (4 * s + (l >> 4)) * N64 + 16 * w + (l & 15)];
      }
  }
  // 512 threads; T: a gate in LDS
  __device__ __forceinline__ void load_rows(const double* G, int K, int w, int l, double* T) {
    static_assert(!TR, "the gates themselves");
    const auto* p = as_global(reinterpret_cast<const d2*>(G));
    const int t = threadIdx.x;
    d2 in[5][4];
#pragma unroll
    for (int x = 0; x < 5; ++x)
      if (x < K) {
#pragma unroll
        for (int u = 0; u < 4; ++u) in[x][u] = p[x * (GATE64 / 2) + t + 512 * u];
      }
#pragma unroll
    for (int x = 0; x < 5; ++x)
      if (x < K) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          *reinterpret_cast<d2*>(T + ((t + 512 * u) >> 5) * GST + 2 * (t & 31)) = in[x][u];
        lds_barrier();
#pragma unroll
        for (int s = 0; s < 16; ++s) g[x][s] = T[(16 * w + (l & 15)) * GST + 4 * s + (l >> 4)];
        lds_barrier();
      }
  }
};

// The workgroup's tiles: there and back over rows of `row` length-sorted tiles,
// so that the tiles of a workgroup, and of workgroups that share a CU, differ
// in length.  `at` is the place in that order; next_tile advances it to the
// next tile (n_tiles: none left).
__device__ __forceinline__ int next_tile(int& at, int row, int n_tiles) {
  for (;; at += gridDim.x) {
    const int y = at / row, x = at - y * row;
    if (y * row >= n_tiles) return n_tiles;
    const int t = y * row + ((y & 1) ? row - 1 - x : x);
    if (t < n_tiles) {
      at += gridDim.x;
      return t;
    }
  }
}

// Field r of an entry: two times the chain's index, plus the parity of its step.
__device__ __forceinline__ int entry_field(uint32_t e, int r) { return (int)((e >> (6 * r)) & 63u); }

// A wave's rows of the product of an entry's gate with the entry's block: acc
// holds row 16w + 4b + k of column i in lane 16k + 4b + i.
template <bool TR>
__device__ __forceinline__ double sched_product(const SchedGates<TR>& gates, uint32_t en, const double2 (&v)[8]) {
  double acc = 0.0;
  switch (en >> 24) {
#define GST_S64_CASE(X)                                                                    \
  _Pragma("unroll") for (int s = 0; s < 8; ++s) {                                          \
    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(gates.g[X][2 * s], v[s].x, acc, 0, 0, 0);     \
    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(gates.g[X][2 * s + 1], v[s].y, acc, 0, 0, 0); \
  }                                                                                        \
  break;
    case 0: GST_S64_CASE(0)
    case 1: GST_S64_CASE(1)
    case 2: GST_S64_CASE(2)
    case 3: GST_S64_CASE(3)
    default: GST_S64_CASE(4)
#undef GST_S64_CASE
  }
  return acc;
}

// An entry's product: FLIP reads the state of the entry's fields with the other
// parity (the reverse sweep) and writes the field's own.
template <bool TR, int FLIP>
__device__ __forceinline__ void sched_step(const SchedGates<TR>& gates, double* V, uint32_t en, int w, int l) {
  const int k4 = l >> 4, b4 = (l >> 2) & 3, j4 = l & 3;
  const int f = (int)((en >> (6 * j4)) & 63u) ^ FLIP;
  const double2* src = reinterpret_cast<const double2*>(V + f * SST + k4 * SKS);
  double2 v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = src[s];
  const double acc = sched_product<TR>(gates, en, v);
  if (f < 2 * SCHED_CHAINS) V[(f ^ 1) * SST + k4 * SKS + 4 * w + b4] = acc;
}

// An entry without chains (the second of a round, or padding).
__device__ __forceinline__ bool sched_empty(uint32_t en) { return (en & 0xffffffu) == SCHED_NONE; }

// Its chains: columns 0 .. n - 1 (the others' fields hold chain 16).
__device__ __forceinline__ int sched_live(uint32_t en) { return SCHED_COLS - __popc(en & SCHED_NONE); }

// A lane's entry's chains, those of the lanes before it, and of all lanes.
struct LiveSum {
  int own, before, all;
};
__device__ __forceinline__ LiveSum sched_live_sum(int own) {
  LiveSum s{own, 0, 0};
#pragma unroll
  for (int bit = 0; bit < 3; ++bit) {
    const unsigned long long m = __ballot(own >> bit & 1);
    s.before += (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)) << bit;
    s.all += __popcll(m) << bit;
  }
  return s;
}

// Eight waves, two per SIMD: waves 0 .. 3 step a round's first entry, waves
// 4 .. 7 its second.
__global__ __launch_bounds__(512, 2) void chain64_fwd_kernel(const Chain64Launch a) {
  __shared__ __align__(16) double V[SLOTS * SST];
  __shared__ __align__(16) double T[N64 * GST];  // a gate on its way into registers
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & 3, z = wave >> 2;
  SchedGates<false> gates;
  gates.load_rows(a.G, a.K, w, l, T);
  const double rho = as_global(a.rho)[l];
  const auto* entries = as_global(a.entries);
  auto* rec = as_global(a.rec_f);
  auto* fin = as_global(a.fin);
  if (blockIdx.x == 0 && wave == 0) {
    if (a.rec_f) rec[(int64_t)a.zero_rec * N64 + l] = 0.0;
    if (l == 0) *a.nonpos = 0ull;  // (the readout counts)
  }
  int at = blockIdx.x;
  for (int tile = next_tile(at, a.tile_row, a.n_tiles); tile < a.n_tiles; tile = next_tile(at, a.tile_row, a.n_tiles)) {
    const int64_t q0 = (int64_t)tile * a.tile_seqs;
    const int n = (int)(q0 + a.tile_seqs < a.S ? a.tile_seqs : a.S - q0);
    int done = (int)uniform64(a.tile_rec[tile]);  // records of the entries before
    const int64_t e0 = sched_at(uniform64(a.tile_rec[tile]), tile);
    const int ne = uniform(a.tile_n[tile]);
    for (int c = wave; c <= SCHED_CHAINS; c += 8) {
      V[2 * c * SST + state_at(l)] = c < n ? rho : 0.0;
      if (c == SCHED_CHAINS) V[(2 * c + 1) * SST + state_at(l)] = 0.0;
    }
    uint32_t next = entries[e0 + min(l, max(ne - 1, 0))];
    lds_barrier();
    for (int eb = 0; eb < ne; eb += 64) {  // the entries' count is a multiple of SCHED_ALIGN
      const uint32_t cur = next;
      const int m = min(ne - eb, 64);
      next = entries[e0 + min(eb + 64 + l, ne - 1)];
      // lane x: the record of column w before entry x, or none
      const LiveSum live = sched_live_sum(l < m ? sched_live(cur) : 0);
      const int rows = a.rec_f && w < live.own ? done + live.before + w : -1;
      done += live.all;
      for (int x = 0; x < m; x += 2) {
        const uint32_t en = (uint32_t)__builtin_amdgcn_readlane((int)cur, x + z);
        const int row = __builtin_amdgcn_readlane(rows, x + z);
        if (!sched_empty(en)) {
          sched_step<false, 0>(gates, V, en, w, l);
          // the state before the entry is still there: the step wrote the other parity
          if (row >= 0) rec[(int64_t)row * N64 + l] = V[entry_field(en, w) * SST + state_at(l)];
        }
        lds_barrier();
      }
    }
    for (int c = wave; c < n; c += 8) {
      const int64_t seq = a.order[q0 + c];
      const int odd = (int)(a.off[seq + 1] - a.off[seq]) & 1;
      fin[(q0 + c) * N64 + l] = V[(2 * c + odd) * SST + state_at(l)];
    }
    lds_barrier();  // the states have been read
  }
}

constexpr int SFS = 80;  // stride (doubles) of an entry's staged states: a half-wave's reads hit distinct banks

// dg[tc] += b f^T over an entry's four columns, for the four 16 x 16 tiles of a
// wave's rows.
__device__ __forceinline__ void add_outer(d4 (&dg)[4], double b, const double (&f)[4]) {
#pragma unroll
  for (int tc = 0; tc < 4; ++tc) dg[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(b, f[tc], dg[tc], 0, 0, 0);
}

// Waves 0 .. 3: the adjoints.  Waves 4 .. 7: dG.  Both pass the same barriers.
__global__ __launch_bounds__(512, 2) void chain64_bwd_kernel(const Chain64Launch a) {
  __shared__ __align__(16) double V[SLOTS * SST];
  __shared__ double F[2][2][SCHED_COLS * SFS];  // the recorded states of a round's entries, double-buffered
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & 3;
  const auto* entries = as_global(a.entries);
  const int64_t P = 1 + N64 + (int64_t)a.M * N64;
  double* head = a.head + (int64_t)blockIdx.x * P;
  if (wave < 4) {
    __builtin_amdgcn_s_setprio(2);  // the chains are what a round waits for
    SchedGates<true> gates;
    gates.load_columns(a.G, a.K, w, l);
    const auto* fin = as_global(a.fin);
    double drho = 0.0;
    int at = blockIdx.x;
    for (int tile = next_tile(at, a.tile_row, a.n_tiles); tile < a.n_tiles;
         tile = next_tile(at, a.tile_row, a.n_tiles)) {
      const int64_t q0 = (int64_t)tile * a.tile_seqs;
      const int n = (int)(q0 + a.tile_seqs < a.S ? a.tile_seqs : a.S - q0);
      const int64_t e0 = sched_at(uniform64(a.tile_rec[tile]), tile);
      const int ne = uniform(a.tile_n[tile]);
      uint32_t next = entries[e0 + max(ne - 1 - l, 0)];
      for (int c = w; c <= SCHED_CHAINS; c += 4) {
        if (c < n) {
          const int64_t seq = a.order[q0 + c];
          const int odd = (int)(a.off[seq + 1] - a.off[seq]) & 1;
          V[(2 * c + odd) * SST + state_at(l)] = fin[(q0 + c) * N64 + l];
        }
        if (c == SCHED_CHAINS) {
          V[2 * c * SST + state_at(l)] = 0.0;
          V[(2 * c + 1) * SST + state_at(l)] = 0.0;
        }
      }
      lds_barrier();
      for (int xb = 0; xb < ne; xb += 64) {
        const uint32_t cur = next;
        const int m = min(ne - xb, 64);
        next = entries[e0 + max(ne - 65 - xb - l, 0)];
        for (int x = 0; x < m; x += 2) {
          const uint32_t en0 = (uint32_t)__builtin_amdgcn_readlane((int)cur, x);
          const uint32_t en1 = (uint32_t)__builtin_amdgcn_readlane((int)cur, x + 1);
          if (!sched_empty(en0)) sched_step<true, 1>(gates, V, en0, w, l);
          if (!sched_empty(en1)) sched_step<true, 1>(gates, V, en1, w, l);
          lds_barrier();
        }
      }
      for (int c = w; c < n; c += 4) drho += V[2 * c * SST + state_at(l)];
      lds_barrier();  // the adjoints have been read
    }
    V[w * SST + l] = drho;
    lds_barrier();
    // the head row: dL/drho of the four waves added in order
    for (int64_t x = threadIdx.x; x < P; x += 256) {
      const int j = (int)x - 1;
      head[x] = x >= 1 && x <= N64 ? (V[j] + V[SST + j]) + (V[2 * SST + j] + V[3 * SST + j]) : 0.0;
    }
    return;
  }
  const int k4 = l >> 4, i16 = l & 15;
  const auto* rec = as_global(a.rec_f);
  d4 dg[5][4];
#pragma unroll
  for (int x = 0; x < 5; ++x)
#pragma unroll
    for (int tc = 0; tc < 4; ++tc) dg[x][tc] = d4{0.0, 0.0, 0.0, 0.0};
  int at = blockIdx.x;
  for (int tile = next_tile(at, a.tile_row, a.n_tiles); tile < a.n_tiles; tile = next_tile(at, a.tile_row, a.n_tiles)) {
    const int64_t e0 = sched_at(uniform64(a.tile_rec[tile]), tile);
    const int ne = uniform(a.tile_n[tile]);
    // The records of 64 entries, backwards from the tile's last one: lane x has the
    // row of column w's state before entry x of them (no chain there: the row of
    // zeros), `end` moves to the first entry's.
    int end = (int)uniform64(a.tile_rec[tile + 1]);
    auto entry = [&](int xb) { return entries[e0 + max(ne - 1 - xb - l, 0)]; };
    auto records = [&](uint32_t en, int xb) {
      const LiveSum live = sched_live_sum(xb + l < ne ? sched_live(en) : 0);
      const int row = w < live.own ? end - live.before - live.own + w : a.zero_rec;
      end -= live.all;
      return row;
    };
    uint32_t cur = entry(0), next = entry(64);
    int rows = records(cur, 0), rows_next = records(next, 64);
    auto state = [&](int rows, int x) {
      return rec[(int64_t)(uint32_t)__builtin_amdgcn_readlane(rows, x) * N64 + l];
    };
    double ring[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) ring[u] = state(rows, u);
    F[0][0][w * SFS + l] = ring[0];
    F[0][1][w * SFS + l] = ring[1];
    ring[0] = state(rows, 4);
    ring[1] = state(rows, 5);
    lds_barrier();
    for (int xb = 0; xb < ne; xb += 64) {
      const int m = min(ne - xb, 64);
      const uint32_t later = entry(xb + 128);
      // the rows of the loads, six entries ahead
      const int here = __shfl(rows, (l + 6) & 63), there = __shfl(rows_next, (l + 6) & 63);
      const int ahead = l < 58 ? here : there;
      for (int x0 = 0; x0 < m; x0 += 4) {
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          // the next round's states, loaded two rounds ago, and the loads that replace them
          F[y ^ 1][0][w * SFS + l] = ring[2 - 2 * y];
          F[y ^ 1][1][w * SFS + l] = ring[3 - 2 * y];
          ring[2 - 2 * y] = state(ahead, x0 + 2 * y);
          ring[3 - 2 * y] = state(ahead, x0 + 2 * y + 1);
#pragma unroll
          for (int z = 0; z < 2; ++z) {
            const uint32_t en = (uint32_t)__builtin_amdgcn_readlane((int)cur, x0 + 2 * y + z);
            // A[i][c] = b of column c (rows 16w + i), B[c][j] = f of column c
            const int fc = (int)((en >> (6 * k4)) & 63u) ^ 1;
            const double bc = V[fc * SST + state_at(16 * w + i16)];
            double fv[4];
#pragma unroll
            for (int tc = 0; tc < 4; ++tc) fv[tc] = F[y][z][k4 * SFS + 16 * tc + i16];
            // one test per gate: with a switch the compiler keeps a second copy of the
            // accumulators (160 spilled registers)
            const uint32_t gk = en >> 24;
#pragma unroll
            for (int X = 0; X < 5; ++X)
              if (gk == (uint32_t)X && !sched_empty(en)) add_outer(dg[X], bc, fv);
          }
          lds_barrier();
        }
      }
      cur = next;
      next = later;
      rows = rows_next;
      rows_next = records(next, xb + 128);
    }
    lds_barrier();  // the adjoints have been read
  }
  lds_barrier();  // the head row
  // tile element C[r][cc] sits in lane 16*(r&3)+cc, register r>>2
#pragma unroll
  for (int x = 0; x < 5; ++x)
    if (x < a.K) {
      double* out = a.dg + ((int64_t)x * gridDim.x + blockIdx.x) * GATE64;
#pragma unroll
      for (int tc = 0; tc < 4; ++tc)
#pragma unroll
        for (int v = 0; v < 4; ++v) out[(16 * w + 4 * v + k4) * N64 + 16 * tc + i16] = dg[x][tc][v];
    }
}

// Gate columns of the gradient: entry e of dG_k is the sum of the chunk
// partials of gate k, added in order with four interleaved partial sums.
// (The tile columns [objective | rho | E] go through the two-stage ordered
// reduction of the other kernels.)
__device__ __forceinline__ void reduce64_body(const Reduce64Launch& a, int64_t bx) {
  __shared__ double red[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t y = bx * 64 + tx;  // index into [K][4096]
  const int64_t Y = (int64_t)a.K * GATE64;
  double v = 0.0;
  if (y < Y) {
    const int k = (int)(y / GATE64);
    const int64_t e = y % GATE64;
    // eight partials loaded at a time (one after another the loads' latency
    // was most of the kernel: 200,960 sequences, 150 chunks a gate, 16.5 -> 8.5 us)
    const double* p = a.chunk_slab + e;
    const int64_t c1 = a.gate_chunk_ptr[k + 1];
    int64_t c = a.gate_chunk_ptr[k] + ty;
    for (; c + 28 < c1; c += 32) {
      double t[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) t[x] = p[(c + 4 * x) * GATE64];
#pragma unroll
      for (int x = 0; x < 8; ++x) v += t[x];
    }
    for (; c < c1; c += 4) v += p[c * GATE64];
  }
  red[ty][tx] = v;
  __syncthreads();
  if (ty != 0 || y >= Y) return;
  v = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
  const bool nonpos = a.nonpos && *a.nonpos != 0;
  if (a.grad && !nonpos) a.grad[1 + N64 + (int64_t)a.M * N64 - 1 + y] = v;
}

__global__ __launch_bounds__(256) void reduce64_kernel(const Reduce64Launch a) { reduce64_body(a, blockIdx.x); }

// Word lists: the head rows in two ordered stages, the second one's launch with the
// gate columns too (a list of one word of 16 gates 41.0 -> 39.3 us).
__global__ __launch_bounds__(256) void head_sum64_stage1(const HeadSum64 a) {
  slab_sum_stage1(a.head, a.n_rows, a.P, a.per, a.part, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void head_sum64_stage2(const HeadSum64 a, const Reduce64Launch gates) {
  const int64_t head = (a.P + 63) / 64;
  if ((int64_t)blockIdx.x < head)
    slab_sum_stage2(a.part, a.n_part, a.P, a.objective, a.grad, nullptr, N64, blockIdx.x);
  else
    reduce64_body(gates, blockIdx.x - head);
}

// ---------------------------------------------------------------------------
// The grouped-chain plan (gst_plan64.h).
//
// A tile holds sixteen chains with one gate word.  Its states form a 64 x 16
// block V; a step is V <- G V, one FP64 MFMA product.  Wave w of the tile's
// workgroup computes rows 16w .. 16w+15 with sixteen 16x16x4 MFMAs over the
// inner index in ascending blocks of four; each MFMA adds its four products
// one after another in ascending order, so every entry is the chain of fused
// multiply-adds acc = fma(G[i][j], v[j], acc), j = 0 .. 63 from acc = 0 (the
// plain definition's order: probabilities are bit-identical to it).  The block
// lives in LDS in the operand order of the MFMA (Vs[kk][lane] = V[4kk +
// lane/16][lane%16]), which is also the order in which the products come out,
// so a step writes its rows straight back for the next one.  The A operands
// come from a copy of the gate set rearranged once per evaluation so that every
// operand load reads 512 consecutive bytes; the next step's operands are
// loaded while the current step runs.
// ---------------------------------------------------------------------------

// GA[k][w][kk][l] = G[k][16w + l%16][4kk + l/16]; GAT the same for G^T; workgroup
// `blk` writes 256 entries of each.  The first one also writes rho into row 0 of
// the state arena, and clears the evaluation's count of p <= 0 entries.
constexpr int PREP_WG = GATE64 / 256;  // workgroups per gate
__device__ __forceinline__ void gate_prep64_body(const double* G, const double* rho, double* GA, double* GAT,
                                                 double* FA, unsigned long long* nonpos, int blk) {
  const int64_t x = (int64_t)blk * 256 + threadIdx.x;
  const double* g = G + x / GATE64 * GATE64;
  const int w = (int)(x >> 10) & 3, kk = (int)(x >> 6) & 15, l = (int)x & 63;
  GA[x] = g[(16 * w + (l & 15)) * N64 + 4 * kk + (l >> 4)];
  GAT[x] = g[(4 * kk + (l >> 4)) * N64 + 16 * w + (l & 15)];
  if (blk == 0) {
    if (threadIdx.x < N64) FA[threadIdx.x] = rho[threadIdx.x];
    if (threadIdx.x == 0 && nonpos) *nonpos = 0ull;
  }
}

__global__ __launch_bounds__(256) void gate_prep64_kernel(const double* G, const double* rho, double* GA, double* GAT,
                                                          double* FA, unsigned long long* nonpos) {
  gate_prep64_body(G, rho, GA, GAT, FA, nonpos, blockIdx.x);
}

__device__ __forceinline__ void load_ops(double (&dst)[16], const double* base, int lane) {
  const auto* g = as_global(base);
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) dst[kk] = g[kk * 64 + lane];
}

// A tile's gate word and events are staged in LDS a chunk of steps at a time,
// so that the loop over the steps reads nothing from global memory whose value
// it needs at once: the only global loads in the loop are the next step's
// operands (the gate, and in the reverse sweep the vectors added at the next
// node), issued a whole step ahead.
constexpr int CH_STEPS = 256;   // steps per staged chunk
constexpr int CH_EVENTS = 1024; // events per staged chunk (a node has at most EV_NODE)
constexpr int EV_NODE = kMaxNodeEvents;  // events of one node at most: its seed and a chain per child
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // a step's row of the column table

// A tile-step's 16 states in LDS: element (row 4k + r4, column c) at
// k * VST + 16 r4 + c, which is where lane 16 r4 + c of an MFMA reads its B
// operand of block k and writes row 4 v + r4 of its output block; the blocks
// are padded by two doubles so that the row-wise reads below spread over the
// banks.
constexpr int VST = 66;

// Levels of short chains: the operands of the next step's gate are loaded while
// the current step runs.
struct LoadGates {
  double an[16];
  __device__ __forceinline__ void start(const double* base, int k, int w, int l) {
    load_ops(an, base + ((int64_t)k * 4 + w) * 1024, l);
  }
  // the gate loaded a step ago times B; each register takes gate k_next's operand
  // (< 0: none) as soon as its MFMA has read it, so one set of 16
  // registers serves both
  __device__ __forceinline__ d4 product(const double* base, int k_next, const double* B, int w, int l) {
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    if (k_next >= 0) {
      const auto* g = as_global(base + ((int64_t)k_next * 4 + w) * 1024);
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) {
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(an[kk], B[kk * VST + l], acc, 0, 0, 0);
        an[kk] = g[kk * 64 + l];
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(an[kk], B[kk * VST + l], acc, 0, 0, 0);
    }
    return acc;
  }
};


// Writes the tile-step's 16 adjoints (columns c = 0..15) to 16 consecutive
// arena rows, two doubles per lane and store, so that every wave store covers
// 1 KB of consecutive memory; non-temporal, since only the gradient GEMM reads
// them (held in the L2 they would be written back at the kernel's end).

__device__ __forceinline__ void store_tile_rows(const double* V, double* out, int tid) {
  auto* g = as_global(reinterpret_cast<d2*>(out));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int f = 2 * (tid + 256 * h);  // column f >> 6, doubles (f & 63) and the next
    const int cc = f >> 6, j = f & 63;
    d2 v;
    v.x = V[(j >> 2) * VST + (j & 3) * 16 + cc];
    v.y = V[((j + 1) >> 2) * VST + ((j + 1) & 3) * 16 + cc];
    __builtin_nontemporal_store(v, &g[f >> 1]);
  }
}

__device__ __forceinline__ void plan64_fwd_body(const Plan64Launch& a, int64_t tile) {
  __shared__ double Vs[2][16 * VST];
  __shared__ uint8_t Ws[CH_STEPS + 1];
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const int c = l & 15, r4 = l >> 4;
  // a tile of a few steps is a chain of memory round trips: its arrays, then the
  // anchors' states and the word, then the first gate's operands
  const int len = uniform(a.tile_len[tile]);
  const auto* word = as_global(a.words + a.tile_word[tile]);
  const int64_t row0 = a.tile_row0[tile];
  const int first = word[0];
  const int64_t anc = a.col_anchor[tile * 16 + c];
  const auto* fa = as_global(a.FA + anc * N64 + 16 * w + r4);
  double f0[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) f0[v] = fa[4 * v];
  LoadGates gs;
  gs.start(a.GA, uniform(first), w, l);
#pragma unroll
  for (int v = 0; v < 4; ++v) Vs[0][(4 * w + v) * VST + l] = f0[v];
  int cur = 0;
  for (int t0 = 0; t0 < len; t0 += CH_STEPS) {
    const int n = len - t0 < CH_STEPS ? len - t0 : CH_STEPS;
    // word[t0 .. t0 + n], the last one the first gate of the next chunk
    for (int x = tid; x <= n && t0 + x < len; x += 256) Ws[x] = word[t0 + x];
    lds_barrier();
    for (int x = 0; x < n; ++x) {
      const int t = t0 + x;
      const d4 acc = gs.product(a.GA, t + 1 < len ? uniform(Ws[x + 1]) : -1, Vs[cur], w, l);
      // rows 16w + 4v + r4 of column c: operand block kk = 4w + v of the next step
      // (stored straight from the registers: measured faster here than the
      // row-wise stores through LDS that the reverse sweep uses)
      auto* dst = as_global(a.FA + (row0 + (int64_t)t * 16 + c) * N64 + 16 * w + r4);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        Vs[cur ^ 1][(4 * w + v) * VST + l] = acc[v];
        dst[4 * v] = acc[v];
      }
      lds_barrier();
      cur ^= 1;
    }
  }
}

__global__ __launch_bounds__(256) void plan64_fwd_kernel(const Plan64Launch a) {
  plan64_fwd_body(a, a.t_begin + blockIdx.x);
}

// Rows 4(4w + v) + r4 of the INJ rows that events of one node add to column c:
// up to EV_NODE rows, a window of them in fixed registers, added later in the
// events' order.
// The node is step x of the staged chunk: its events are Ev[Es[x] ..
// Es[x + 1]), ascending by column, and the step's row of the column table says
// where column c's lie, so no lane scans the others'.  The loads run over the
// most events of one column at this step (a uniform count); a lane with fewer
// loads rows of the step's other events, which `n` masks out where they are
// added.
// R rows of a column per lane, the first of them row0, four apart.
template <int W, int R>
struct NodeAdds {
  double r[W][R];
  int n;     // this column's events at the node
  int most;  // the most events of one column at the node (uniform)
};

// Events e0 .. e0 + W - 1 of the node (a window of W rows; a node has up to
// EV_NODE, so a window smaller than that is loaded in several rounds).
template <int W, int R>
__device__ __forceinline__ void load_node_adds(NodeAdds<W, R>& q, const int32_t* Es, const int32_t* Ev, const u32x4* Cc,
                                               int x, int e0, int c, int row0, const double* inj) {
  const auto* g = as_global(inj);
  const int jb = uniform(Es[x]), tot = uniform(Es[x + 1]) - jb;
  const auto* row = reinterpret_cast<const uint8_t*>(Cc + x);
  q.most = uniform((int)row[15]);
  const int lo = c > 0 ? (int)row[c - 1] : 0, hi = c < 15 ? (int)row[c] : tot;
  q.n = hi - lo;
  int src[W];
#pragma unroll
  for (int e = 0; e < W; ++e) {
    const int j = jb + (lo + e0 + e < tot ? lo + e0 + e : tot - 1);
    src[e] = Ev[j < 0 ? 0 : (j < CH_EVENTS ? j : CH_EVENTS - 1)];
  }
#pragma unroll
  for (int e = 0; e < W; ++e)
#pragma unroll
    for (int v = 0; v < R; ++v) q.r[e][v] = 0.0;
#pragma unroll
  for (int e = 0; e < W; ++e)
    if (e0 + e < q.most)
#pragma unroll
      for (int v = 0; v < R; ++v) q.r[e][v] = g[(int64_t)src[e] * N64 + row0 + 4 * v];
}

// Adds the window's events to `add` in their order (absent ones add zero); the
// first window starts the sum with its first row, so the node's sum is the same
// chain of additions whatever the window.
template <int W, int R>
__device__ __forceinline__ double node_add(const NodeAdds<W, R>& q, int e0, double add, int v) {
#pragma unroll
  for (int e = 0; e < W; ++e) {
    const double r = e0 + e < q.n ? q.r[e][v] : 0.0;
    add = (e0 == 0 && e == 0) ? r : add + r;
  }
  return add;
}

// A node's events summed: the first window loaded earlier (q), the others now.
template <int W, int R>
__device__ __forceinline__ void node_sum(NodeAdds<W, R>& q, const int32_t* Es, const int32_t* Ev, const u32x4* Cc, int x,
                                         int c, int row0, const double* inj, double (&add)[R]) {
#pragma unroll
  for (int v = 0; v < R; ++v) add[v] = node_add(q, 0, 0.0, v);
  for (int e0 = W; e0 < q.most; e0 += W) {
    load_node_adds(q, Es, Ev, Cc, x, e0, c, row0, inj);
#pragma unroll
    for (int v = 0; v < R; ++v) add[v] = node_add(q, e0, add[v], v);
  }
}

// A chunk of a tile's reverse sweep, staged in LDS: the steps [t0, t1) with at
// most CH_STEPS steps and CH_EVENTS events, and the events of step t0 - 1, which
// are added at the end of step t0.
struct ChunkLds {
  // Ws[x] = word[t0 - 1 + x] (x = 0 only if t0 > 0), EV_FLAG set if the step
  // before it has events
  uint8_t Ws[CH_STEPS + 1];
  int32_t Es[CH_STEPS + 2];     // events before step s0 + x
  int32_t Ev[CH_EVENTS];
  u32x4 Cc[CH_STEPS + 1];       // the column table of step s0 + x
};
constexpr int EV_FLAG = 0x80;  // (K <= 5)

struct Chunk {
  int t0, s0;
};

__device__ __forceinline__ Chunk stage_chunk(ChunkLds& S, const Plan64Launch& a, int64_t tile, int t1, int tid) {
  const auto* word = as_global(a.words + a.tile_word[tile]);
  const int64_t tev = a.tile_ev[tile];
  const auto* evp = as_global(a.ev_ptr + tev);
  const auto* cend = as_global(reinterpret_cast<const u32x4*>(a.ev_cend) + tev);
  const auto* evs = as_global(a.ev_src);
  int t0 = t1 - CH_STEPS > 0 ? t1 - CH_STEPS : 0;
  // all of a thread's first loads at once (the guess t0 holds unless the chunk
  // has more events than its list)
  const int64_t e1 = evp[t1];
  int s0 = t0 > 0 ? t0 - 1 : 0;
  int64_t e0 = evp[s0];
  struct Row {
    uint8_t word;
    int64_t before, here, ev;
    u32x4 cols;
  };
  auto load = [&](int x) {
    // step t0 - 1 + x: its gate, and whether the step before it has events
    const int t = t0 - 1 + x < 0 ? 0 : (t0 - 1 + x < t1 ? t0 - 1 + x : t1 - 1);
    Row r;
    r.word = word[t];
    r.before = evp[t > 0 ? t - 1 : 0];
    r.here = evp[t];
    // and step s0 + x
    const int s = s0 + x < t1 ? s0 + x : t1 - 1;
    r.ev = evp[s0 + x < t1 ? s0 + x : t1];
    r.cols = cend[s];
    return r;
  };
  Row r = load(tid);
  if (uniform64(e0) + CH_EVENTS < uniform64(e1) && t1 - t0 > 1) {
    while (t1 - t0 > 1 && uniform64(evp[t0 > 0 ? t0 - 1 : 0]) + CH_EVENTS < uniform64(e1)) t0 = t1 - (t1 - t0) / 2;
    s0 = t0 > 0 ? t0 - 1 : 0;
    e0 = evp[s0];
    r = load(tid);
  }
  for (int j = tid; j < (int)(e1 - e0); j += 256) S.Ev[j] = (int32_t)evs[e0 + j];
  for (int x = tid;;) {
    if (x <= t1 - t0 && (x > 0 || t0 > 0)) S.Ws[x] = r.word | (r.here > r.before ? EV_FLAG : 0);
    if (x <= t1 - s0) S.Es[x] = (int32_t)(r.ev - e0);
    if (x < t1 - s0) S.Cc[x] = r.cols;
    x += 256;
    if (x > t1 - s0) break;
    r = load(x);
  }
  lds_barrier();
  return Chunk{t0, s0};
}

// Reverse sweep of a tile.  b_t, the adjoint of the node after step t, is
// G_{t+1}^T b_{t+1} plus the node's seed and the adjoints of the chains anchored
// there (in that order, summed first); it is stored, and G_t^T b_t with the
// events of node t-1 added becomes b_{t-1}.  The events' rows and the next gate's
// operands are loaded a step ahead.  At the end each
// chain delivers G_0^T b_0 to its anchor.
constexpr int EV_WINDOW = 3;  // events of a node held at once (more cost occupancy)
__device__ __forceinline__ void plan64_bwd_body(const Plan64Launch& a, int64_t tile) {
  __shared__ double Bs[2][16 * VST];
  __shared__ ChunkLds S;
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const int c = l & 15, r4 = l >> 4, row = 16 * w + r4;
  const int len = uniform(a.tile_len[tile]);
  const int64_t row0 = a.tile_row0[tile];
  LoadGates gs;
  gs.start(a.GAT, uniform((int)as_global(a.words + a.tile_word[tile])[len - 1]), w, l);
  int cur = 0;
  for (int t1 = len; t1 > 0;) {
    const Chunk ck = stage_chunk(S, a, tile, t1, tid);
    const int t0 = ck.t0, s0 = ck.s0, n = t1 - t0;
    // the events of node t - 1 of a step t, its first window loaded a step ahead
    NodeAdds<EV_WINDOW, 4> q;
    auto load = [&](int x) {
      q.n = 0;
      q.most = 0;
      if (x >= 0 && (uniform(S.Ws[x + 1]) & EV_FLAG))
        load_node_adds(q, S.Es, S.Ev, S.Cc, t0 + x - 1 - s0, 0, c, row, a.INJ);
    };
    if (t1 == len) {
      // b of the last node: its events alone
      NodeAdds<EV_WINDOW, 4> last;
      load_node_adds(last, S.Es, S.Ev, S.Cc, t1 - 1 - s0, 0, c, row, a.INJ);
      load(n - 1);
      double add[4];
      node_sum(last, S.Es, S.Ev, S.Cc, t1 - 1 - s0, c, row, a.INJ, add);
#pragma unroll
      for (int v = 0; v < 4; ++v) Bs[0][(4 * w + v) * VST + l] = add[v];
      lds_barrier();
    } else {
      load(n - 1);
    }
    for (int x = n - 1; x >= 0; --x) {
      const int t = t0 + x;
      const bool ev = (uniform(S.Ws[x + 1]) & EV_FLAG) != 0;
      NodeAdds<EV_WINDOW, 4> now = q;
      load(x - 1);
      const d4 acc = gs.product(a.GAT, t > 0 ? uniform(S.Ws[x]) & ~EV_FLAG : -1, Bs[cur], w, l);
      store_tile_rows(Bs[cur], a.BA + (row0 + (int64_t)t * 16) * N64, tid);
      double add[4] = {0.0, 0.0, 0.0, 0.0};
      if (ev) {
        asm volatile("" ::: "memory");  // (kept a branch: a step without events waits for no memory)
        node_sum(now, S.Es, S.Ev, S.Cc, t - 1 - s0, c, row, a.INJ, add);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Bs[cur ^ 1][(4 * w + v) * VST + l] = acc[v] + add[v];
      lds_barrier();
      cur ^= 1;
    }
    t1 = t0;
  }
  const int64_t ch = a.col_chain[tile * 16 + c];
  if (ch >= 0) {
    auto* out = as_global(a.INJ + (a.n_slots + ch) * N64 + r4);
#pragma unroll
    for (int v = 0; v < 4; ++v) out[4 * (4 * w + v)] = Bs[cur][(4 * w + v) * VST + l];
  }
}

// Four workgroups per CU (at most 128 registers): the levels of 2,636 and 1,701
// tiles 39.6 and 42.1 -> 35.9 and 40.3 us against three.
__global__ __launch_bounds__(256, 4) void plan64_bwd_kernel(const Plan64Launch a) {
  plan64_bwd_body(a, a.t_begin + blockIdx.x);
}

// ---------------------------------------------------------------------------
// Levels of long chains: a tile's sixteen chains are split over four workgroups
// of four, which need nothing of each other.  Such a level has few tiles (113 of
// up to 386 steps in a list of 200,960 sequences), and what it takes is the time
// of one step, times the longest chain.  With 16 x 16 x 4 products a step was
// sixteen dependent MFMAs of 64 cycles and an exchange of the states through
// LDS; the 4 x 4 x 4 product of four blocks (wave w: the blocks are its rows
// 16w + 4b .. + 3, the columns the workgroup's four) takes 22 cycles in a dependent
// chain, adds in the same ascending order, and reads the same operand layout of
// the gates.  A wave's operands of all K <= 5 gates stay in registers, a step
// picks its gate by a uniform branch, and two workgroups share a CU.  Quarters of
// a tile without chains are skipped (here and in the gradient).
// The level of that list: forward 289 -> 157 us, reverse 367 -> 190 us, a step
// about 1,000 and 1,200 cycles, of which 352 are the products and most of the rest the
// way through LDS (write, barrier, read).  Eight columns per workgroup, two
// independent products each: 168 and 224 us.
// ---------------------------------------------------------------------------
constexpr int QC = 4;       // columns of a workgroup
constexpr int QWG = 16 / QC; // workgroups per tile

struct RegGates {
  double g[5][16];
  __device__ __forceinline__ void init(const double* base, int K, int w, int l) {
#pragma unroll
    for (int k = 0; k < 5; ++k)
      if (k < K) load_ops(g[k], base + ((int64_t)k * 4 + w) * 1024, l);
  }
  // The wave's 16 x 64 block of gate k times the four columns, once all waves have
  // written theirs; B: the lane's operands, two blocks of four rows per 256 bytes.
  // The barrier stands in each case, so that the branches run while the wave's
  // own write is on its way; four reads are kept ahead of the products (all
  // eight up front delay the first product, two leave each pair waiting).
  __device__ __forceinline__ double product(int k, const d2* B) {
    constexpr int AHEAD = 4;
    d2 b[8];
    double acc = 0.0;
    switch (k) {
#define GST_P64_CASE(K)                                                                        \
  case K:                                                                                      \
    asm volatile("; gate " #K "\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");           \
    _Pragma("unroll") for (int h = 0; h < AHEAD; ++h) b[h] = B[h * 16];                        \
    __builtin_amdgcn_sched_barrier(0);                                                         \
    _Pragma("unroll") for (int h = 0; h < 8; ++h) {                                            \
      if (h + AHEAD < 8) b[h + AHEAD] = B[(h + AHEAD) * 16];                                   \
      acc = __builtin_amdgcn_mfma_f64_4x4x4f64(g[K][2 * h], b[h].x, acc, 0, 0, 0);             \
      acc = __builtin_amdgcn_mfma_f64_4x4x4f64(g[K][2 * h + 1], b[h].y, acc, 0, 0, 0);         \
      __builtin_amdgcn_sched_barrier(0);                                                       \
    }                                                                                          \
    break;
      GST_P64_CASE(0) GST_P64_CASE(1) GST_P64_CASE(2) GST_P64_CASE(3)
      default:
        GST_P64_CASE(4)
#undef GST_P64_CASE
    }
    return acc;
  }
};

// A lane's element of the workgroup's 64 x 4 states: its row, its column, its
// place in LDS, and where its operands lie.  Element (row 4kk + i, column j) lies at
// 32(kk / 2) + 8i + 2j + kk % 2, so that a lane reads its operands of two blocks kk
// at once.
struct QuarterLane {
  int row, c, at, rd;
  __device__ __forceinline__ QuarterLane(int q, int w, int l) {
    const int i = l >> 4, b = (l >> 2) & 3, j = l & 3;
    row = 16 * w + 4 * b + i;
    c = QC * q + j;
    at = (2 * w + (b >> 1)) * 32 + i * 8 + j * 2 + (b & 1);
    rd = i * 4 + j;
  }
};

__device__ __forceinline__ void plan64_fwd_long(const Plan64Launch& a, int64_t tile, int q) {
  __shared__ __align__(16) double Vs[2][N64 * QC];
  __shared__ uint8_t Ws[CH_STEPS + 1];
  if (uniform64(a.col_chain[tile * 16 + QC * q]) < 0) return;
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const QuarterLane e(q, w, l);
  RegGates gs;
  gs.init(a.GA, a.K, w, l);
  Vs[0][e.at] = as_global(a.FA)[a.col_anchor[tile * 16 + e.c] * N64 + e.row];
  const int len = uniform(a.tile_len[tile]);
  const auto* word = as_global(a.words + a.tile_word[tile]);
  auto* dst = as_global(a.FA + (a.tile_row0[tile] + e.c) * N64 + e.row);
  int cur = 0;
  for (int t0 = 0; t0 < len; t0 += CH_STEPS) {
    const int n = len - t0 < CH_STEPS ? len - t0 : CH_STEPS;
    for (int x = tid; x < n; x += 256) Ws[x] = word[t0 + x];
    lds_barrier();
    int k = uniform(Ws[0]);
    for (int x = 0; x < n; ++x) {
      const int kn = Ws[x + 1];  // (the last step's: unused)
      const double f = gs.product(k, reinterpret_cast<const d2*>(Vs[cur]) + e.rd);
      cur ^= 1;
      Vs[cur][e.at] = f;
      *dst = f;
      dst += 16 * N64;
      k = uniform(kn);
    }
  }
}

// The reverse sweep (as plan64_bwd_body); a lane stores its element of b_t when
// it is made, 128 bytes of four rows per wave and store.
__device__ __forceinline__ void plan64_bwd_long(const Plan64Launch& a, int64_t tile, int qd) {
  __shared__ __align__(16) double Bs[2][N64 * QC];
  __shared__ ChunkLds S;
  if (uniform64(a.col_chain[tile * 16 + QC * qd]) < 0) return;
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const QuarterLane e(qd, w, l);
  const int len = uniform(a.tile_len[tile]);
  RegGates gs;
  gs.init(a.GAT, a.K, w, l);
  auto* dst = as_global(a.BA + (a.tile_row0[tile] + (int64_t)(len - 1) * 16 + e.c) * N64 + e.row);
  double b = 0.0;
  int cur = 0;
  for (int t1 = len; t1 > 0;) {
    const Chunk ck = stage_chunk(S, a, tile, t1, tid);
    const int t0 = ck.t0, s0 = ck.s0;
    NodeAdds<EV_NODE, 1> q;
    if (t1 == len) {
      // b of the last node: its events alone
      load_node_adds(q, S.Es, S.Ev, S.Cc, t1 - 1 - s0, 0, e.c, e.row, a.INJ);
      b = node_add(q, 0, 0.0, 0);
      Bs[0][e.at] = b;
    }
    int k = uniform(S.Ws[t1 - t0]);
    for (int x = t1 - t0 - 1; x >= 0; --x) {
      const int kn = S.Ws[x];
      const bool ev = (k & EV_FLAG) != 0;  // events of node t0 + x - 1, loaded before the product
      if (ev) load_node_adds(q, S.Es, S.Ev, S.Cc, t0 + x - 1 - s0, 0, e.c, e.row, a.INJ);
      __builtin_nontemporal_store(b, dst);
      dst -= 16 * N64;
      b = gs.product(k & ~EV_FLAG, reinterpret_cast<const d2*>(Bs[cur]) + e.rd);
      double add = 0.0;
      if (ev) {
        // kept a branch: as a select it would have every step wait for the
        // stores before it (reverse 239 -> 192 us)
        asm volatile("" ::: "memory");
        add = node_add(q, 0, 0.0, 0);
      }
      b += add;
      cur ^= 1;
      Bs[cur][e.at] = b;
      k = uniform(kn);
    }
    t1 = t0;
  }
  const int64_t ch = a.col_chain[tile * 16 + e.c];
  if (ch >= 0) as_global(a.INJ)[(a.n_slots + ch) * N64 + e.row] = b;
}

__global__ __launch_bounds__(256, 2) void plan64_fwd_long_kernel(const Plan64Launch a) {
  plan64_fwd_long(a, a.t_begin + blockIdx.x / QWG, blockIdx.x % QWG);
}

__global__ __launch_bounds__(256, 2) void plan64_bwd_long_kernel(const Plan64Launch a) {
  plan64_bwd_long(a, a.t_begin + blockIdx.x / QWG, blockIdx.x % QWG);
}

// The gate gradient of the grouped-chain plan: one workgroup per chunk of
// tile-steps of one gate, wave w owning rows 16w .. 16w+15 of dG.  A tile-step
// contributes sum_c b_c f_c^T over its columns (quarters without chains left
// out): a quarter is one MFMA per 16 x 16 output tile.  A tile-step's 32 rows (its
// adjoints, consecutive, and the states before them, consecutive except at step
// 0, where they are the columns' anchors) are staged in LDS, the next one's loaded
// meanwhile; the chunk's rows are looked up once.
// The rows' bytes bound it (650 MB in the list of 200,960 sequences, 158 us).
// Three workgroups share a CU (their LDS), and the plan cuts the chunks so that
// whole rounds of workgroups run: 773 chunks of 64 on 768 places took 196 us, 750
// of 66 take 158 us.
constexpr int TS_CHUNK_MAX = GEMM64_TS_CHUNK_MAX;

constexpr int TS_SST = 80;  // padded row stride (doubles) of the staged rows: a half-wave's operand reads hit distinct banks

// The 32 rows of tile-step x (16 adjoint rows, then the 16 state rows before
// them), 16 bytes per thread and load, a row per 32 consecutive threads.  Rows
// from `rows` on are not defined (quarters of the tile without chains): the
// first row's bytes come in their place, and no product reads them.
__device__ __forceinline__ void load_ts_rows(d2 (&rg)[4], const double* BA, const double* FA, int64_t rb,
                                             const int32_t* rf, int rows, int tid) {
  const auto* gb = as_global(reinterpret_cast<const d2*>(BA));
  const auto* gf = as_global(reinterpret_cast<const d2*>(FA));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int item = tid + 256 * i, at = (item >> 5) & 15, j = item & 31;
    const int row = at < rows ? at : 0;
    rg[i] = item < 512 ? gb[(rb + row) * (N64 / 2) + j] : gf[(int64_t)rf[row] * (N64 / 2) + j];
  }
}

__device__ __forceinline__ void store_ts_rows(const d2 (&rg)[4], double* Sb, double* Sf, int tid) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int item = tid + 256 * i, row = (item >> 5) & 15, j = item & 31;
    double* dst = (item < 512 ? Sb : Sf) + row * TS_SST + 2 * j;
    *reinterpret_cast<d2*>(dst) = rg[i];
  }
}

__device__ __forceinline__ void gemm64_ts_body(const Gemm64TsLaunch& a, int64_t ch) {
  __shared__ int64_t Rb[TS_CHUNK_MAX];       // adjoint row of column 0 at each tile-step
  __shared__ int32_t Rf[TS_CHUNK_MAX][16];   // the columns' state rows before it (a row is 512 bytes)
  __shared__ int Rn[TS_CHUNK_MAX];           // its columns, rounded up to whole quarters
  __shared__ __align__(16) double Sb[2][16 * TS_SST];  // a tile-step's adjoint rows, double-buffered
  __shared__ __align__(16) double Sf[2][16 * TS_SST];  // its state rows
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int z = lane >> 4, ii = lane & 15;
  const int64_t x0 = a.chunk_beg[ch];
  const int n = (int)(a.chunk_end[ch] - x0);  // <= TS_CHUNK_MAX (checked on the host)
  for (int e = tid; e < n * 16; e += 256) {
    const int x = e >> 4, c = e & 15;
    const int64_t tile = a.ts_tile[x0 + x];
    const int t = a.ts_step[x0 + x];
    const int64_t r0 = a.tile_row0[tile] + (int64_t)t * 16;
    // (the sixteen threads of a tile-step run together)
    const unsigned long long live = __ballot(a.col_chain[tile * 16 + c] >= 0) >> (lane & 48) & 0xffff;
    if (c == 0) {
      Rb[x] = r0;
      Rn[x] = (__popcll(live) + 3) / 4 * 4;
    }
    Rf[x][c] = (int32_t)(t > 0 ? r0 - 16 + c : a.col_anchor[tile * 16 + c]);
  }
  __syncthreads();
  d4 acc[4];
#pragma unroll
  for (int tc = 0; tc < 4; ++tc) acc[tc] = d4{0.0, 0.0, 0.0, 0.0};
  d2 rg[4];
  if (n > 0) {
    load_ts_rows(rg, a.BA, a.FA, Rb[0], Rf[0], Rn[0], tid);
    store_ts_rows(rg, Sb[0], Sf[0], tid);
  }
  lds_barrier();
  for (int x = 0; x < n; ++x) {
    const int cur = x & 1;
    if (x + 1 < n) load_ts_rows(rg, a.BA, a.FA, Rb[x + 1], Rf[x + 1], Rn[x + 1], tid);
    const double* B = Sb[cur] + z * TS_SST + 16 * w + ii;
    const double* F = Sf[cur] + z * TS_SST + ii;
    const int rows = uniform(Rn[x]);
    double av = B[0], bv[4] = {F[0], F[16], F[32], F[48]};
    for (int r = 0; r < rows; r += 4) {
      const int rn = (r + 4 < rows ? r + 4 : 0) * TS_SST;  // the next four columns' operands
      const double an = B[rn], bn[4] = {F[rn], F[rn + 16], F[rn + 32], F[rn + 48]};
#pragma unroll
      for (int tc = 0; tc < 4; ++tc) acc[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[tc], acc[tc], 0, 0, 0);
      av = an;
#pragma unroll
      for (int tc = 0; tc < 4; ++tc) bv[tc] = bn[tc];
    }
    if (x + 1 < n) store_ts_rows(rg, Sb[cur ^ 1], Sf[cur ^ 1], tid);
    lds_barrier();
  }
  double* out = a.slab + ch * GATE64;
#pragma unroll
  for (int tc = 0; tc < 4; ++tc)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 4 * v + (lane >> 4), cc = lane & 15;
      out[(16 * w + r) * N64 + 16 * tc + cc] = acc[tc][v];
    }
}

// The root's adjoint: its seed and the chains anchored there.
__device__ __forceinline__ void root64_body(const Root64Launch& a) {
  const int j = threadIdx.x;
  if (j >= N64) return;
  double v = a.root_slot >= 0 ? a.INJ[a.root_slot * N64 + j] : 0.0;
  for (int i = 0; i < a.n_root_chains; ++i) v += a.INJ[(a.n_slots + a.root_chains[i]) * N64 + j];
  a.out[j] = v;
}

// The chunks, and in the last workgroup the root.
__global__ __launch_bounds__(256) void gemm64_ts_kernel(const Gemm64TsLaunch a, const Root64Launch root) {
  if ((int)blockIdx.x < a.n_chunks)
    gemm64_ts_body(a, blockIdx.x);
  else
    root64_body(root);
}

// Readouts per seed slot (the sequences ending at one node): p = E f, the
// objective, dL/dp, the seed E^T (sum of the slot's dL/dp), and dL/dE, for
// sixteen slots at a time on the matrix cores.  A wave takes the slot groups
// wv, wv + (waves of the launch), ... and, per group:
//   P^T = F^T E^T      (16 slots x 16 outcomes, K = 64: the slots' states as
//                       the A operand, E in registers as the B operand)
//   per (slot, outcome), in P's output layout: the objective terms and dL/dp
//   dE += D^T F        (outcomes x states, K = 16 slots)
//   S^T = D E          (slots x states, K = outcomes: the seeds)
// where D holds dL/dp (slots x outcomes).  F and D change layout through a
// small LDS tile per wave.  Lane l = 16 r4 + c owns, in an output block, rows
// 4v + r4 (v = 0..3) of column c.  Each wave writes one partial row
// [objective | 0 | dL/dE]; every sum has a fixed order.
// Its bytes would take 40 us in the list of 200,960 sequences (180,107 slots:
// their states, counts and seeds); it takes 48, 97 before the next group's loads
// ran ahead of the seeds' stores and the counts of equal words came added up
// (a second word's were three dependent loads, in most groups of sixteen).
constexpr int RO_FST = 66;  // padded row stride (doubles) of a wave's staged states
constexpr int RO_DST = 17;  // the same for its dL/dp tile
constexpr int RO_EST = 80;  // the same for the effects

// Workgroup blk of n_blocks (the waves' slot groups depend on the count, so a
// request's sums are the same in any launch that gives it n_blocks workgroups).
// PACK: the slots of a plan; otherwise slot s is the one sequence slot_seq[s],
// its state row s (a variant of its own: the choice at run time cost the plan's
// evaluation 18 us on that list).
template <bool PACK>
__device__ __forceinline__ void readout64_body(const Readout64Launch& a, int64_t blk, int64_t n_blocks) {
  __shared__ __align__(16) double Fs[READOUT64_WAVES][16 * RO_FST];
  __shared__ double Ds[READOUT64_WAVES][16 * RO_DST];
  __shared__ double Es[16 * RO_EST];
  __shared__ double Ep[16 * 64];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = l & 15, r4 = l >> 4;
  const int64_t wv = blk * READOUT64_WAVES + w;
  const int64_t nw = n_blocks * READOUT64_WAVES;
  const int M = a.M;
  const auto* gE = as_global(a.E);
  const auto* g_pack = as_global(a.slot_pack);
  const auto* g_cnt = as_global(a.slot_cnt);
  const auto* g_seq = as_global(a.slot_seq);
  const auto* g_counts = as_global(a.counts);
  const auto* g_W = as_global(a.W);
  auto* g_probs = as_global(a.probs);
  const bool grad = a.want_grad != 0;
  // E in LDS, rows beyond M zero: for S^T, and as the B operands of P^T, Ep[kk][l] = E[c][4kk + r4]
  for (int x = threadIdx.x; x < 16 * N64; x += READOUT64_WAVES * 64) {
    const int m = x >> 6, j = x & 63;
    const double e = m < M ? gE[x] : 0.0;
    Es[m * RO_EST + j] = e;
    Ep[(j >> 2) * 64 + (j & 3) * 16 + m] = e;
  }
  __syncthreads();
  d4 dE[4];
#pragma unroll
  for (int tc = 0; tc < 4; ++tc) dE[tc] = d4{0.0, 0.0, 0.0, 0.0};
  double obj = 0.0;
  unsigned nonpos = 0;
  double* Fw = Fs[w];
  double* Dw = Ds[w];
  const int64_t n_groups = (a.n_slots + 15) / 16;
  // Slot 16 gi + c: its state row (groups past the end read a row that exists)
  auto row_of = [&](int64_t gi) {
    const int64_t sc = gi * 16 + c;
    return PACK ? g_pack[4 * (sc < a.n_slots ? sc : 0)] : (sc < a.n_slots ? sc : a.n_slots - 1);
  };
  // a group's sixteen rows, read whole: two rows of 512 B per load, 16 B per lane
  d2 rv[8];
  auto load_rows = [&](int64_t rowc) {
    const auto* fa2 = as_global(reinterpret_cast<const d2*>(a.FA));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t rr = __shfl(rowc, 2 * i + (l >> 5));
      rv[i] = fa2[rr * (N64 / 2) + (l & 31)];
    }
  };
  // Slots 16 gi + 4v + r4 of the output rows: the first sequence, the range of
  // the sequences (low words, only their difference is used) and (plans) their
  // counts of outcome c added up.  Raw loads, the conditions where they are used: a
  // load whose value is used here would be waited for.
  int64_t seq_n[4];
  int beg_n[4], end_n[4];
  double cnt_n[4];
  const auto* g_pack32 = as_global(reinterpret_cast<const int32_t*>(a.slot_pack));
  auto load_slots = [&](int64_t gi) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t s = gi * 16 + 4 * v + r4, b = s < a.n_slots ? s : 0;
      if (PACK) {
        seq_n[v] = g_pack[4 * b + 1];
        beg_n[v] = g_pack32[8 * b + 4];
        end_n[v] = g_pack32[8 * b + 6];
        cnt_n[v] = g_cnt[b * M + (c < M ? c : 0)];
      } else {
        seq_n[v] = g_seq[b];
        beg_n[v] = 0;
        end_n[v] = 1;
        cnt_n[v] = 0.0;
      }
    }
  };
  int64_t row_next = 0;
  if (wv < n_groups) {
    load_rows(row_of(wv));
    load_slots(wv);
    row_next = row_of(wv + nw);
  }
  for (int64_t gi = wv; gi < n_groups; gi += nw) {
    // the rows into the wave's tile, then the A operand of P^T (elements
    // 4kk + r4) from there.  The next group's rows and slots are loaded now, and
    // the one after's row numbers: a load issued behind the seeds' stores would
    // wait for them
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<d2*>(&Fw[(2 * i + (l >> 5)) * RO_FST + 2 * (l & 31)]) = rv[i];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int64_t seq0[4];
    int many[4];
    double n0[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      seq0[v] = seq_n[v];
      many[v] = gi * 16 + 4 * v + r4 < a.n_slots ? end_n[v] - beg_n[v] : 0;
      n0[v] = 0.0;  // the counts, or the first sequence's weight
      if (many[v] > 0 && c < M) {
        if (a.mode == MODE_LOGLIK) n0[v] = PACK ? cnt_n[v] : (double)g_counts[seq0[v] * M + c];
        if (a.mode == MODE_VJP) n0[v] = g_W[seq0[v] * M + c];
      }
    }
    load_rows(row_next);
    load_slots(gi + nw);
    row_next = row_of(gi + 2 * nw);
    double fA[16];
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) fA[kk] = Fw[c * RO_FST + 4 * kk + r4];
    d4 p = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) p = __builtin_amdgcn_mfma_f64_16x16x4f64(fA[kk], Ep[kk * 64 + l], p, 0, 0, 0);
    // sequence q of the slot of row v
    auto seq_of = [&](int v, int q) {
      return q == 0 ? seq0[v] : g_seq[g_pack[4 * (gi * 16 + 4 * v + r4) + 2] + q];
    };
    double dps[4] = {0.0, 0.0, 0.0, 0.0};
    if (a.mode == MODE_LOGLIK) {
      // the sequences of a slot have one probability: their counts count together
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double N = n0[v], lp = log(p[v]), ratio = N / p[v];
        if (N > 0.0) {
          if (p[v] <= 0.0) {
            obj = INFINITY;
            for (int q = 0; q < many[v]; ++q) nonpos += g_counts[seq_of(v, q) * M + c] > 0;
          } else {
            obj -= N * lp;
            dps[v] = -ratio;
          }
        }
      }
    } else if (a.mode == MODE_VJP && c < M) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dps[v] = n0[v];
        for (int q = 1; q < many[v]; ++q) dps[v] += g_W[seq_of(v, q) * M + c];
      }
    }
    if (a.probs && c < M) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        for (int q = 0; q < many[v]; ++q) g_probs[seq_of(v, q) * M + c] = p[v];
    }
    if (!grad) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) Dw[(4 * v + r4) * RO_DST + c] = dps[v];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // dE += D^T F: A = dps (outcome c, slot 4kk + r4), B = F[slot 4kk + r4][16tc + c]
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int tc = 0; tc < 4; ++tc)
        dE[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(dps[kk], Fw[(4 * kk + r4) * RO_FST + 16 * tc + c], dE[tc], 0, 0,
                                                      0);
    // S^T = D E: A = D[slot c][outcome 4kk + r4], B = E
    double dA[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) dA[kk] = Dw[c * RO_DST + 4 * kk + r4];
    d4 st[4];
#pragma unroll
    for (int tc = 0; tc < 4; ++tc) {
      st[tc] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        if (4 * kk < M)
          st[tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(dA[kk], Es[(4 * kk + r4) * RO_EST + 16 * tc + c], st[tc], 0, 0,
                                                        0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t s = gi * 16 + 4 * v + r4;
      if (s < a.n_slots) {
        auto* out = as_global(a.INJ + s * N64 + c);
#pragma unroll
        for (int tc = 0; tc < 4; ++tc) out[16 * tc] = st[tc][v];
      }
    }
    // the tiles are rewritten by the next group
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (a.slab) {
    const int64_t Pc = 1 + N64 + (int64_t)M * N64;
    double* out = a.slab + wv * Pc;
    const double o = wave_sum(obj);
    if (l == 0) out[0] = o;
    out[1 + l] = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = 4 * v + r4;
      if (m < M)
#pragma unroll
        for (int tc = 0; tc < 4; ++tc) out[1 + N64 + m * N64 + 16 * tc + c] = dE[tc][v];
    }
  }
  const unsigned np = (unsigned)wave_sum((double)nonpos);
  if (l == 0 && np) {
    atomicAdd(a.status + 1, (unsigned long long)np);
    atomicAdd(a.nonpos, (unsigned long long)np);
  }
}

template <bool PACK>
__global__ __launch_bounds__(READOUT64_WAVES * 64) void readout64_kernel(const Readout64Launch a) {
  readout64_body<PACK>(a, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Batched forms of the grouped-chain plan kernels: request blockIdx.y (z for
// the slab sum), its arguments read before anything is stored, its own grid.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gate_prep64_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.y];
  if ((int)blockIdx.x >= q.tiles.K * PREP_WG) return;
  // the tile kernels read the operand layouts (const there); the prep writes them
  gate_prep64_body(q.G, q.rho, const_cast<double*>(q.tiles.GA), const_cast<double*>(q.tiles.GAT), q.tiles.FA,
                   nullptr, blockIdx.x);  // (the batch clears its counts together)
}

// The tile of workgroup `blk` of a level, per_tile workgroups each; -1: the level
// has none, or is of the other kind.
__device__ __forceinline__ int64_t batch_tile(const Plan64Req& q, int level, int want_long, int blk, int per_tile) {
  if (level >= q.n_levels || (int)q.level_long[level] != want_long) return -1;
  const int64_t t = q.level_tile[level] + blk / per_tile;
  return t < q.level_tile[level + 1] ? t : -1;
}

__global__ __launch_bounds__(256) void plan64_fwd_batch(const Plan64Req* r, int level) {
  const Plan64Req& q = r[blockIdx.y];
  const int64_t t = batch_tile(q, level, 0, blockIdx.x, 1);
  if (t < 0) return;
  const Plan64Launch a = q.tiles;
  plan64_fwd_body(a, t);
}

__global__ __launch_bounds__(256, 2) void plan64_fwd_long_batch(const Plan64Req* r, int level) {
  const Plan64Req& q = r[blockIdx.y];
  const int64_t t = batch_tile(q, level, 1, blockIdx.x, QWG);
  if (t < 0) return;
  const Plan64Launch a = q.tiles;
  plan64_fwd_long(a, t, blockIdx.x % QWG);
}

__global__ __launch_bounds__(256, 4) void plan64_bwd_batch(const Plan64Req* r, int level) {
  const Plan64Req& q = r[blockIdx.y];
  const int64_t t = q.want_grad ? batch_tile(q, level, 0, blockIdx.x, 1) : -1;
  if (t < 0) return;
  const Plan64Launch a = q.tiles;
  plan64_bwd_body(a, t);
}

__global__ __launch_bounds__(256, 2) void plan64_bwd_long_batch(const Plan64Req* r, int level) {
  const Plan64Req& q = r[blockIdx.y];
  const int64_t t = q.want_grad ? batch_tile(q, level, 1, blockIdx.x, QWG) : -1;
  if (t < 0) return;
  const Plan64Launch a = q.tiles;
  plan64_bwd_long(a, t, blockIdx.x % QWG);
}

__global__ __launch_bounds__(READOUT64_WAVES * 64) void readout64_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.y];
  const int nb = q.ro_blocks;
  if ((int)blockIdx.x >= nb) return;
  const Readout64Launch a = q.ro;
  readout64_body<true>(a, blockIdx.x, nb);
}

__global__ __launch_bounds__(256) void gemm64_ts_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.y];
  if (!q.want_grad || (int)blockIdx.x > q.gemm.n_chunks) return;
  if ((int)blockIdx.x < q.gemm.n_chunks) {
    const Gemm64TsLaunch a = q.gemm;
    gemm64_ts_body(a, blockIdx.x);
  } else {
    const Root64Launch a = q.root;
    root64_body(a);
  }
}

__global__ __launch_bounds__(256) void slab_sum64_stage1_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.z];
  if (!q.slab || (int64_t)blockIdx.x * 64 >= q.P || (int)blockIdx.y >= q.red_parts) return;
  slab_sum_stage1(q.slab, q.n_slabs, q.P, q.red_per, q.part, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void slab_sum64_stage2_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.y];
  if (!q.slab || (int64_t)blockIdx.x * 64 >= q.P) return;
  slab_sum_stage2(q.part, q.red_parts, q.P, q.objective, q.grad, q.extra_rho, N64, blockIdx.x);
}

__global__ __launch_bounds__(256) void reduce64_batch(const Plan64Req* r) {
  const Plan64Req& q = r[blockIdx.y];
  if (!q.want_grad || !q.r64.grad || (int64_t)blockIdx.x * 64 >= (int64_t)q.r64.K * GATE64) return;
  const Reduce64Launch a = q.r64;
  reduce64_body(a, blockIdx.x);
}

}  // namespace

hipError_t launch_gate_prep64(const double* G, const double* rho, int K, double* GA, double* GAT, double* FA,
                              unsigned long long* nonpos, hipStream_t stream) {
  if (K < 1) return hipErrorInvalidValue;
  gst_launch(gate_prep64_kernel, dim3(K * PREP_WG), dim3(256), 0, stream, G, rho, GA, GAT, FA, nonpos);
  return hipGetLastError();
}

hipError_t launch_gemm64_ts(const Gemm64TsLaunch& a, const Root64Launch& root, hipStream_t stream) {
  if (a.n_chunks < 0) return hipErrorInvalidValue;
  gst_launch(gemm64_ts_kernel, dim3(a.n_chunks + 1), dim3(256), 0, stream, a, root);
  return hipGetLastError();
}

hipError_t launch_plan64_fwd(const Plan64Launch& a, int n_tiles, bool long_chains, hipStream_t stream) {
  if (n_tiles <= 0) return hipSuccess;
  if (a.K < 1 || a.K > 5) return hipErrorInvalidValue;
  if (long_chains)
    gst_launch(plan64_fwd_long_kernel, dim3(QWG * n_tiles), dim3(256), 0, stream, a);
  else
    gst_launch(plan64_fwd_kernel, dim3(n_tiles), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_plan64_bwd(const Plan64Launch& a, int n_tiles, bool long_chains, hipStream_t stream) {
  if (n_tiles <= 0) return hipSuccess;
  if (a.K < 1 || a.K > 5) return hipErrorInvalidValue;
  if (long_chains)
    gst_launch(plan64_bwd_long_kernel, dim3(QWG * n_tiles), dim3(256), 0, stream, a);
  else
    gst_launch(plan64_bwd_kernel, dim3(n_tiles), dim3(256), 0, stream, a);
  return hipGetLastError();
}

int gemm64_ts_blocks_per_cu() {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm64_ts_kernel, 256, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

int readout64_blocks_per_cu() {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, readout64_kernel<true>, READOUT64_WAVES * 64, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_readout64(const Readout64Launch& a, int n_blocks, hipStream_t stream) {
  if (n_blocks <= 0 || a.M < 1 || a.M > 16) return hipErrorInvalidValue;
  if (a.slot_pack)
    gst_launch(readout64_kernel<true>, dim3(n_blocks), dim3(READOUT64_WAVES * 64), 0, stream, a);
  else
    gst_launch(readout64_kernel<false>, dim3(n_blocks), dim3(READOUT64_WAVES * 64), 0, stream, a);
  return hipGetLastError();
}

static bool chain64_ok(const Chain64Launch& a, int n_blocks) {
  return a.K >= 1 && a.K <= 5 && a.tile_seqs >= 1 && a.tile_seqs <= SCHED_CHAINS && a.tile_row >= 1 && n_blocks >= 1;
}

hipError_t launch_chain64_fwd(const Chain64Launch& a, int n_blocks, hipStream_t stream) {
  if (!chain64_ok(a, n_blocks) || !a.nonpos) return hipErrorInvalidValue;
  gst_launch(chain64_fwd_kernel, dim3(n_blocks), dim3(512), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_chain64_bwd(const Chain64Launch& a, int n_blocks, hipStream_t stream) {
  if (!chain64_ok(a, n_blocks) || !a.rec_f || a.M < 1 || a.M > 16) return hipErrorInvalidValue;
  gst_launch(chain64_bwd_kernel, dim3(n_blocks), dim3(512), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_gate_prep64_batch(const Plan64Req* reqs, int n, int K_max, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  if (K_max < 1 || K_max > 5) return hipErrorInvalidValue;
  gst_launch(gate_prep64_batch, dim3(K_max * PREP_WG, n), dim3(256), 0, stream, reqs);
  return hipGetLastError();
}

hipError_t launch_plan64_fwd_batch(const Plan64Req* reqs, int n, int level, int grid_x, bool long_chains,
                                   hipStream_t stream) {
  if (n <= 0 || grid_x <= 0) return hipSuccess;
  if (long_chains)
    gst_launch(plan64_fwd_long_batch, dim3(QWG * grid_x, n), dim3(256), 0, stream, reqs, level);
  else
    gst_launch(plan64_fwd_batch, dim3(grid_x, n), dim3(256), 0, stream, reqs, level);
  return hipGetLastError();
}

hipError_t launch_plan64_bwd_batch(const Plan64Req* reqs, int n, int level, int grid_x, bool long_chains,
                                   hipStream_t stream) {
  if (n <= 0 || grid_x <= 0) return hipSuccess;
  if (long_chains)
    gst_launch(plan64_bwd_long_batch, dim3(QWG * grid_x, n), dim3(256), 0, stream, reqs, level);
  else
    gst_launch(plan64_bwd_batch, dim3(grid_x, n), dim3(256), 0, stream, reqs, level);
  return hipGetLastError();
}

hipError_t launch_readout64_batch(const Plan64Req* reqs, int n, int grid_x, hipStream_t stream) {
  if (n <= 0 || grid_x <= 0) return hipSuccess;
  gst_launch(readout64_batch, dim3(grid_x, n), dim3(READOUT64_WAVES * 64), 0, stream, reqs);
  return hipGetLastError();
}

hipError_t launch_gemm64_ts_batch(const Plan64Req* reqs, int n, int chunks_max, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  gst_launch(gemm64_ts_batch, dim3(chunks_max + 1, n), dim3(256), 0, stream, reqs);
  return hipGetLastError();
}

hipError_t launch_slab_sum64_batch(const Plan64Req* reqs, int n, int grid_x, int parts_max, hipStream_t stream) {
  if (n <= 0 || grid_x <= 0) return hipSuccess;
  if (parts_max < 1 || parts_max > 64) return hipErrorInvalidValue;
  gst_launch(slab_sum64_stage1_batch, dim3(grid_x, parts_max, n), dim3(256), 0, stream, reqs);
  gst_launch(slab_sum64_stage2_batch, dim3(grid_x, n), dim3(256), 0, stream, reqs);
  return hipGetLastError();
}

hipError_t launch_reduce64_batch(const Plan64Req* reqs, int n, int grid_x, hipStream_t stream) {
  if (n <= 0 || grid_x <= 0) return hipSuccess;
  gst_launch(reduce64_batch, dim3(grid_x, n), dim3(256), 0, stream, reqs);
  return hipGetLastError();
}

hipError_t launch_head_sum64(const HeadSum64& a, const Reduce64Launch& gates, hipStream_t stream) {
  if (a.n_rows < 1 || a.n_part < 1 || a.n_part > 64 || (int64_t)a.per * a.n_part < a.n_rows) return hipErrorInvalidValue;
  const unsigned head = (unsigned)((a.P + 63) / 64);
  gst_launch(head_sum64_stage1, dim3(head, (unsigned)a.n_part), dim3(256), 0, stream, a);
  gst_launch(head_sum64_stage2, dim3(head + (gates.grad ? gates.K * (GATE64 / 64) : 0)), dim3(256), 0, stream, a, gates);
  return hipGetLastError();
}

hipError_t launch_reduce64(const Reduce64Launch& a, hipStream_t stream) {
  const int64_t Y = (int64_t)a.K * GATE64;
  if (Y == 0 || !a.grad) return hipSuccess;
  gst_launch(reduce64_kernel, dim3((unsigned)((Y + 63) / 64)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace gst
