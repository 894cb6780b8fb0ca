// One tile of a grouped schedule (see gst_sched.hip), as the program of a wave:
// written against the lanes' exchanges (`Lanes`) and the staged window of the words
// (`Win`), so that it also runs on the CPU with every access to the window checked.
#pragma once
#include <stdint.h>

#include "gst_internal.h"

namespace gst {

constexpr int SCHED_WINDOW = 512;  // steps of every word staged at a time

// Adds to `rank` whether the chain D lanes further round the row waits for the
// same gate (bits 28..31 of the key) with a larger key.
template <int D, class Lanes>
__host__ __device__ inline void rank_against(const Lanes& wave, uint32_t key, int& rank) {
  const uint32_t other = wave.template round<D>(key);
  rank += (other - key - 1u) < (1u << 28) - 1u && (other >> 28) == (key >> 28) ? 1 : 0;
}

template <class Win, class Lanes>
__host__ __device__ inline void sched_tile(const SchedBuild& a, int64_t tile, Win& words, const Lanes& wave) {
  const int lane = wave.lane(), c = lane & 15;
  const bool chain = lane < SCHED_CHAINS;  // the other lanes only stage
  const int64_t q0 = tile * a.tile_seqs;
  const int n = (int)(q0 + a.tile_seqs < a.S ? a.tile_seqs : a.S - q0);
  int64_t beg = 0;
  int len = 0;
  if (c < n) {
    const int64_t seq = a.order[q0 + c];
    beg = a.off[seq];
    len = (int)(a.off[seq + 1] - beg);
  }
  auto least = [](int x, int y) { return x < y ? x : y; };
  const int longest = wave.first(len);  // the order is by length, descending
  uint32_t* out = a.entries + sched_at(a.tile_rec[tile], tile);
  int e = 0;
  int pos = 0;
  if (n == 1) {
    // one chain: a round per step, its second entry empty (a word of 100 gates took
    // 90 us entry by entry)
    const int64_t b = wave.from(beg, 0);
    for (int t = lane; t < longest; t += 64) {
      out[2 * t] = ((uint32_t)a.gates[b + t] << 24) | (SCHED_NONE & ~63u) | (uint32_t)(t & 1);
      out[2 * t + 1] = SCHED_NONE;
    }
    e = 2 * longest;
    if (e % SCHED_ALIGN) {
      if (lane < 2) out[e + lane] = SCHED_NONE;
      e += 2;
    }
    if (lane == 0) a.tile_n[tile] = e;
    return;
  }
  for (int w0 = 0; w0 < longest; w0 += SCHED_WINDOW) {
    wave.sync();
    for (int x = 0; x < n; ++x) {
      const int64_t b = wave.from(beg, x) + w0;
      const int m = least(wave.from(len, x) - w0, SCHED_WINDOW);
      for (int t = lane; t < m; t += 64) words.put(x, t, a.gates[b + t]);
    }
    wave.sync();
    const int stop = least(len, w0 + SCHED_WINDOW);
    int g = chain && pos < stop ? (int)words.get(c, pos - w0) : 15;
    for (;;) {
      const bool on = chain && pos < stop;
      if (!wave.ballot(on)) break;
      // rank among the chains with the same gate: most steps left first
      const uint32_t key = ((uint32_t)g << 28) | ((uint32_t)least(len - pos, (1 << 24) - 1) << 4) | (uint32_t)(15 - c);
      int rank = 0;
      rank_against<1>(wave, key, rank);
      rank_against<2>(wave, key, rank);
      rank_against<3>(wave, key, rank);
      rank_against<4>(wave, key, rank);
      rank_against<5>(wave, key, rank);
      rank_against<6>(wave, key, rank);
      rank_against<7>(wave, key, rank);
      rank_against<8>(wave, key, rank);
      rank_against<9>(wave, key, rank);
      rank_against<10>(wave, key, rank);
      rank_against<11>(wave, key, rank);
      rank_against<12>(wave, key, rank);
      rank_against<13>(wave, key, rank);
      rank_against<14>(wave, key, rank);
      rank_against<15>(wave, key, rank);
      // a round's two entries: twice the gate that most chains wait for
      bool left = on, taken = false;
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        int best = 0, most = 0;
        for (int k = 0; k < a.K; ++k) {
          const int m = __builtin_popcountll(wave.ballot(left && g == k));
          best = m > most ? k : best;
          most = m > most ? m : most;
        }
        const bool take = left && g == best && rank < SCHED_COLS;
        uint32_t entry = (uint32_t)best << 24;
#pragma unroll
        for (int r = 0; r < SCHED_COLS; ++r) {
          const unsigned long long m = wave.ballot(take && rank == r);
          const unsigned long long odd = wave.ballot(take && rank == r && (pos & 1));
          const uint32_t id = m ? (uint32_t)__builtin_ctzll(m) : (uint32_t)SCHED_CHAINS;
          entry |= (id * 2u + (odd ? 1u : 0u)) << (6 * r);
        }
        if (lane == 0) out[e] = entry;
        ++e;
        if (left && g == best) rank -= SCHED_COLS;  // the gate's next four, if it is taken twice
        left = left && !take;
        taken = taken || take;
      }
      if (taken) {
        ++pos;
        g = pos < stop ? (int)words.get(c, pos - w0) : 15;
      }
    }
  }
  // the reverse sweeps run whole groups of entries
  const uint32_t none = SCHED_NONE;
  for (; e % SCHED_ALIGN; ++e)
    if (lane == 0) out[e] = none;
  if (lane == 0) a.tile_n[tile] = e;
}

}  // namespace gst
