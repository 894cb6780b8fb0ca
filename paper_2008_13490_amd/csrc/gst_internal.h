// Internal declarations shared by the host-side library code and the kernels.
#pragma once
#include <stdint.h>
#include <hip/hip_ext.h>

#include <vector>

#include "../../include/gst.h"
#include "gst_param_tables.h"
#include "gst_tiles.h"
#include <hip/hip_runtime.h>

namespace gst {

// Kernel timing.  While a LaunchTimer is installed on the calling thread,
// every launch asks it for a pair of HIP events that the runtime stamps with
// the kernel's own start and end (hipExtLaunchKernelGGL), so that no marker
// is queued between kernels.
struct LaunchTimer {
  virtual bool events(hipEvent_t* start, hipEvent_t* stop) = 0;
  virtual ~LaunchTimer() = default;
};
LaunchTimer*& launch_timer();  // per thread; null = no timing

template <typename F, typename... Args>
inline void gst_launch(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t stream, Args... args) {
  hipEvent_t a = nullptr, b = nullptr;
  if (LaunchTimer* t = launch_timer())
    if (!t->events(&a, &b)) a = b = nullptr;
  hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, stream, a, b, 0u, args...);
}


// Evaluation modes of the sequence kernel.
enum Mode : int { MODE_PROBS = 0, MODE_LOGLIK = 1, MODE_VJP = 2 };

// One launch of the sequence ("leaf") kernel: sequence q of (off, gates) starts
// at rho and applies its gates in time order.
struct LeafLaunch {
  int D, M, K;                 // D = 4^n (4, 16 or 64)
  int few;                     // the variant that loads rows ahead
  const double* rho;           // [D]
  const double* E;             // [M][D]
  const double* G;             // [K][D][D]
  int64_t n_items;
  const int64_t* off;          // [S+1]
  const uint8_t* gates;        // [off[S]]
  const int32_t* counts;       // [S][M]  (MODE_LOGLIK)
  const double* W;             // [S][M]  (MODE_VJP)
  double* probs;               // [S][M] or null
  int mode;
  int want_grad;
  int max_len;                 // longest chain of any item
  double* slab;                // [gridDim.x][P], P = 1 + D + M*D + K*D*D
  double* ckpt;                // checkpoint scratch, ckpt_per_team doubles per team
  int64_t ckpt_per_team;
  unsigned long long* status;  // [0] bad gate indices, [1] p <= 0 with N > 0
};
// The byte that the sequence kernel reads in place of a gate index past the end
// of a word: the gate set's, which exists whatever the list is (the indices of a
// list of empty words have no first byte).
__host__ __device__ inline const uint8_t* pad_index(const LeafLaunch& a) {
  return reinterpret_cast<const uint8_t*>(a.rho);
}

// Kernels of the shared-prefix plan.  Row conventions:
//   state arena FA: row 0 = rho, row 1 + j = state after trunk step j,
//                   row 1 + nTS + x = state before item step x;
//   adjoint arena BA: row j = adjoint after trunk step j,
//                     row nTS + x = adjoint after item step x.
// Items per chunk of the item kernel: each chunk has its own row of partial
// sums, so a request's sums do not depend on how many workgroups run them.
constexpr int kItemChunk = 32;

struct PlanArgs {
  int D, M, K;
  const double* rho;
  const double* E;
  const double* G;
  int64_t nTS;                   // trunk steps
  // trunks (level range t_begin..t_end)
  int64_t t_begin, t_end;
  const int64_t* trunk_ptr;      // [n_trunks + 1]
  const int64_t* trunk_anchor;   // [n_trunks] location (state after trunk step), -1 = rho
  const int32_t* trunk_src;      // [n_trunks] source-arena row of the adjoint at the anchor, -1 = rho
  // each trunk's chain as ops: bits 0..6 gate index, or jump level with bit 7
  // set; bits 8..15 the steps the op spans; op_slot = injection slot of the
  // state after the op (-1 none)
  const int64_t* op_ptr;         // [n_trunks + 1]
  const uint32_t* op_desc;
  const int32_t* op_slot;
  // items
  int64_t n_items;
  const int64_t* items;          // [n_items][4] seq, beg, end, anchor location
  const int64_t* item_step_ptr;  // [n_items + 1]
  const uint8_t* gates;          // sequence gate indices (beg/end index into it)
  const int32_t* item_src;       // [n_items] source-arena row of the item's adjoint, -1 = rho
  const uint8_t* item_kv;        // [n_items][16] the first 16 gate indices of each item's word (0 past its end)
  const int32_t* item_cnt;       // [n_items][M] the counts in item order (requests with counts)
  const int32_t* counts;
  const double* W;
  double* probs;
  int mode;
  int want_grad;
  // arenas and injections: the adjoints arriving at stored states are rows
  // of the source arena, slot by slot; inj holds each slot's sum
  double* FA;
  double* BA;
  double* src_adj;               // [source rows][D]
  const double* inj;             // [n_inj][D]
  double* slab;                  // [blocks][1 + D + M*D]: objective, dL/drho, dL/dE
  unsigned long long* status;
  unsigned long long* req_nonpos;  // optional per-request count of p <= 0 with N > 0
  // germ-power jumps (segments of period 0): each trunk's jump pattern (0 =
  // none), whose product powers the trunk kernels build in LDS
  const uint32_t* trunk_jpat;
  const uint8_t* trunk_jg3;
  const uint8_t* trunk_jlev;     // the jump levels each trunk builds
  int jump_levels;               // the most any trunk builds (sizes the LDS)
  double* jump_t;                // [n_trunks][jump_levels][16][16]: the forward sweep's jump
                                 // matrices, transposed, for the reverse sweep
  int item_blocks;               // item workgroups; the item launch adds the forward fill workgroups
  // fill tasks: the states inside each jump
  int64_t n_fill;
  const int64_t* fill_first;
  const int64_t* fill_in;
  const int32_t* fill_n;
  const uint32_t* fill_pattern;
  const uint8_t* fill_gate3;
  // batched launches only: the levels, the trunk range of each ([n_levels + 1],
  // device), the first head row of each level's reverse trunk workgroups
  // ([n_levels]), and the forward fill workgroups of the item launch
  int n_levels;
  const int64_t* lvl_trunk;
  const int64_t* lvl_head;
  int fill_blocks;
};

// inj[slot] = the sum of source-arena rows inj_ptr[slot] .. inj_ptr[slot + 1]
// - 1 (the adjoints of the items and trunks anchored at the slot's state).
struct InjectLaunch {
  int D;
  int64_t s_begin, s_end;
  const int64_t* inj_ptr;
  const double* src_adj;    // [source rows][D]
  double* inj;              // [n_inj][D]
  // batched launches only: levels (0 = no reverse sweep) and the slot range of
  // each ([n_levels + 1], device)
  int n_levels;
  const int64_t* lvl_inj;
};

constexpr int JUMP_STEPS_MAX = 255;  // steps of a germ-power jump (8 bits of its op)
// dG from the reverse sweep, as D x D tiles of one gate each.  Record chunk c adds
// sum over records r in [chunk_beg[c], chunk_end[c]) of BA[rec_b[r]] FA[rec_f[r]]^T
// into tile chunk_tile[c].  The steps inside germ-power jumps have no records: a
// jump group is up to sixteen jumps of one pattern and length n (column c the
// arena rows jump_first[16 g + c] .. + n - 1, from the state row jump_in[16 g + c];
// column 0 always exists, -1: none); its adjoints run from the jump's end back
// through the pattern, and phase ph of the pattern goes to tile jump_meta[8 g + 4 + ph].
struct GemmLaunch {
  int D, M, K;
  int64_t n_chunks;            // record chunks
  const int64_t* chunk_tile;
  const int64_t* chunk_beg;
  const int64_t* chunk_end;
  const int64_t* rec_b;
  const int64_t* rec_f;
  int64_t n_jump_groups;
  const int64_t* jump_first;   // [n_jump_groups][16]
  const int64_t* jump_in;      // [n_jump_groups][16]
  const int32_t* jump_meta;    // [n_jump_groups][8]: steps, pattern, fourth gate, 0, the phases' tiles
  const double* G;
  const double* FA;
  const double* BA;
  int64_t zero_row;            // FA rows of zeros: this one and JUMP_STEPS_MAX after it
  double* tiles;  // [tiles][D*D]: each a contribution to its gate's gradient
};
// Workgroups of the gradient launch: four jump groups each, then a record chunk each.
__host__ __device__ inline int64_t grad_blocks_for(const GemmLaunch& g) { return (g.n_jump_groups + 3) / 4 + g.n_chunks; }

// Ordered sum of the sharing plan's partial results.  Head rows hold
// [objective | dL/drho | dL/dE] (width H = 1 + D + M*D); the gradient
// kernel leaves D x D tiles, those of gate k being rows chunk_ptr[k] ..
// chunk_ptr[k+1] of `tiles`.  Output column x of the width
// P = H + K*D*D result (0: objective, x >= 1: grad[x-1]) adds the rows of its
// own region in two fixed stages.  `part` holds n_part * P doubles.
struct PlanReduce {
  int D, M, K;
  int n_head;
  const double* head;
  const double* tiles;
  int64_t chunk_ptr[9];  // K + 1 entries; K <= max_gates_for(D) <= 8
  int64_t P;
  int n_part;        // reduce_parts of the largest region
  int n_part_tiles;  // ... of the largest gate
  double* part;
  double* objective;
  double* grad;
};
// Workgroups of the first stage: (block of 64 columns, part), the blocks with head
// columns in n_part parts, the blocks of gate columns alone in n_part_tiles (sixteen
// fits: 14,144 workgroups with n_part everywhere, 4,928 now: the launch 17.0 -> 11.5 us).
__host__ __device__ inline int64_t reduce_head_blocks(const PlanReduce& r) {
  const int64_t blocks = (r.P + 63) / 64, head = (1 + r.D + (int64_t)r.M * r.D + 63) / 64;
  return head < blocks ? head : blocks;
}
__host__ __device__ inline int64_t reduce_stage1_blocks(const PlanReduce& r) {
  const int64_t head = reduce_head_blocks(r);
  return head * r.n_part + ((r.P + 63) / 64 - head) * r.n_part_tiles;
}

// Batched evaluation of many requests (persistent kernel, tile queue).
struct BatchReq {
  const double* rho;
  const double* E;
  const double* G;
  const int64_t* off;
  const uint8_t* gates;
  const int64_t* order;    // sequence order (by length, descending) or null
  const int32_t* counts;
  const double* W;
  double* probs;
  double* slab;            // [n_tiles][P] of this request
  int M, K, mode, want_grad;
};
struct BatchLaunch {
  int D;
  int kmax;
  const BatchReq* reqs;            // null: every tile belongs to `one`
  BatchReq one;
  const BatchTile* tiles;
  int n_tiles;
  int few;                         // the variant that loads rows ahead
  unsigned* queue;
  double* ckpt;
  int64_t ckpt_per_team;
  unsigned long long* status;
  unsigned long long* req_nonpos;  // [n_req]
};
struct BatchReduceItem {
  int req;
  int n_tiles;
  int64_t P;
  int64_t col0;
  double* slab;  // [n_tiles][P]; stage 1 leaves the chunk sums in the first row of each chunk
  double* objective;
  double* grad;
};
struct BatchReduce {
  const BatchReduceItem* items;    // null: block b reduces columns [64b, 64b+64) of `one`
  BatchReduceItem one;
  const unsigned long long* req_nonpos;
};
// One-qubit requests with K <= 4 gates: one chain per lane, a wave per tile
// of 64 sequences (gst_lane1q.hip).  ckpt_per_team of the launch is the
// checkpoint stride of one wave.
bool lane1q_supported(int K);
int lane1q_ckpt_per_wave(int64_t max_len);
int lane1q_blocks_per_cu(int K);
hipError_t launch_lane1q(const BatchLaunch& a, int K, int n_blocks, hipStream_t stream);
// Resident workgroups per CU of the batched kernel (occupancy with its LDS).
int batch_blocks_per_cu(int D, int kmax, bool few);
hipError_t launch_batch(const BatchLaunch& a, int n_blocks, hipStream_t stream);
hipError_t launch_queue_reset(unsigned* q, unsigned long long* req_nonpos, int n_req, hipStream_t stream);
// Chunks of the two-stage tile-slab sum for a request of n_tiles tiles; the
// launch takes the largest over its items.
int batch_reduce_chunks(int64_t n_tiles);
hipError_t launch_batch_reduce(const BatchReduce& a, int n_items, int max_chunks, hipStream_t stream);

// Grouped schedules (gst_sched.hip): tiles of up to 16 consecutive chains of a
// length-sorted order.  An entry advances up to four chains by one gate, and
// entries 2m and 2m + 1 (a round) advance different chains: bits
// 6r .. 6r + 5 hold, for column r, the chain's index in the tile times two plus
// the parity of its step (chain 16: no chain), bits 24..27 the gate.  Tile t has
// tile_n[t] entries, a multiple of SCHED_ALIGN (padded with entries without chains),
// from sched_at(tile_rec[t], t) on: a step takes a round at most.
constexpr int SCHED_CHAINS = 16, SCHED_COLS = 4, SCHED_ALIGN = 4;
constexpr uint32_t SCHED_NONE = (2u * SCHED_CHAINS) * (1u | 1u << 6 | 1u << 12 | 1u << 18);
__host__ __device__ inline int64_t sched_at(int64_t steps_before, int64_t tile) {
  return 2 * steps_before + SCHED_ALIGN * tile;
}
struct SchedBuild {
  const int64_t* off;
  const uint8_t* gates;
  const int64_t* order;      // sequences by length, descending
  int64_t S;
  int K;
  int tile_seqs;             // chains per tile (<= SCHED_CHAINS)
  const int64_t* tile_rec;   // [tiles + 1]: the steps of the tiles before
  int* tile_n;               // [tiles]
  uint32_t* entries;         // [sched_at(steps, tiles) + 1]
};
hipError_t launch_sched(const SchedBuild& a, int64_t n_tiles, hipStream_t stream);

// Three-qubit lists without shared prefixes (D = 64): tiles of a grouped
// schedule, one workgroup each (see gst_kernels64.hip).
struct Chain64Launch {
  int K;
  const double* rho;         // [64]
  const double* G;           // [K][64][64]
  const int64_t* off;        // [S+1]
  const int64_t* order;      // sequences by length, descending
  int64_t S;
  int tile_seqs;             // chains per tile (consecutive in `order`)
  int n_tiles;
  int tile_row;              // workgroups take the tiles there and back in rows of this many
  const int* tile_n;         // [n_tiles]
  const uint32_t* entries;
  const int64_t* tile_rec;   // [n_tiles + 1]: the chain-steps of the tiles before
  int zero_rec;              // all of them
  double* rec_f;             // [zero_rec + 1][64]: the states before each entry's columns with a chain, entry
                             // by entry, then a row of zeros (null: not recorded)
  double* fin;               // [S][64], in `order`: final states (forward), seeds (reverse)
  unsigned long long* nonpos;  // forward: cleared
  int M;                     // reverse: width of the head rows, 1 + 64 + 64 M
  double* head;              // reverse: [gridDim.x] head rows, [0 | dL/drho | 0]
  double* dg;                // reverse: [K][gridDim.x][4096]: each workgroup's dL/dG
};
struct Reduce64Launch {            // gate columns only
  int M, K;
  const double* chunk_slab;        // [n_chunks][4096]
  const int64_t* gate_chunk_ptr;   // [K + 1] chunk range of each gate
  double* grad;
  const unsigned long long* nonpos;
};
// Three-qubit sharing plan with grouped chains (gst_plan64.h): tiles of
// sixteen chains with one word, stepped together on the matrix cores.
struct Plan64Launch {
  const double* GA;          // [K][4][16][64]: A operands of G, GA[k][w][kk][l] = G[k][16w + l%16][4kk + l/16]
  const double* GAT;         // [K][4][16][64]: the same for G^T
  int64_t t_begin;           // first tile of the launch (one workgroup per tile)
  const int64_t* tile_row0;
  const int32_t* tile_len;
  const int64_t* tile_word;
  const int64_t* tile_ev;
  const int64_t* col_anchor; // [n_tiles][16]
  const int64_t* col_chain;  // [n_tiles][16]
  const uint8_t* words;
  const int64_t* ev_ptr;
  const uint8_t* ev_cend;    // [tile-steps][16]: byte c < 15 the step's events of columns <= c, byte 15 the most of one column
  const int64_t* ev_src;     // < 2^31
  double* FA;                // [n_rows][64], row 0 = rho
  double* BA;                // [n_rows][64]
  double* INJ;               // [n_slots + n_chains][64]
  int64_t n_slots;
  int K;                     // gates (<= 5)
};
// dG over tile-steps: chunk c adds, for its gate, over its tile-steps (tile,
// t), sum over the tile's 16 columns of BA[row(c, t)] FA[row(c, t - 1)]^T (row
// t - 1 = -1: the column's anchor).
struct Gemm64TsLaunch {
  const double* BA;
  const double* FA;
  const int64_t* tile_row0;
  const int64_t* col_anchor;
  const int64_t* col_chain;  // -1: no chain (columns are filled from the first)
  const int64_t* ts_tile;
  const int32_t* ts_step;
  const int64_t* chunk_beg;
  const int64_t* chunk_end;
  double* slab;              // [n_chunks][4096]
  int n_chunks;
};
constexpr int GEMM64_TS_CHUNK_MAX = 96;  // tile-steps per chunk at most (staged in LDS)
int gemm64_ts_blocks_per_cu();
constexpr int READOUT64_WAVES = 4;
struct Readout64Launch {
  int M;
  const double* E;
  const double* FA;
  int64_t n_slots;
  const int64_t* slot_seq;
  const int64_t* slot_pack;  // [n_slots][4]: node row, first sequence, the slot's range in slot_seq
                             // (null: slot s is the one sequence slot_seq[s], its state row s)
  const double* slot_cnt;    // [n_slots][M]: the counts of the slot's sequences added up (null without a plan)
  const int32_t* counts;
  const double* W;
  double* probs;
  int mode, want_grad;
  double* INJ;               // seeds: rows 0 .. n_slots-1
  double* slab;              // [waves][1 + 64 + 64 M]
  unsigned long long* status;
  unsigned long long* nonpos;
};
struct Root64Launch {        // the adjoint of rho: root seed + chains anchored at rho (ascending)
  const double* INJ;
  int64_t root_slot;         // -1 none
  int64_t n_slots;
  const int64_t* root_chains;
  int n_root_chains;
  double* out;               // [64]
};
hipError_t launch_gate_prep64(const double* G, const double* rho, int K, double* GA, double* GAT, double* FA,
                              unsigned long long* nonpos, hipStream_t stream);
hipError_t launch_plan64_fwd(const Plan64Launch& a, int n_tiles, bool long_chains, hipStream_t stream);
hipError_t launch_plan64_bwd(const Plan64Launch& a, int n_tiles, bool long_chains, hipStream_t stream);
hipError_t launch_readout64(const Readout64Launch& a, int n_blocks, hipStream_t stream);
// the gradient GEMM and the root's adjoint, one launch
hipError_t launch_gemm64_ts(const Gemm64TsLaunch& a, const Root64Launch& root, hipStream_t stream);
int readout64_blocks_per_cu();

hipError_t launch_chain64_fwd(const Chain64Launch& a, int n_blocks, hipStream_t stream);
hipError_t launch_chain64_bwd(const Chain64Launch& a, int n_blocks, hipStream_t stream);
hipError_t launch_reduce64(const Reduce64Launch& a, hipStream_t stream);
struct HeadSum64 {           // ordered sum of head rows [objective | rho | E]
  const double* head;        // [n_rows][P]
  int n_rows, n_part, per;   // n_part parts of `per` rows
  int64_t P;
  double* part;              // [n_part][P]
  double* objective;
  double* grad;
};
hipError_t launch_head_sum64(const HeadSum64& a, const Reduce64Launch& gates, hipStream_t stream);

// One request of a batched launch of three-qubit grouped-chain plans: the
// arguments of its standalone launch sequence.  The batched kernels take
// request blockIdx.y (z for the slab sum), copy its arguments to registers and
// run the standalone kernels' bodies on its own grid; workgroups beyond that
// grid exit, so every request gets the bits of its standalone evaluation.
struct Plan64Req {
  Plan64Launch tiles;         // t_begin unused: the level ranges below
  const int64_t* level_tile;  // [n_levels + 1] tile ranges of the levels
  const uint8_t* level_long;  // [n_levels] 1: the level keeps the gates in registers
  int n_levels;
  int want_grad;
  const double* G;            // the gate set and rho, for the operand layouts
  const double* rho;
  Readout64Launch ro;
  int ro_blocks;
  Gemm64TsLaunch gemm;        // n_chunks = 0: no gradient GEMM
  Root64Launch root;
  // the ordered sum of the readout's wave rows (slab = null: none)
  const double* slab;
  int n_slabs, red_parts, red_per;
  int64_t P;                  // 1 + 64 + 64 M
  double* part;
  double* objective;
  double* grad;
  const double* extra_rho;    // the root adjoint, with the gradient
  Reduce64Launch r64;         // r64.grad = null: no gate columns
};
hipError_t launch_gate_prep64_batch(const Plan64Req* reqs, int n, int K_max, hipStream_t stream);
hipError_t launch_plan64_fwd_batch(const Plan64Req* reqs, int n, int level, int grid_x, bool long_chains,
                                   hipStream_t stream);
hipError_t launch_readout64_batch(const Plan64Req* reqs, int n, int grid_x, hipStream_t stream);
hipError_t launch_plan64_bwd_batch(const Plan64Req* reqs, int n, int level, int grid_x, bool long_chains,
                                   hipStream_t stream);
hipError_t launch_gemm64_ts_batch(const Plan64Req* reqs, int n, int chunks_max, hipStream_t stream);
hipError_t launch_slab_sum64_batch(const Plan64Req* reqs, int n, int grid_x, int parts_max, hipStream_t stream);
hipError_t launch_reduce64_batch(const Plan64Req* reqs, int n, int grid_x, hipStream_t stream);

hipError_t launch_trunk_fwd(const PlanArgs& a, hipStream_t stream);
hipError_t launch_trunk_bwd(const PlanArgs& a, hipStream_t stream);
hipError_t launch_items(const PlanArgs& a, int n_blocks, hipStream_t stream);
// Workgroups of the item launch: one per 16 items, at most max_blocks (> 0);
// item_blocks_per_cu is the kernel's occupancy.  The launch adds
// fill_blocks_for(n_fill) workgroups of forward fill tasks when it has them.
int item_blocks_for(int64_t n_items, int64_t max_blocks);
int item_blocks_per_cu(int D, int K, int M);
int fill_blocks_for(int64_t n_fill);
int trunk_blocks_for(int64_t n_trunks);
hipError_t launch_inject(const InjectLaunch& a, hipStream_t stream);
hipError_t launch_grad_gemm(const GemmLaunch& a, hipStream_t stream);
hipError_t launch_reduce_plan(const PlanReduce& a, hipStream_t stream);

// The plans of n requests with the same D in one launch per kernel: request y
// takes args[y], inject[y], gemm[y], reduce[y] (device arrays).  Each launch
// spans the most workgroups any request's standalone launch has (grid_x);
// K_max and jl_max size the LDS.  The sequence is: trunk_fwd per level
// ascending, items, then (inject, trunk_bwd) per level descending,
// grad_gemm, reduce.
struct PlanBatch {
  const PlanArgs* args;
  const InjectLaunch* inject;
  const GemmLaunch* gemm;
  const PlanReduce* reduce;
};
hipError_t launch_trunk_fwd_batch(const PlanBatch& b, int D, int n, int level, int grid_x, int K_max, int jl_max,
                                  hipStream_t stream);
hipError_t launch_items_batch(const PlanBatch& b, int D, int n, int grid_x, int K_max, int M_max,
                              hipStream_t stream);
hipError_t launch_inject_batch(const PlanBatch& b, int n, int level, int grid_x, hipStream_t stream);
hipError_t launch_trunk_bwd_batch(const PlanBatch& b, int D, int n, int level, int grid_x, int K_max, int jl_max,
                                  hipStream_t stream);
hipError_t launch_grad_gemm_batch(const PlanBatch& b, int D, int n, int grid_x, hipStream_t stream);
hipError_t launch_reduce_plan_batch(const PlanBatch& b, int n, int grid_x, int stage1_x, hipStream_t stream);
// Predictions of repeated gate applications: V = block-start states
// [n_pairs][Q][D], probs [n_pairs][r_max + 1][M]; pair = preparation * n_gates + gate.
// Few short preparation words travel in the kernels' arguments (a copy to the
// device costs the host more than the kernels take: four words, five gates and r to
// 1000, the call and a distance 23.5 -> 20.8 us).
constexpr int PREDICT_PREPS = 64, PREDICT_STEPS = 512, PREDICT_GATES = 64;
struct PredictWords {
  int32_t prep_off[PREDICT_PREPS + 1];
  uint8_t prep_gates[PREDICT_STEPS];
  uint8_t gate_of[PREDICT_GATES];
};
struct PredictLaunch {
  int D, M, K;
  const double* rho;
  const double* E;
  const double* G;
  int n_pairs, n_gates;
  const int64_t* prep_off;    // [n_prep + 1]; null: the words and gates are in `words`
  const uint8_t* prep_gates;
  const int32_t* gate_of;     // [n_gates]
  PredictWords words;
  int r_max, levels, Q;       // blocks of 2^(levels-1) repetitions, Q blocks
  double* V;
  double* probs;
};
// The block-start chain (V), then the blocks with their readouts (probs).
hipError_t launch_predict_chain(const PredictLaunch& a, hipStream_t stream);
hipError_t launch_predict_fill(const PredictLaunch& a, hipStream_t stream);
hipError_t launch_tv_distance(const double* p, const double* q, int64_t n, int M, double* out, hipStream_t stream);

// Parameterizations of the gate set (TP and CPTP estimation modes).  theta and
// grad_theta in the layout of gst.h; grad_full = [rho | effects | gates].
struct ParamLaunch {
  int mode;          // 1 = TP, 2 = CPTP
  int n, D, d, M, K;
  double sqrt_d, inv_sqrt_d;
  const double* theta;
  const double* targets;    // CPTP: G0 [K][D][D]
  const double* grad_full;  // backward
  double* rho;              // forward outputs
  double* E;
  double* G;
  double* grad_theta;       // backward output
  const double* ty;         // CPTP structure tables of the generator (D <= 16):
  const double* tzr;        //   y [D][D], z [D (j)][D][D] (real and imaginary parts)
  const double* tzi;
};
hipError_t launch_param_forward(const ParamLaunch& a, hipStream_t stream);
hipError_t launch_param_backward(const ParamLaunch& a, hipStream_t stream);


// The allocation-free evaluation (gst_noalloc.hip): the scratch array's address
// on `device`, resolved once per device (0 or a gst_status), and gst_loglik on a
// given scratch buffer (gst_api.cpp).
int scratch_bind(int device);
int ctx_device(const gst_ctx* ctx);
int loglik_into_scratch(gst_ctx* ctx, const gst_gateset* gs, const gst_seqlist* sl, const int32_t* counts,
                        double* probs, double* objective, double* grad, void* scratch, size_t scratch_bytes);

__host__ __device__ inline int64_t slab_width(int D, int M, int K) { return 1 + D + (int64_t)M * D + (int64_t)K * D * D; }

hipError_t launch_leaf(const LeafLaunch& a, int n_blocks, hipStream_t stream);
int leaf_blocks_for(int D, int64_t n_items);
int leaf_ckpt_interval(int D);
int leaf_teams_per_block(int D);
int max_gates_for(int D);

// out[p] = sum of slab[w][p] over w (fixed two-stage order) plus extra_rho on
// the rho entries; writes objective (p = 0) and the gradient (p >= 1).  The
// kernels write +inf into their objective partial for p <= 0 with N > 0; the
// objective is then +inf and grad is left untouched.  `part` holds
// reduce_parts(n_slabs) * P doubles of scratch.
int reduce_parts(int n_slabs);
hipError_t launch_reduce(const double* slab, int n_slabs, int64_t P, double* objective, double* grad,
                         const double* extra_rho, int D, double* part, hipStream_t stream);

}  // namespace gst
