// Batched evaluation of many requests in one persistent launch.
//
// Work is cut into tiles; a tile is a run of sequences of ONE request (the
// request's sequences sorted by length, cut into tiles of a size fixed by the
// request alone).  Workgroups take tiles from an atomic queue; the gate set of
// a tile's request is staged into LDS when it differs from the one already
// there.  Every tile writes its own slab of partial sums, and each request's
// slabs are added in tile order afterwards, so a request's results do not
// depend on which workgroup ran which tile, nor on the other requests of the
// batch.
//
// The per-sequence work is that of the plain sequence kernel (gst_seq.h).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gst_device.h"
#include "gst_internal.h"
#include "gst_seq.h"

namespace gst {
namespace {

// The tile index a workgroup works on sits in the last 16 bytes.  (A static
// __shared__ variable would be placed before the dynamic area and shift it
// off the 16-byte alignment that the row reads of ds_read_b128 need.)
__host__ __device__ inline size_t batch_lds_core(int K) { return (seq_lds_bytes(K) + 15) / 16 * 16; }
__host__ __device__ inline size_t batch_lds_bytes(int K) { return batch_lds_core(K) + 16; }

template <int D, int KT, bool PRE>
__global__ __launch_bounds__(256, seq_waves(PRE)) void batch_kernel(const BatchLaunch a) {
  extern __shared__ double lds_raw[];
  int& tile_sh = *reinterpret_cast<int*>(reinterpret_cast<char*>(lds_raw) + batch_lds_core(a.kmax));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, team = lane >> 4;
  int staged = -1;
  const Lds s = carve(lds_raw, a.kmax);
  const int64_t gteam = ((int64_t)blockIdx.x * WAVES + wave) * TPW + team;
  double* ck = a.ckpt + gteam * a.ckpt_per_team;
  for (;;) {
    if (tid == 0) tile_sh = (int)atomicAdd(a.queue, 1u);
    __syncthreads();
    const int tile = uniform(tile_sh);
    __syncthreads();
    if (tile >= a.n_tiles) break;
    const BatchTile* tp = a.tiles + tile;
    const int req = uniform(tp->req);
    const int64_t q0 = uniform64(tp->q0);
    const int nq = (int)(uniform64(tp->q1) - q0);
    const BatchReq* rp = a.reqs ? a.reqs + req : &a.one;
    const int K = uniform(rp->K), M = uniform(rp->M), mode = uniform(rp->mode);
    const auto* g_off = as_global(uniform_ptr(rp->off));
    const auto* g_order = as_global(uniform_ptr(rp->order));
    const auto* g_gates = as_global(uniform_ptr(rp->gates));
    if (req != staged) {
      stage_gateset_compact<D>(s, rp->G, rp->E, rp->rho, K, M);  // the tile loop is short of registers
      staged = req;
    }
    const SeqArgs q{K,
                    M,
                    mode,
                    uniform(rp->want_grad) != 0,
                    g_gates,
                    as_global(uniform_ptr(rp->counts)),
                    as_global(uniform_ptr(rp->W)),
                    as_global(uniform_ptr(rp->probs)),
                    ck};
    SeqSums<KT> sum;
    sum.clear();
    Pairs* st = wave_pairs(lds_raw, a.kmax, wave);
    for (int x = wave * TPW + team; x - team < nq; x += WAVES * TPW) {
      const bool has = x < nq;
      const int64_t seq = has ? g_order[q0 + x] : 0;
      const int64_t beg = has ? g_off[seq] : 0;
      const int L = has ? (int)(g_off[seq + 1] - beg) : 0;
      seq_group<D, KT, PRE>(q, s, st, has, seq, g_gates + beg, L, sum);
    }
    if (sum.bad) atomicAdd(a.status + 0, (unsigned long long)sum.bad);
    if (sum.nonpos) {
      atomicAdd(a.status + 1, (unsigned long long)sum.nonpos);
      atomicAdd(a.req_nonpos + req, (unsigned long long)sum.nonpos);
    }
    if (q.grad || mode == MODE_LOGLIK) {
      write_slab<D, KT>(lds_raw + lds_main_bytes(a.kmax) / 8, sum, M, K,
                        rp->slab + (int64_t)tp->local * slab_width(D, M, K));
      __syncthreads();  // the row has been read
    }
  }
}

__global__ void queue_reset_kernel(unsigned* q, unsigned long long* req_nonpos, int n_req) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 6) q[16 * t] = 0u;  // the queues of the six tile groups (16 words apart)
  for (int r = t; r < n_req; r += gridDim.x * blockDim.x) req_nonpos[r] = 0ull;
}

// For every request: the sum of its tile slabs, in two stages whose order
// depends on the request's own tile count only, so that its sums are the same
// alone and in any batch.  Stage 1: block (item, c) adds the rows of chunk c
// (tiles [c R, c R + R)) over the item's 64 columns, as four interleaved
// partial sums combined in a fixed order, and stores the chunk sum over the
// chunk's first row (every read of that row is done before the barrier).
// Stage 2: the chunk sums in ascending c, the same way.  Many chunks per
// column block keep enough loads in flight to fill the chip; a single pass
// over all rows leaves a request of P columns with only P / 64 workgroups.
constexpr int RED_CHUNK = 32;

__device__ inline BatchReduceItem reduce_item(const BatchReduce& a, int b) {
  if (a.items) return a.items[b];
  BatchReduceItem it = a.one;
  it.col0 = (int64_t)b * 64;
  return it;
}

__global__ __launch_bounds__(256) void batch_reduce_chunks_kernel(const BatchReduce a) {
  __shared__ double red[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const BatchReduceItem it = reduce_item(a, blockIdx.x);
  const int64_t x = it.col0 + tx;
  for (int c = blockIdx.y; (int64_t)c * RED_CHUNK < it.n_tiles; c += gridDim.y) {  // uniform over the block
    const int t0 = c * RED_CHUNK, t1 = min(it.n_tiles, t0 + RED_CHUNK);
    double v = 0.0;
    if (x < it.P) {
#pragma unroll
      for (int j = 0; j < RED_CHUNK / 4; ++j) {
        const int t = t0 + ty + 4 * j;
        if (t < t1) v += it.slab[(int64_t)t * it.P + x];
      }
    }
    red[ty][tx] = v;
    __syncthreads();
    if (ty == 0 && x < it.P) it.slab[(int64_t)t0 * it.P + x] = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void batch_reduce_final_kernel(const BatchReduce a) {
  __shared__ double red[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const BatchReduceItem it = reduce_item(a, blockIdx.x);
  const int n_chunks = (it.n_tiles + RED_CHUNK - 1) / RED_CHUNK;
  const int64_t x = it.col0 + tx;
  double v = 0.0;
  if (x < it.P)
    for (int c = ty; c < n_chunks; c += 4) v += it.slab[(int64_t)c * RED_CHUNK * it.P + x];
  red[ty][tx] = v;
  __syncthreads();
  if (ty != 0 || x >= it.P) return;
  v = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
  const bool nonpos = a.req_nonpos[it.req] != 0;
  if (x == 0) {
    if (it.objective) *it.objective = nonpos ? INFINITY : v;
  } else if (it.grad && !nonpos) {
    it.grad[x - 1] = v;
  }
}

}  // namespace

// Accumulators for six gates cover the two-qubit configurations; with more the
// gate set leaves room for two workgroups per CU, and one-qubit requests come
// here with more than four gates only: those load ahead whatever their number.
// `few`: the variant that loads rows ahead.
int batch_blocks_per_cu(int D, int kmax, bool few) {
  int n = 0;
  const size_t bytes = batch_lds_bytes(kmax);
  const hipError_t e =
      D != 16    ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<4, KMAX, true>, 256, bytes)
      : kmax > 6 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<16, KMAX, true>, 256, bytes)
      : few      ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<16, 6, true>, 256, bytes)
                 : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<16, 6, false>, 256, bytes);
  return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_batch(const BatchLaunch& a, int n_blocks, hipStream_t stream) {
  const size_t bytes = batch_lds_bytes(a.kmax);
  if (a.kmax < 1 || a.kmax > KMAX) return hipErrorInvalidValue;
  if (a.D == 16 && a.kmax <= 6 && !a.few)
    gst_launch(batch_kernel<16, 6, false>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 16 && a.kmax <= 6)
    gst_launch(batch_kernel<16, 6, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 16)
    gst_launch(batch_kernel<16, KMAX, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else if (a.D == 4)
    gst_launch(batch_kernel<4, KMAX, true>, dim3(n_blocks), dim3(256), bytes, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_queue_reset(unsigned* q, unsigned long long* req_nonpos, int n_req, hipStream_t stream) {
  int blocks = (n_req + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 256) blocks = 256;
  gst_launch(queue_reset_kernel, dim3(blocks), dim3(256), 0, stream, q, req_nonpos, n_req);
  return hipGetLastError();
}

int batch_reduce_chunks(int64_t n_tiles) { return (int)((n_tiles + RED_CHUNK - 1) / RED_CHUNK); }

hipError_t launch_batch_reduce(const BatchReduce& a, int n_items, int max_chunks, hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  if (max_chunks > 0)
    gst_launch(batch_reduce_chunks_kernel, dim3(n_items, max_chunks < 65535 ? max_chunks : 65535), dim3(256), 0,
               stream, a);
  gst_launch(batch_reduce_final_kernel, dim3(n_items), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace gst
