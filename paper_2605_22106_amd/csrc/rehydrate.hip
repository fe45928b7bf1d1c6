// arbor_rehydrate: lazy rehydration of evicted blocks that re-enter Path*
// (Sec. 4 "Lazy rehydration"; Alg. 2 Transition branch).  The token span of a
// block is never discarded; its K/V record lives in a token-major host store
// [N][L][Hkv][D] that the kernels read directly over the host link.
//
// Launches on one stream:
//   plan     one workgroup: pages needed per node, (node, page)-ordered pop
//            offsets, ENOPAGES check before any change, new free-stack top;
//   move     kSegs waves per (node, layer, kv head) plane: the first moves the
//            resident rows to slot = position (higher slots only, so chunks are
//            staged in registers and walked from the top) and then copies the
//            evicted rows below the former count from the store; the others
//            copy those above it, whose slots held no row;
//   finalize new page-table entries, slot_pos = identity, c_i = n_i.
// The moves read the old bookkeeping (a popped page is read off the free
// stack), which only the last launch changes.
#include "arbor_internal.h"
#include "walk_stats.h"

namespace arbor {

namespace {

__global__ __launch_bounds__(1024) void rehyd_plan(Tree t, Pool pl, const uint8_t *__restrict__ on_path,
                                                   int32_t *__restrict__ pop_base,
                                                   int32_t *__restrict__ todo,
                                                   int32_t *__restrict__ meta,
                                                   const int32_t *__restrict__ k,
                                                   int64_t *__restrict__ row, int32_t *status) {
  if (blockIdx.x == 1) {
    // a walk's event: its statistics read nothing that the plan changes, so
    // they run beside it (a launch of their own ahead of the plan took 7 to 8.5
    // us on 9,841 blocks)
    walk_stats_body(t, k, on_path, 0, 1, 1, row, status);
    return;
  }
  __shared__ int64_t sm[2 * 16];
  if (status_failed(status)) {
    if (threadIdx.x == 0) meta[0] = meta[2] = 0;
    return;
  }
  const int P = pl.P;
  // each thread takes a run of consecutive blocks (their path flags loaded
  // eight at a time; only Path* blocks load their sizes), and one scan
  // places the runs, so the blocks are listed in ascending id
  constexpr int kGrp = 8;
  const int nt = blockDim.x;
  const int per = (t.V + nt - 1) / nt;
  const int r0 = min(t.V, (int)threadIdx.x * per), r1 = min(t.V, r0 + per);
  auto need_of = [&](int i) -> int64_t {
    const int n = t.n_full[i], c = t.n_kept[i];
    return c < n ? (int64_t)((n + P - 1) / P - (c + P - 1) / P) : -1;   // -1: nothing to restore
  };
  int64_t my_pages = 0, my_nodes = 0;
  for (int ib = r0; ib < r1; ib += kGrp) {
    uint8_t f[kGrp];
#pragma unroll
    for (int u = 0; u < kGrp; ++u) f[u] = ib + u < r1 ? on_path[ib + u] : 0;
#pragma unroll
    for (int u = 0; u < kGrp; ++u) {
      if (f[u]) {
        const int64_t nd = need_of(ib + u);
        if (nd >= 0) {
          my_pages += nd;
          ++my_nodes;
        }
      }
    }
  }
  const int64_t v[2] = {my_pages, my_nodes};
  int64_t ex[2], tot[2];
  block_exclusive_scan_n<2>(v, ex, tot, sm);
  const int64_t run_pages = tot[0], run_nodes = tot[1];
  int64_t op = ex[0], on = ex[1];
  for (int ib = r0; ib < r1 && my_nodes > 0; ib += kGrp) {
    uint8_t f[kGrp];
#pragma unroll
    for (int u = 0; u < kGrp; ++u) f[u] = ib + u < r1 ? on_path[ib + u] : 0;
#pragma unroll
    for (int u = 0; u < kGrp; ++u) {
      if (f[u]) {
        const int64_t nd = need_of(ib + u);
        if (nd >= 0) {
          pop_base[ib + u] = (int32_t)op;
          todo[on] = ib + u;
          op += nd;
          ++on;
        }
      }
    }
  }
  if (threadIdx.x == 0) {
    const int top = *pl.free_top;
    if (run_pages > top) {
      // nothing to move; the last launch raises the error, so that the
      // statistics beside this workgroup see the status that the event began with
      meta[0] = 0;
      meta[2] = 1;
      return;
    }
    meta[0] = (int32_t)run_nodes;
    meta[1] = top;
    meta[2] = 0;
    *pl.free_top = top - (int32_t)run_pages;
  }
}

// Where a node's rows are while it is being restored: its old pages, and the
// pages it pops from the free stack.
struct NodePages {
  const int32_t *page_table, *free_stack;
  int64_t po;
  int old_pages, pop;          // pop: stack entry of its first new page
  __device__ __forceinline__ int page(int q) const {
    return q < old_pages ? page_table[po + q] : free_stack[pop - (q - old_pages)];
  }
};

constexpr int kSegs = 4;       // waves of a plane
constexpr int kSeg = kWave;    // positions that a wave copies at a time

// Rows of one (layer, kv head) plane: LPR lanes per row, 16 bytes per lane.
// HBM-bound: each restored row is read from the store and written to the pool
// once.  A wave finds the resident positions and pages of 64 positions first,
// one per lane, so the copies wait on nothing but their rows, and the stores
// are non-temporal: 2,800 tokens of the 8B shape take 109 us instead of 222
// (with ordinary stores 193; 8 waves a plane 119, half the rows in flight 120).
template <int LPR>
__device__ void rehyd_plane(const Tree &t, const Pool &pl, const NodePages &np, int64_t tb, int n,
                            int c, int seg, int l, int g, const char *__restrict__ hk,
                            const char *__restrict__ hv, int lane) {
  constexpr int RPP = kWave / LPR;
  constexpr int PASSES = 8;
  constexpr int CH = RPP * PASSES;
  static_assert(kSeg % CH == 0, "whole chunks per segment");
  const int P = pl.P;
  char *kb = static_cast<char *>(pl.k);
  char *vb = static_cast<char *>(pl.v);
  const int sub = lane % LPR;
  const int rsel = lane / LPR;
  const int64_t row_bytes = (int64_t)pl.D * pl.esize;
  // resident rows: slot s -> slot pos(s) >= s; from the top chunk downwards
  for (int ctop = seg == 0 ? c : 0; ctop > 0; ctop -= CH) {
    uint4 kr[PASSES], vr[PASSES];
    int64_t dst[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const int s = ctop - CH + ps * RPP + rsel;
      dst[ps] = -1;
      if (s >= 0 && s < ctop) {
        const int spage = t.page_table[np.po + s / P];
        const int p = pl.slot_pos[(int64_t)spage * P + s % P];
        if (p != s) {
          const int64_t so = row_byte_offset(pl, l, spage, g, s % P) + sub * 16;
          kr[ps] = *reinterpret_cast<const uint4 *>(kb + so);
          vr[ps] = *reinterpret_cast<const uint4 *>(vb + so);
          dst[ps] = row_byte_offset(pl, l, np.page(p / P), g, p % P) + sub * 16;
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      if (dst[ps] >= 0) {
        store16_nt(kb + dst[ps], kr[ps]);
        store16_nt(vb + dst[ps], vr[ps]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // evicted rows from the token-span record, kSeg positions at a time: the
  // first wave those below the old count (their slots held the rows just
  // moved), and every wave its share of the rest
  const int64_t hstride = (int64_t)pl.L * pl.Hkv * row_bytes;
  const int64_t hoff = ((int64_t)l * pl.Hkv + g) * row_bytes + sub * 16;
  const int low = (c + kSeg - 1) / kSeg;
  const int n_seg = (n + kSeg - 1) / kSeg;
  const int own = (seg + kSegs - 1) % kSegs;       // the first wave's turn comes last
  // position of resident slot s; the positions ascend with the slots
  auto pos_of = [&](int s) __attribute__((always_inline)) -> int {
    const int spage = t.page_table[np.po + s / P];
    return pl.slot_pos[(int64_t)spage * P + s % P];
  };
  const int e_first = seg == 0 && low > 0 ? 0 : low + own;
  // a slot at most 64 before the first one of the wave's segments, by 64 probes a
  // round; later segments go on from where the last one ended, so a block's
  // slots are visited once (all of them for every segment: a transition of blocks
  // of 32,768 tokens took 137 ms, now 26)
  int s_lo = 0;
  for (int left = e_first > 0 && e_first < n_seg ? c : 0; left > kWave;) {
    const int step = (left + kWave - 1) / kWave;
    const bool probe = lane * step < left;
    const int below = popc(ballot(probe && pos_of(s_lo + (probe ? lane * step : 0)) <
                                               e_first * kSeg));
    if (below == 0) break;
    const int skip = (below - 1) * step;
    s_lo += skip;
    left = min(step, left - skip);
  }
  for (int e = e_first; e < n_seg;
       e = e + 1 < low ? e + 1 : (e < low ? low + own : e + kSegs)) {
    const int p0 = e * kSeg, p = p0 + lane;
    // lane j: position p0 + j's page, and whether it is resident
    const int page = p < n ? np.page(p / P) : 0;
    uint64_t kept = 0;
    for (int s0 = s_lo; s0 < c; s0 += kWave) {
      const int s = s0 + lane;
      const int pos = s < c ? pos_of(s) : INT32_MAX;
      const bool in = pos >= p0 && pos < p0 + kSeg;
      if (ballot(in))
        kept |= wave_allreduce(in ? 1ull << (pos - p0) : 0ull,
                               [](uint64_t x, uint64_t y) { return x | y; });
      const int below = popc(ballot(pos < p0 + kSeg));
      s_lo = s0 + below;
      if (below < kWave) break;
    }
    const uint64_t need = ballot(p < n) & ~kept;
    const char *sk = hk + (tb + p0) * hstride + hoff, *sv = hv + (tb + p0) * hstride + hoff;
    for (int j0 = 0; j0 < kSeg && p0 + j0 < n; j0 += CH) {
      uint4 kr[PASSES], vr[PASSES];
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const int j = j0 + ps * RPP + rsel;
        if ((need >> j) & 1) {
          kr[ps] = *reinterpret_cast<const uint4 *>(sk + j * hstride);
          vr[ps] = *reinterpret_cast<const uint4 *>(sv + j * hstride);
        }
      }
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const int j = j0 + ps * RPP + rsel;
        const int pj = __shfl(page, j, kWave);
        if ((need >> j) & 1) {
          const int64_t d = row_byte_offset(pl, l, pj, g, (p0 + j) % P) + sub * 16;
          store16_nt(kb + d, kr[ps]);
          store16_nt(vb + d, vr[ps]);
        }
      }
    }
  }
}

template <int LPR>
__global__ __launch_bounds__(256) void rehyd_move(Tree t, Pool pl, const char *__restrict__ hk,
                                                  const char *__restrict__ hv,
                                                  const int32_t *__restrict__ pop_base,
                                                  const int32_t *__restrict__ todo,
                                                  const int32_t *__restrict__ meta,
                                                  int32_t *status) {
  if (status_failed(status)) return;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int planes = pl.L * pl.Hkv;
  const int64_t total = (int64_t)meta[0] * planes * kSegs;
  const int top = meta[1];
  // the planes of one token lie side by side in the store: plane innermost
  for (int64_t w = (int64_t)blockIdx.x * 4 + wave; w < total; w += (int64_t)gridDim.x * 4) {
    const int i = todo[w / ((int64_t)planes * kSegs)];
    const int seg = (int)(w / planes % kSegs);
    const int rem = (int)(w % planes);
    const int l = rem / pl.Hkv;
    const int g = rem % pl.Hkv;
    const int n = t.n_full[i], c = t.n_kept[i];
    const NodePages np{t.page_table, pl.free_stack, t.page_off[i], (c + pl.P - 1) / pl.P,
                       top - 1 - pop_base[i]};
    const int64_t tb = t.tok_off[i];
    rehyd_plane<LPR>(t, pl, np, tb, n, c, seg, l, g, hk, hv, lane);
  }
}

__global__ __launch_bounds__(256) void rehyd_finalize(Tree t, Pool pl,
                                                      const int32_t *__restrict__ pop_base,
                                                      const int32_t *__restrict__ todo,
                                                      const int32_t *__restrict__ meta,
                                                      int32_t *status) {
  if (status_failed(status)) return;
  if (meta[2]) {
    if (blockIdx.x == 0 && threadIdx.x == 0) status_error(status, ARBOR_ENOPAGES);
    return;
  }
  const int lane = lane_id();
  const int P = pl.P;
  const int top = meta[1];
  for (int w = blockIdx.x * 4 + (threadIdx.x >> 6); w < meta[0]; w += gridDim.x * 4) {
    const int i = todo[w];
    const int n = t.n_full[i], c = t.n_kept[i];
    const NodePages np{t.page_table, pl.free_stack, t.page_off[i], (c + P - 1) / P,
                       top - 1 - pop_base[i]};
    const int n_pages = (n + P - 1) / P;
    for (int s = lane; s < n_pages * P; s += kWave)
      pl.slot_pos[(int64_t)np.page(s / P) * P + s % P] = s < n ? s : -1;
    for (int q = np.old_pages + lane; q < n_pages; q += kWave) t.page_table[np.po + q] = np.page(q);
    if (lane == 0) t.n_kept[i] = n;
  }
}

}  // namespace

size_t rehydrate_workspace(const arbor_sizes_t *sz) {
  return (size_t)sz->num_nodes * 8 + 4096;
}

// stats_k, stats_row: the keep-counts and the statistics row of a walk's
// Transition event (NULL: no statistics).
int launch_rehydrate(const arbor_geom_t *geom, arbor_tree_t *tree, arbor_pool_t *pool,
                     const uint8_t *on_path, const void *host_k, const void *host_v,
                     int32_t *status, void *workspace, size_t workspace_bytes,
                     hipStream_t stream, const int32_t *stats_k, int64_t *stats_row) {
  Tree t = make_tree(tree);
  Pool pl = make_pool(geom, pool);
  if (t.V <= 0) return ARBOR_OK;
  Carve cv(workspace, workspace_bytes);
  int32_t *pop_base = cv.take<int32_t>(t.V);
  int32_t *todo = cv.take<int32_t>(t.V);
  int32_t *meta = cv.take<int32_t>(4);
  if (!cv.ok) return ARBOR_EWORKSPACE;
  const dim3 node_grid((t.V + 3) / 4 < 4096 ? (t.V + 3) / 4 : 4096);
  hipLaunchKernelGGL(rehyd_plan, dim3(stats_row ? 2 : 1), dim3(1024), 0, stream, t, pl, on_path,
                     pop_base, todo, meta, stats_k, stats_row, status);
  const int64_t planes = (int64_t)t.V * pl.L * pl.Hkv * kSegs;
  const int move_blocks = (int)((planes + 3) / 4 < 8192 ? (planes + 3) / 4 : 8192);
  const int row_bytes = pl.D * pl.esize;
#define ARBOR_MOVE_LAUNCH(LPR)                                                                  \
  hipLaunchKernelGGL(rehyd_move<LPR>, dim3(move_blocks), dim3(256), 0, stream, t, pl,            \
                     static_cast<const char *>(host_k), static_cast<const char *>(host_v),       \
                     pop_base, todo, meta, status)
  if (row_bytes == 128) ARBOR_MOVE_LAUNCH(8);
  else if (row_bytes == 256) ARBOR_MOVE_LAUNCH(16);
  else ARBOR_MOVE_LAUNCH(32);
#undef ARBOR_MOVE_LAUNCH
  hipLaunchKernelGGL(rehyd_finalize, node_grid, dim3(256), 0, stream, t, pl, pop_base, todo, meta,
                     status);
  return hip_ok(hipGetLastError());
}

}  // namespace arbor
