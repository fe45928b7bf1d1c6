// arbor_allocate: tree-aware keep-counts under a global token budget.
//
// Eq. 2 gives the off-path retention ratio r_i = clip(alpha w_i, r_min, 1) with
// w_i = eta s_i^gamma e^{-lambda_d d_i} e^{-lambda_Delta Delta_i}; Eq. 3 turns it
// into k_i = min(n_i, max(K_min, |T_i|, floor(r_i n_i))).  The KKT view of
// Sec. 4 sets the one global scale alpha so that the total meets the budget.
// Token j of block i is kept exactly when alpha >= j / (w_i n_i) ("price"), so
// the largest feasible alpha keeps every price below the (E+1)-th smallest one,
// E being the budget left after the floors.  Path* nodes (Alg. 2 Transition)
// are pinned at n_i; when the floors alone overflow (Alg. 2 Pressure) the
// lowest-priority blocks are drained towards K_min, found by a weighted radix
// select over the bit patterns of w_i.
//
// Finding the (E+1)-th smallest price without listing every token: the prices
// of block i are j / W_i for consecutive j, so the number of prices up to x is
// floor(x W_i) - F_i (clamped), exact up to rounding at the two ends.  A
// search over x on exact counts brackets the order statistic between two
// values whose counts lie on either side of E; only the few prices left in
// the bracket are listed and ranked (positive doubles order like their bits).
//
// Small trees (kLdsNodes) run in one 1024-thread workgroup with all per-node
// state in LDS.  Larger ones take two launches: alloc_nodes, one thread per
// block over the whole chip (geometry, floors, weights, eligible prices and
// their totals per workgroup), then alloc_cut, one workgroup (the search and
// the counts, or the Pressure drain).  fp64, no contraction, so the prices
// are the same IEEE quotients any fp64 implementation computes.
#include "arbor_internal.h"
#include "walk_stats.h"

#pragma clang fp contract(off)

namespace arbor {

namespace {

constexpr int AT = 1024;
constexpr int kLdsNodes = 512;    // per-node state in LDS up to this many nodes
constexpr int kGeoNodes = 16384;  // parent and down links in LDS up to this many
constexpr int kCandLds = 1536;    // listed prices
constexpr int kNodeBytes = 2 * 8 + 8 * 4 + 1;
constexpr int kNodeThreads = 256; // blocks of a workgroup of alloc_nodes
constexpr int kCutThreads = 512;  // threads of alloc_cut
constexpr int kRegNodes = 20;     // blocks of a thread of alloc_cut held in registers
constexpr int kCutPts = 3;        // test points of a search round
constexpr int kSnapFrom = 10, kSnapEvery = 6;   // search rounds that look for ties
constexpr int kDecay = 128;                    // tabulated depths and distances

// The decay factors exp(-lambda_d d) and exp(-lambda_Delta Delta) for small
// integer d and Delta are tabulated per call by the host with the C library's
// exp, the same doubles an fp64 reference on the host obtains, so that ties
// between prices of different nodes break the same way (a device exp may
// round the last bit differently).
struct AllocParams {
  double alpha_max, gamma, lambda_d, lambda_delta, eta, r_min;
  int k_min, l_tail;
  int rehydrate;   // Path* blocks count n_i (restored) or their resident c_i
  int k_protect;   // 0: Path* blocks pinned; > 0: they take part with this floor
  double dexp[kDecay], texp[kDecay];
};

// s^gamma, correctly rounded for the integer exponents 1..4: s is an fp32
// value, so s * s is exact in fp64 and one more product rounds once
__device__ __forceinline__ double pow_gamma(double s, double gamma) {
  if (gamma == 1.0) return s;
  if (gamma == 2.0) return s * s;
  if (gamma == 3.0) return (s * s) * s;
  if (gamma == 4.0) return (s * s) * (s * s);
  return pow(s, gamma);
}

// Per-node working state.  parent / n_full / n_kept are the tree's arrays or
// LDS copies of them; `path` is the on-path output or its LDS copy.
struct Nodes {
  int32_t *parent, *n_full, *n_kept;
  int32_t *depth, *down, *F, *cnt, *cap;
  double *W, *w;
  uint8_t *path;
};

// Totals of one workgroup of alloc_nodes.
struct NodeSums {
  int64_t path_tok, sum_F, sum_red, total;
  int64_t kmin, kmax;    // price keys of the eligible prices
  int64_t flags;         // malformed | NaN s << 21 | s outside [0, 1] << 42 (at most one
                         //   of each per workgroup)
};

// A block as alloc_cut reads it, in one 16-byte load.
struct __attribute__((aligned(16))) NodeRec {
  int32_t F, cnt;                  // F: -1 on pinned Path* blocks
  double W;                        // 1 on blocks without eligible prices
};

struct AllocWs {
  int32_t *down;
  NodeRec *rec;
  double *w;
  NodeSums *sums;                  // per workgroup of alloc_nodes
  int32_t *gated;                  // 1: a Pressure event that does not fire
};

__device__ __forceinline__ double price(int j, double W) {
  return W > 0.0 ? (double)j / W : __builtin_inf();
}

// Number of j in (F, c] whose price satisfies pred (prices ascend with j).
template <class Pred>
__device__ int count_prefix(int F, int c, double W, Pred pred) {
  int lo = F + 1, hi = c, ans = F;
  while (lo <= hi) {
    const int mid = lo + ((hi - lo) >> 1);
    if (pred(price(mid, W))) {
      ans = mid;
      lo = mid + 1;
    } else {
      hi = mid - 1;
    }
  }
  return ans - F;
}

// Largest m in [F, F + cnt] with price(m) <= x (m = F: none), starting from
// the rounded estimate floor(x W) and correcting it by exact comparisons.
// The product y = x W carries a relative error of at most 2^-53, and so does
// each quotient j / W: an integer j with j > y (1 + 2^-50) has a price above
// x, one with j < y (1 - 2^-50) a price below it.  Only an estimate that close
// to the boundary needs the divisions.
__device__ int last_le(double x, int F, int cnt, double W) {
  const double yr = x * W;
  double y = __builtin_floor(yr);
  // (a NaN estimate, 0 * inf, starts from F)
  y = !(y >= (double)F) ? (double)F : (y > (double)(F + cnt) ? (double)(F + cnt) : y);
  int m = (int)y;
  const bool up_ok = m == F + cnt || (double)(m + 1) > yr * (1.0 + 0x1p-50);
  const bool down_ok = m == F || (double)m < yr * (1.0 - 0x1p-50);
  if (up_ok && down_ok && yr < __builtin_inf()) return m;
#pragma unroll 1
  while (m < F + cnt && price(m + 1, W) <= x) ++m;
#pragma unroll 1
  while (m > F && price(m, W) > x) --m;
  return m;
}

// Largest m in [F, F + cnt] with price(m) < x (m = F: none), as last_le.
__device__ int last_lt(double x, int F, int cnt, double W) {
  const double yr = x * W;
  double y = __builtin_floor(yr);
  y = !(y >= (double)F) ? (double)F : (y > (double)(F + cnt) ? (double)(F + cnt) : y);
  int m = (int)y;
  const bool up_ok = m == F + cnt || (double)(m + 1) > yr * (1.0 + 0x1p-50);
  const bool down_ok = m == F || (double)m < yr * (1.0 - 0x1p-50);
  if (up_ok && down_ok && yr < __builtin_inf()) return m;
#pragma unroll 1
  while (m < F + cnt && price(m + 1, W) < x) ++m;
#pragma unroll 1
  while (m > F && !(price(m, W) < x)) --m;
  return m;
}

// last_le and last_lt where they agree and need no division: floor(x W),
// clamped, unless x W lies within 2^-50 of an integer (or is no number), which
// sets *near.
// (lo = F, hi = F + cnt)
__device__ __forceinline__ int last_fast(double x, double lo, double hi, double W, bool &near) {
  const double yr = x * W;
  near |= !(__builtin_fabs(yr - __builtin_rint(yr)) > yr * 0x1p-50) && !(yr >= hi + 1.0);
  return (int)__builtin_fmin(__builtin_fmax(__builtin_floor(yr), lo), hi);
}

// Eligible prices of a block: those in (F, cap] that are finite and at most
// amax.  Prices ascend with j, so when the last one qualifies they all do.
__device__ int eligible(int F, int cap, double W, double amax) {
  if (cap <= F || !(W > 0.0)) return 0;
  const double last = price(cap, W);
  if (last <= amax && last < __builtin_inf()) return cap - F;
  if (last < __builtin_inf()) return last_le(amax, F, cap - F, W) - F;
  return count_prefix(F, cap, W, [amax](double x) { return x <= amax && x < __builtin_inf(); });
}

__device__ __forceinline__ int64_t wave_min_i64(int64_t v) {
  return wave_allreduce(v, [](int64_t a, int64_t b) { return a < b ? a : b; });
}

// block-wide sums of v[0..NS) and minima of v[NS..N) in one exchange; sm
// holds 16 N values
// Threads from `live` on hold the identities, so their waves skip the
// wave-level reductions; the wave totals are combined by wave 0 alone, which
// hands the results back through sm.
template <int NS, int N>
__device__ void block_reduce_n(int64_t (&v)[N], int64_t *sm, int live) {
  const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (w * kWave < live) {
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = q < NS ? wave_sum(v[q]) : wave_min_i64(v[q]);
  }
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < N; ++q) sm[16 * q + w] = v[q];
  __syncthreads();
  if (w == 0) {
    const bool in = lane < nw;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int64_t r = q < NS ? wave_sum(in ? sm[16 * q + lane] : (int64_t)0)
                               : wave_min_i64(in ? sm[16 * q + lane] : INT64_MAX);
      if (lane == 0) sm[16 * q] = r;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = sm[16 * q];
  __syncthreads();
}

// block-wide sum of v[0] and minima of v[1], v[2] in one exchange
__device__ void block_min_sum3(int64_t (&v)[3], int64_t *sm) {
  const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v[0] = wave_sum(v[0]);
  v[1] = wave_min_i64(v[1]);
  v[2] = wave_min_i64(v[2]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) sm[16 * q + w] = v[q];
  __syncthreads();
  const bool in = lane < nw;
  v[0] = wave_sum(in ? sm[lane] : (int64_t)0);
  v[1] = wave_min_i64(in ? sm[16 + lane] : INT64_MAX);
  v[2] = wave_min_i64(in ? sm[32 + lane] : INT64_MAX);
  __syncthreads();
}

// The rank-th smallest (0-based) of the keys src[0, n), 0 <= rank < n, all of them
// in [kmin, kmax].  Keys are taken relative to kmin, and each pass splits the remaining
// range [lo, lo + span] into 256 equal power-of-two buckets: the listed prices
// are spread fairly evenly over their small range, so one pass usually leaves
// at most 64 candidates, which one wave then ranks directly.  src and dst
// (room for n keys) are both overwritten.
// Called by the whole block; contains __syncthreads.
__device__ uint64_t select_rank(uint64_t *src, uint64_t *dst, int64_t n, int64_t rank,
                                uint64_t kmin, uint64_t kmax) {
  __shared__ unsigned hist4[4 * 256];
  __shared__ int64_t s_wtot[4];
  __shared__ int s_chosen;
  __shared__ int64_t s_below;
  __shared__ unsigned s_ncand;
  __shared__ uint64_t s_key;
  const int tid = threadIdx.x, lane = lane_id();
  if (kmin == kmax) return kmin;
  int64_t ncand = n;
  uint64_t lo = kmin, span = kmax - kmin;
  while (ncand > kWave) {
    if (span == 0) return lo;   // every candidate left is lo
    // buckets of 2^shift keys: span >> shift < 256
    const int bits = 64 - __builtin_clzll(span);
    const int shift = bits > 8 ? bits - 8 : 0;
    for (int bn = tid; bn < 4 * 256; bn += blockDim.x) hist4[bn] = 0;
    __syncthreads();
    unsigned *myh = hist4 + 256 * ((tid >> 6) & 3);
    for (int64_t e = tid; e < ncand; e += blockDim.x)
      atomicAdd(&myh[(src[e] - lo) >> shift], 1u);
    __syncthreads();
    // bucket holding the element of rank `rank` (first 256 threads, 4 waves)
    const unsigned h =
        tid < 256 ? hist4[tid] + hist4[256 + tid] + hist4[512 + tid] + hist4[768 + tid] : 0u;
    const int64_t inc = wave_inclusive_scan<int64_t>((int64_t)h);
    if (tid < 256 && lane == kWave - 1) s_wtot[tid >> 6] = inc;
    __syncthreads();
    if (tid < 256) {
      int64_t base = 0;
      for (int w = 0; w < (tid >> 6); ++w) base += s_wtot[w];
      const int64_t ex = base + inc - (int64_t)h;
      if (ex <= rank && rank < ex + (int64_t)h) {
        s_chosen = tid;
        s_below = ex;
      }
    }
    __syncthreads();
    const uint64_t chosen = (uint64_t)s_chosen;
    rank -= s_below;
    const uint64_t blo = chosen << shift;
    if (shift == 0) return lo + blo;
    if (tid == 0) s_ncand = 0;
    __syncthreads();
    for (int64_t e0 = 0; e0 < ncand; e0 += blockDim.x) {
      const int64_t e = e0 + tid;
      const bool keep = e < ncand && ((src[e] - lo) >> shift) == chosen;
      const uint64_t bk = ballot(keep);
      unsigned base = 0;
      if (lane == 0 && bk) base = atomicAdd(&s_ncand, (unsigned)popc(bk));
      base = lane_value(base, 0);
      if (keep) dst[base + rank_below(bk, lane)] = src[e];
    }
    __syncthreads();
    ncand = s_ncand;
    const uint64_t rest = span - blo;
    lo += blo;
    span = rest < (1ull << shift) - 1ull ? rest : (1ull << shift) - 1ull;
    uint64_t *tmp = src;
    src = dst;
    dst = tmp;
    __syncthreads();
  }
  // at most 64 left: lane l holds candidate l and counts the smaller ones
  if (tid < kWave) {
    const uint64_t k = lane < ncand ? src[lane] : ~0ull;
    int less = 0, leq = 0;
    for (int j = 0; j < (int)ncand; ++j) {
      const uint64_t kj = lane_value(k, j);
      less += kj < k ? 1 : 0;
      leq += kj <= k ? 1 : 0;
    }
    if (lane < ncand && less <= rank && rank < leq) s_key = k;
  }
  __syncthreads();
  return s_key;
}

__device__ __forceinline__ double key_value(uint64_t k) {
  return __longlong_as_double((long long)k);
}

// What one block brings to the allocation: floor, cap, weights and its eligible
// prices.  di: depth, best: distance to the nearest active leaf, on: Path*
// (not pinned); flags a bad score in err (2: NaN, 4: outside [0, 1]).
struct NodeTerms {
  int F, cap, cnt;
  double W, w;
  uint64_t lo, hi;   // keys of its first and last eligible price (cnt > 0)
};
__device__ __forceinline__ NodeTerms node_terms(const AllocParams &p, const double *dexp,
                                                const double *texp, bool on, int n, int c,
                                                float sf, int di, int best, int &err) {
  NodeTerms r;
  r.cap = on && p.rehydrate ? n : c;
  // s_i = clip(sigmoid(.), 0, 1) lies in [0, 1]
  if (!(sf == sf)) err |= 2;
  else if (!(sf >= 0.f && sf <= 1.f)) err |= 4;
  const double s = (double)sf;
  // Eq. 3 at the ratio floor r_min, capped; a Path* block under floor
  // protection keeps at least k_protect
  int f = max(p.k_min, min(p.l_tail, n));
  f = max(f, (int)floor(p.r_min * (double)n));
  f = min(r.cap, min(n, f));
  if (on) f = max(f, min(r.cap, p.k_protect));
  r.F = f;
  // the Eq. 2 weight without alpha, in the same operation order as
  // ((eta^[off path] * s^gamma) * e^{-lambda_d d}) * e^{-lambda_Delta Delta}
  double w = (on ? 1.0 : p.eta) * pow_gamma(s, p.gamma);
  w = w * (di < kDecay ? dexp[di] : exp(-p.lambda_d * (double)di));
  w = w * (best < kDecay ? texp[best] : exp(-p.lambda_delta * (double)best));
  // -0 (s = -0 with an odd gamma) as +0: the Pressure order compares bit
  // patterns, in which -0 would rank above every positive weight
  r.w = w == 0.0 ? 0.0 : w;
  r.W = r.w * (double)n;
  r.cnt = eligible(f, r.cap, r.W, p.alpha_max);
  r.lo = r.hi = 0;
  if (r.cnt > 0) {
    r.lo = (uint64_t)__double_as_longlong(price(f + 1, r.W));
    r.hi = (uint64_t)__double_as_longlong(price(f + r.cnt, r.W));
  }
  return r;
}

// Pressure (Alg. 2): the floors exceed the budget by `excess`; the blocks of
// lowest priority are drained to min(K_min, c).  Called by the whole workgroup.
template <class Floor>
__device__ void pressure_drain(const AllocParams &p, int V, const uint8_t *path, Floor &&F,
                               const double *w, const int32_t *n_kept, int64_t sum_red,
                               int64_t excess, int32_t *__restrict__ k_out, int32_t *status,
                               int64_t *sm) {
  __shared__ unsigned long long hist64[256];
  const int tid = threadIdx.x;
  if (sum_red < excess) {
    for (int i = tid; i < V; i += (int)blockDim.x) {
      if (!path[i]) k_out[i] = min(p.k_min, n_kept[i]);
      else if (p.k_protect > 0) k_out[i] = F(i);   // Path* keeps its floor
    }
    if (tid == 0) status_warn(status, ARBOR_OVER_BUDGET);
    return;
  }
  // smallest priority value W* whose cumulative reducible count reaches excess
  uint64_t prefix = 0, pmask = 0;
  int64_t need = excess;
  for (int shift = 56; shift >= 0; shift -= 8) {
    for (int b = tid; b < 256; b += (int)blockDim.x) hist64[b] = 0;
    __syncthreads();
    for (int i = tid; i < V; i += (int)blockDim.x) {
      if (path[i]) continue;
      const uint64_t key = (uint64_t)__double_as_longlong(w[i]);
      if ((key & pmask) != prefix) continue;
      const int red = F(i) - min(p.k_min, n_kept[i]);
      if (red > 0) atomicAdd(&hist64[(key >> shift) & 255ull], (unsigned long long)red);
    }
    __syncthreads();
    int chosen = 255;
    int64_t acc = 0;
    for (int b = 0; b < 256; ++b) {
      const int64_t h = (int64_t)hist64[b];
      if (acc + h >= need) {
        chosen = b;
        break;
      }
      acc += h;
    }
    need -= acc;
    prefix |= (uint64_t)chosen << shift;
    pmask |= 255ull << shift;
    __syncthreads();
  }
  // nodes below W* drain fully; nodes at W* drain in id order until `need`
  int64_t run = 0;
  for (int base = 0; base < V; base += (int)blockDim.x) {
    const int i = base + tid;
    int64_t red = 0;
    uint64_t key = 0;
    const bool off = i < V && !path[i];
    if (off) {
      red = F(i) - min(p.k_min, n_kept[i]);
      key = (uint64_t)__double_as_longlong(w[i]);
    }
    const bool tie = off && key == prefix;
    int64_t tot;
    const int64_t ex = block_exclusive_scan<int64_t>(tie ? red : 0, sm, &tot);
    if (off) {
      int kk = F(i);
      if (key < prefix) {
        kk -= (int)red;
      } else if (tie) {
        const int64_t before = run + ex;
        if (before < need) kk -= (int)min<int64_t>(red, need - before);
      }
      k_out[i] = kk;
    } else if (i < V && p.k_protect > 0) {
      k_out[i] = F(i);                                // Path* keeps its floor
    }
    run += tot;
  }
}

// Larger trees, first launch for trees beyond kGeoNodes blocks: the distance of
// each Path* block down to its nearest active leaf, in the workspace (one
// workgroup; alloc_nodes forms it in LDS for smaller ones).
__global__ __launch_bounds__(AT) void alloc_path(Tree t, const int32_t *__restrict__ active,
                                                 int n_active, int32_t *status, AllocWs ws) {
  if (status_failed(status)) return;
  for (int i = threadIdx.x; i < t.V; i += AT) ws.down[i] = INT32_MAX;
  __syncthreads();
  for (int j = threadIdx.x; j < n_active; j += AT) {
    const int l = active[j];
    if (l < 0 || l >= t.V) continue;
    int k = 0;
    for (int a = l;; ++k) {
      atomicMin(&ws.down[a], k);
      const int pa = a > 0 ? t.parent[a] : -1;
      if (pa < 0 || pa >= a) break;
      a = pa;
    }
  }
}

// Larger trees: geometry, floors, weights and eligible prices, one thread per
// block.  Every workgroup copies the parent links to LDS and marks the active
// chains itself (a chain is short, and a copy of the links costs less than
// the launch that would share the marks), so nothing waits on another
// workgroup.  One workgroup for all blocks took 35 us of its 41 here on the
// 9,841-block tree; this kernel takes 8.5 us.
template <bool IN_LDS>
__global__ __launch_bounds__(kNodeThreads) void alloc_nodes(
    Tree t, const int32_t *__restrict__ active, int n_active, int64_t budget,
    const float *__restrict__ s_in, AllocParams p, int32_t *__restrict__ k_out,
    int32_t *__restrict__ delta_out, uint8_t *__restrict__ on_path, int32_t *status, AllocWs ws,
    int gate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ int64_t sm[6 * 16];
  __shared__ double s_dexp[kDecay], s_texp[kDecay];
  __shared__ int s_err;
  constexpr int NT = kNodeThreads;
  const int tid = threadIdx.x, V = t.V;
  const int i = blockIdx.x * NT + tid;
  const bool live = i < V;
  // the thread's block, its score and the decay tables: loads issued
  // together, ahead of the status check, so they cost one round trip
  int par0 = 0, n = 0, c = 0;
  float s0 = 0.f;
  if (live) {
    par0 = t.parent[i];
    n = t.n_full[i];
    c = t.n_kept[i];
    s0 = s_in[i];
  }
  const int leaf0 = tid < n_active ? active[tid] : 0;
  static_assert(kNodeThreads >= kDecay, "one table entry per thread");
  double dx = 0.0, tx = 0.0;
  if (tid < kDecay) {
    dx = p.dexp[tid];
    tx = p.texp[tid];
  }
  if (status_failed(status)) return;
  if (tid < kDecay) {
    s_dexp[tid] = dx;
    s_texp[tid] = tx;
  }
  if (tid == 0) s_err = 0;
  if (gate) {
    // a Pressure event (Alg. 2): it fires only when the resident tokens
    // reach the budget it is given; otherwise every count stays as it is
    int64_t m = 0;
#pragma unroll 8
    for (int x = tid; x < V; x += NT) m += t.n_kept[x];
    m = block_sum<int64_t>(m, sm);
    if (blockIdx.x == 0 && tid == 0) *ws.gated = m < budget;
    if (m < budget) {
      if (live) k_out[i] = c;
      return;
    }
  } else if (blockIdx.x == 0 && tid == 0) {
    *ws.gated = 0;
  }
  int32_t *const s_par = reinterpret_cast<int32_t *>(dyn);
  int32_t *const s_down = s_par + V;
  const int32_t *par = IN_LDS ? s_par : t.parent;
  const int32_t *down = IN_LDS ? s_down : ws.down;
  if constexpr (IN_LDS) {
#pragma unroll 8
    for (int x = tid; x < V; x += NT) {
      s_par[x] = t.parent[x];
      s_down[x] = INT32_MAX;
    }
  }
  __syncthreads();
  int err = 0;
  for (int j = tid; j < n_active; j += NT) {
    const int l = j == tid ? leaf0 : active[j];
    if (l < 0 || l >= V) {
      err |= 1;
      continue;
    }
    if constexpr (IN_LDS) {
      int k = 0;
      for (int a = l;; ++k) {
        atomicMin(&s_down[a], k);
        const int pa = a > 0 ? s_par[a] : -1;
        if (pa < 0 || pa >= a) break;       // (the block's own thread reports it)
        a = pa;
      }
    }
  }
  __syncthreads();
  // depth d_i and Delta_i = min over ancestors a (incl. i) of the steps up to a
  // plus the distance from a down to its nearest active leaf
  int64_t v[6] = {0, 0, 0, 0, INT64_MAX, INT64_MAX};
  if (live) {
    if (!((i == 0 ? par0 == -1 : (par0 >= 0 && par0 < i)) && n >= 0 && c >= 0 && c <= n)) err |= 1;
    int d = 0, best = INT32_MAX;
    for (int a = i;; ++d) {
      const int dn = down[a];
      if (dn != INT32_MAX) best = min(best, d + dn);
      if (a == 0) break;
      const int pa = par[a];
      if (pa < 0 || pa >= a) {
        err |= 1;
        break;
      }
      a = pa;
    }
    const bool on = down[i] != INT32_MAX;
    delta_out[i] = best;
    on_path[i] = on ? 1 : 0;
    if (on && p.k_protect == 0) {
      // pinned (invariant (i), full protection): restored by rehydration to
      // n_i, or c_i when evicted tokens stay lost
      const int keep = p.rehydrate ? n : c;
      k_out[i] = keep;
      v[0] = keep;
      ws.rec[i] = NodeRec{-1, 0, 1.0};
    } else if (!err) {
      const NodeTerms r = node_terms(p, s_dexp, s_texp, on, n, c, s0, d, best, err);
      ws.rec[i] = NodeRec{r.F, r.cnt, r.cnt > 0 ? r.W : 1.0};
      ws.w[i] = r.w;
      v[1] = r.F;
      // Pressure lowers only off-path blocks
      if (!on) v[2] = r.F - min(p.k_min, c);
      v[3] = r.cnt;
      if (r.cnt > 0) {
        v[4] = (int64_t)r.lo;
        v[5] = INT64_MAX - (int64_t)r.hi;
      }
    }
  }
  if (err) atomicOr(&s_err, err);
  block_reduce_n<4>(v, sm, NT);            // (its barriers also settle s_err)
  if (tid == 0) {
    const int64_t e = s_err;
    ws.sums[blockIdx.x] = NodeSums{v[0], v[1], v[2], v[3], v[4], INT64_MAX - v[5],
                                   (e & 1) | ((e >> 1) & 1) << 21 | ((e >> 2) & 1) << 42};
  }
}

// block-wide sums of three counts kept as doubles (exact: below 2^53); sm holds
// 48 values
__device__ void block_sum3_f64(double (&v)[3], double *sm) {
  const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = wave_sum(v[q]);
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) sm[16 * q + w] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = wave_sum(lane < nw ? sm[16 * q + lane] : 0.0);
}

// Larger trees, last launch (one workgroup): the totals, then alpha from the
// price order statistic, or Pressure.  A search round counts the prices up to
// kCutPts keys over every block; up to kCutThreads * kRegNodes blocks sit in registers
// (REG), so a round costs its fp64 work, five operations per block and key,
// and few keys a round, placed by interpolation, cost least.  The counts are
// floor(x W), which may be off by one where x W lies within a rounding of an
// integer: the bracket that they leave is counted exactly before it is used,
// and a search that it does not confirm is done again on exact counts.
// 9,841 blocks with scores drawn from [0, 1] take 42 us in all (both
// launches), against 320 for rounds of 64 keys that every wave read from L2
// and a listing of all prices within rounding of the cut; 1,024 threads of ten
// blocks (whose reductions cost twice as much) take 55, 256 threads 52.  More
// blocks stream from the workspace each round.
template <bool REG>
__global__ __launch_bounds__(kCutThreads) void alloc_cut(Tree t, int64_t budget, AllocParams p,
                                                int32_t *__restrict__ k_out,
                                                const uint8_t *__restrict__ on_path,
                                                int32_t *status, AllocWs ws, int n_sums) {
  __shared__ int64_t sm[7 * 16];
  __shared__ double sc[2][48];
  __shared__ uint64_t s_cand[2 * kCandLds];
  const int tid = threadIdx.x, V = t.V;
  constexpr int NR = REG ? kRegNodes : 1;
  // a block's floor and floor + count as doubles, as the search reads them
  struct Blk {
    double lo, hi, W;
    __device__ __forceinline__ int F() const { return (int)lo; }
    __device__ __forceinline__ int cnt() const { return (int)hi - (int)lo; }
  };
  auto blk = [](const NodeRec &n) __attribute__((always_inline)) {
    return Blk{(double)n.F, (double)(n.F + n.cnt), n.W};
  };
  Blk rec[NR];
  if constexpr (REG) {
    // (issued together with the status word)
    NodeRec raw[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) raw[r] = ws.rec[min(tid + r * kCutThreads, V - 1)];
#pragma unroll
    for (int r = 0; r < NR; ++r)
      rec[r] = tid + r * kCutThreads < V ? blk(raw[r]) : Blk{-1.0, -1.0, 1.0};
  }
  if (status_failed(status)) return;
  if (*ws.gated) return;
  // f(i, block) for each of the thread's blocks: from the registers (the search
  // only: a pass of this kind is unrolled), or as a loop over the workspace
  // (which the L2 holds)
  auto each_reg = [&](auto &&f) __attribute__((always_inline)) {
    if constexpr (REG) {
#pragma unroll
      for (int r = 0; r < NR; ++r) f(tid + r * kCutThreads, rec[r]);
    } else {
#pragma unroll 4
      for (int i = tid; i < V; i += kCutThreads) f(i, blk(ws.rec[i]));
    }
  };
  auto each = [&](auto &&f) __attribute__((always_inline)) {
    NodeRec next = ws.rec[min(tid, V - 1)];
#pragma unroll 1
    for (int i = tid; i < V; i += kCutThreads) {
      const Blk cur = blk(next);
      next = ws.rec[min(i + kCutThreads, V - 1)];
      f(i, cur);
    }
  };
  int64_t v[7] = {0, 0, 0, 0, 0, INT64_MAX, INT64_MAX};
  for (int e = tid; e < n_sums; e += kCutThreads) {
    const NodeSums s = ws.sums[e];
    v[0] += s.path_tok;
    v[1] += s.sum_F;
    v[2] += s.sum_red;
    v[3] += s.total;
    v[4] += s.flags;
    v[5] = min(v[5], s.kmin);
    v[6] = min(v[6], INT64_MAX - s.kmax);
  }
  block_reduce_n<5>(v, sm, min(n_sums, kCutThreads));
#pragma unroll
  for (int q = 0; q < 7; ++q) v[q] = lane_value(v[q], 0);
  const int64_t path_tok = v[0], sum_F = v[1], sum_red = v[2], total = v[3];
  if (v[4]) {
    constexpr int64_t k21 = (1 << 21) - 1;
    if (tid == 0)
      status_error(status, !(v[4] & k21) && ((v[4] >> 21) & k21) ? ARBOR_ENONFINITE : ARBOR_EINVAL);
    return;
  }
  const int64_t b_off = budget - path_tok;
  if (sum_F > b_off) {
    pressure_drain(p, V, on_path, [&](int i) { return ws.rec[i].F; }, ws.w, t.n_kept, sum_red,
                   sum_F - b_off, k_out, status, sm);
    return;
  }
  const int64_t E = b_off - sum_F;
  if (total <= E) {
    each([&](int i, const Blk &n) __attribute__((always_inline)) {
      if (n.lo >= 0.0) k_out[i] = (int)n.hi;
    });
    return;
  }
  // the floors of the thread's register slots, padding included (a slot's count
  // is floor(x W), clamped, less its floor)
  double F0 = 0.0;
  each_reg([&](int, const Blk &n) __attribute__((always_inline)) { F0 += n.lo; });
  uint64_t answer = 0;
  for (bool exact = false;; exact = true) {
    // count(<= ka) = cA <= E < cB = count(<= kb), from below every price to the
    // largest one (keys of finite positive doubles; -1: below a zero price)
    int64_t ka = v[5] - 1, kb = INT64_MAX - v[6];
    double cA = 0.0, cB = (double)total;
    const double Ed = (double)E;
    bool even = true;                    // place the keys evenly, not by interpolation
    for (int round = 0; kb - ka > 1 && cB - cA > (double)kCandLds; ++round) {
      if (round >= kSnapFrom && (round - kSnapFrom) % kSnapEvery == 0) {
        // the bracket's ends onto prices: many equal prices (blocks of one size
        // and weight) would hold up the search to the last bit
        int64_t w[3] = {0, INT64_MAX, INT64_MAX};
        const double xa = ka >= 0 ? key_value((uint64_t)ka) : 0.0, xb = key_value((uint64_t)kb);
        each([&](int, const Blk &n) __attribute__((always_inline)) {
          const int m_lo = ka >= 0 ? last_le(xa, n.F(), n.cnt(), n.W) : n.F();
          const int m_hi = last_le(xb, n.F(), n.cnt(), n.W);
          if (m_hi > m_lo) {
            w[1] = min(w[1], (int64_t)__double_as_longlong(price(m_lo + 1, n.W)));
            w[2] = min(w[2], INT64_MAX - (int64_t)__double_as_longlong(price(m_hi, n.W)));
          }
        });
        block_min_sum3(w, sm);
        if (w[1] == INT64_MAX) break;    // (rounded counts, and no price at all)
        ka = lane_value(w[1], 0) - 1;
        kb = INT64_MAX - lane_value(w[2], 0);
        if (kb - ka <= 1) break;
      }
      const int64_t span = kb - ka;
      int64_t x[kCutPts];
      if (even) {
#pragma unroll
        for (int q = 0; q < kCutPts; ++q) x[q] = ka + span / (kCutPts + 1) * (q + 1);
      } else {
        const double f = (Ed - cA + 0.5) / (cB - cA);
        const int64_t xi = ka + lane_value((int64_t)(f * (double)span), 0), dx = span / 8;
#pragma unroll
        for (int q = 0; q < kCutPts; ++q) {
          const int64_t o = (q - kCutPts / 2) * dx;
          x[q] = o < kb - xi ? xi + o : kb - 1;
        }
      }
      double c[kCutPts], xv[kCutPts];
#pragma unroll
      for (int q = 0; q < kCutPts; ++q) {
        x[q] = min(max(x[q], ka + 1), kb - 1);
        xv[q] = key_value((uint64_t)x[q]);
        c[q] = exact ? 0.0 : -F0;
      }
      if (!exact) {
        each_reg([&](int, const Blk &n) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < kCutPts; ++q)
            c[q] += __builtin_fmin(__builtin_fmax(__builtin_floor(xv[q] * n.W), n.lo), n.hi);
        });
      } else {
        // (over the blocks alone, without the slots' padding: each brings its floor)
        each([&](int, const Blk &n) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < kCutPts; ++q)
            c[q] += (double)(last_le(xv[q], n.F(), n.cnt(), n.W) - n.F());
        });
      }
      static_assert(kCutPts == 3, "one block_sum3_f64 per round");
      block_sum3_f64(c, sc[round & 1]);
      // (wave-uniform: kept in scalar registers, beside the blocks)
#pragma unroll
      for (int q = 0; q < kCutPts; ++q) c[q] = lane_value(c[q], 0);
      // the keys ascend and their counts with them
#pragma unroll
      for (int q = 0; q < kCutPts; ++q)
        if (c[q] <= Ed) {
          ka = x[q];
          cA = c[q];
        }
#pragma unroll
      for (int q = kCutPts - 1; q >= 0; --q)
        if (c[q] > Ed) {
          kb = x[q];
          cB = c[q];
        }
      // interpolation that shrinks the bracket less than even keys would gives
      // way to them for a round
      even = !even && kb - ka > span / (kCutPts + 1);
    }
    // the bracket's exact counts: the prices up to ka, and the thread's prices
    // in (ka, kb] with their places in the list
    const double xa = ka >= 0 ? key_value((uint64_t)ka) : 0.0, xb = key_value((uint64_t)kb);
    int64_t below = 0, mine = 0;
    auto range = [&](const Blk &n, int &m_lo, int &m_hi) __attribute__((always_inline)) {
      bool near = ka < 0;
      m_lo = last_fast(xa, n.lo, n.hi, n.W, near);
      m_hi = last_fast(xb, n.lo, n.hi, n.W, near);
      if (near) {
        m_lo = ka >= 0 ? last_le(xa, n.F(), n.cnt(), n.W) : n.F();
        m_hi = last_le(xb, n.F(), n.cnt(), n.W);
      }
    };
    each([&](int, const Blk &n) __attribute__((always_inline)) {
      int m_lo, m_hi;
      range(n, m_lo, m_hi);
      below += m_lo - n.F();
      mine += m_hi - m_lo;
    });
    const int64_t v2[2] = {below, mine};
    int64_t ex[2], tot[2];
    __syncthreads();                       // (the search's last reads of its exchange)
    block_exclusive_scan_n<2>(v2, ex, tot, sm);
    const bool held = tot[0] <= E && tot[0] + tot[1] > E;
    if (held && kb - ka <= 1) {
      answer = (uint64_t)kb;
      break;
    }
    if (!held || tot[1] > kCandLds) {
      if (!exact) continue;
      // exact counts that do not agree with themselves: the blocks changed
      // under the search.  No count was written, so no later launch may run.
      if (tid == 0) status_error(status, ARBOR_ECORRUPT);
      return;
    }
    // the listed prices and their order statistic
    if (mine > 0) {
      int64_t off = ex[1];
      each([&](int, const Blk &n) __attribute__((always_inline)) {
        int m_lo, m_hi;
        range(n, m_lo, m_hi);
#pragma unroll 1
        for (int j = m_lo; j < m_hi; ++j)
          s_cand[off++] = (uint64_t)__double_as_longlong(price(j + 1, n.W));
      });
    }
    __syncthreads();
    answer = select_rank(s_cand, s_cand + kCandLds, tot[1], E - tot[0], (uint64_t)(ka + 1),
                         (uint64_t)kb);
    break;
  }
  // the prices below the cut, all of them eligible ones (the cut is)
  const double cut = key_value(answer);
  each([&](int i, const Blk &n) __attribute__((always_inline)) {
    bool near = false;
    int m = last_fast(cut, n.lo, n.hi, n.W, near);
    if (near) m = last_lt(cut, n.F(), n.cnt(), n.W);
    if (n.lo >= 0.0) k_out[i] = m;
  });
}

// Small trees: one workgroup, all per-node state in LDS.
__global__ __launch_bounds__(AT) void allocate_kernel(Tree t, const int32_t *__restrict__ active,
                                                      int n_active, int64_t budget,
                                                      const float *__restrict__ s_in, AllocParams p,
                                                      int32_t *__restrict__ k_out,
                                                      int32_t *__restrict__ delta_out,
                                                      uint8_t *__restrict__ on_path,
                                                      int32_t *status, int gate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ int64_t sm[7 * 16];
  __shared__ int s_err;
  __shared__ double s_cnt[2][kWave];
  __shared__ uint64_t s_x[2][kWave];
  __shared__ double s_dexp[kDecay], s_texp[kDecay];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = lane_id();
  const int V = t.V;
  // each thread's first node, its score and the decay tables: loads issued
  // together, ahead of the status check, so they cost one round trip
  int par0 = 0, nf0 = 0, nk0 = 0;
  float s0 = 0.f;
  if (tid < V) {
    par0 = t.parent[tid];
    nf0 = t.n_full[tid];
    nk0 = t.n_kept[tid];
    s0 = s_in[tid];
  }
  double dx = 0.0, tx = 0.0;
  if (tid < kDecay) {
    dx = p.dexp[tid];
    tx = p.texp[tid];
  }
  if (status_failed(status)) return;
  if (tid < kDecay) {
    s_dexp[tid] = dx;
    s_texp[tid] = tx;
  }
  if (tid == 0) s_err = 0;
  if (gate) {
    // a Pressure event (Alg. 2): it fires only when the resident tokens
    // reach the budget it is given; otherwise every count stays as it is
    int64_t m = 0;
    for (int i = tid; i < V; i += AT) m += i == tid ? nk0 : t.n_kept[i];
    m = block_sum<int64_t>(m, sm);
    if (m < budget) {
      for (int i = tid; i < V; i += AT) k_out[i] = i == tid ? nk0 : t.n_kept[i];
      return;
    }
  }

  // listed prices and the per-wave counts of the search after the node state
  const size_t node_lds = ((size_t)V * kNodeBytes + 15) / 16 * 16;
  uint64_t *const cand_lds = reinterpret_cast<uint64_t *>(dyn + node_lds);
  double *const s_part = reinterpret_cast<double *>(cand_lds + kWave);
  Nodes nd;
  {
    double *dp = reinterpret_cast<double *>(dyn);
    nd.W = dp;
    nd.w = dp + V;
    int32_t *ip = reinterpret_cast<int32_t *>(dp + 2 * V);
    nd.parent = ip;
    nd.n_full = ip + V;
    nd.n_kept = ip + 2 * V;
    nd.depth = ip + 3 * V;
    nd.down = ip + 4 * V;
    nd.F = ip + 5 * V;
    nd.cnt = ip + 6 * V;
    nd.cap = ip + 7 * V;
    nd.path = reinterpret_cast<uint8_t *>(ip + 8 * V);
    if (tid < V) {
      nd.parent[tid] = par0;
      nd.n_full[tid] = nf0;
      nd.n_kept[tid] = nk0;
    }
  }
  __syncthreads();

  // ---- geometry: validation, depth d_i, Path*, Delta_i (Sec. 3) ----------
  for (int i = tid; i < V; i += AT) {
    const int par = i == tid ? par0 : nd.parent[i];
    const int n = i == tid ? nf0 : nd.n_full[i];
    const int c = i == tid ? nk0 : nd.n_kept[i];
    bool ok = (i == 0) ? (par == -1) : (par >= 0 && par < i);
    ok = ok && n >= 0 && c >= 0 && c <= n;
    int d = 0;
    for (int a = i; ok && a > 0;) {
      const int pa = nd.parent[a];
      if (pa < 0 || pa >= a) {
        ok = false;
        break;
      }
      a = pa;
      ++d;
    }
    if (!ok) atomicOr(&s_err, 1);
    nd.depth[i] = d;
    nd.down[i] = 0x7fffffff;
    nd.path[i] = 0;
  }
  __syncthreads();
  if (n_active < 1) s_err = 1;
  __syncthreads();
  for (int j = tid; j < n_active && !s_err; j += AT) {
    const int l = active[j];
    if (l < 0 || l >= V) {
      atomicOr(&s_err, 1);
      continue;
    }
    const int dl = nd.depth[l];
    for (int a = l; a >= 0; a = nd.parent[a]) {
      nd.path[a] = 1;
      atomicMin(&nd.down[a], dl - nd.depth[a]);
    }
  }
  __syncthreads();
  if (s_err) {
    if (tid == 0) status_error(status, ARBOR_EINVAL);
    return;
  }
  // Delta_i = min over ancestors a (incl. i) of (d_i - d_a) + (distance from a
  // down to its nearest active leaf)
  // The eligible prices of each block (finite, at most alpha_max) and their
  // key range are counted here too, so one exchange gives every total.
  int64_t path_tok = 0, sum_F = 0, sum_red = 0, total = 0;
  uint64_t kmin = ~0ull, kmax = 0ull;
  for (int i = tid; i < V; i += AT) {
    int best = 0x7fffffff;
    const int di = nd.depth[i];
    for (int a = i; a >= 0; a = nd.parent[a]) {
      const int dn = nd.down[a];
      if (dn != 0x7fffffff) best = min(best, di - nd.depth[a] + dn);
    }
    delta_out[i] = best;
    const int n = i == tid ? nf0 : nd.n_full[i];
    const int c = i == tid ? nk0 : nd.n_kept[i];
    const bool on = nd.path[i] != 0;
    on_path[i] = nd.path[i];
    if (on && p.k_protect == 0) {
      // pinned (invariant (i), full protection): restored by rehydration to
      // n_i, or c_i when evicted tokens stay lost
      const int keep = p.rehydrate ? n : c;
      k_out[i] = keep;
      path_tok += keep;
      nd.cap[i] = keep;
      nd.F[i] = 0;
      nd.W[i] = 0.0;
      nd.w[i] = 0.0;
      nd.cnt[i] = 0;
      continue;
    }
    int err = 0;
    const NodeTerms r = node_terms(p, s_dexp, s_texp, on, n, c, s0, di, best, err);
    if (err) atomicOr(&s_err, err);
    nd.cap[i] = r.cap;
    nd.F[i] = r.F;
    nd.W[i] = r.W;
    nd.w[i] = r.w;
    nd.cnt[i] = r.cnt;
    sum_F += r.F;
    // Pressure lowers only off-path blocks
    if (!on) sum_red += r.F - min(p.k_min, c);
    total += r.cnt;
    if (r.cnt > 0) {
      kmin = r.lo < kmin ? r.lo : kmin;
      kmax = r.hi > kmax ? r.hi : kmax;
    }
  }
  {
    // four sums and two minima in one exchange (finite positive keys are
    // below 2^63: the maximum is taken as the minimum of INT64_MAX - key)
    int64_t v[6] = {path_tok, sum_F, sum_red, total,
                    kmin == ~0ull ? INT64_MAX : (int64_t)kmin, INT64_MAX - (int64_t)kmax};
    block_reduce_n<4>(v, sm, V);
    path_tok = v[0];
    sum_F = v[1];
    sum_red = v[2];
    total = v[3];
    kmin = (uint64_t)v[4];
    kmax = (uint64_t)(INT64_MAX - v[5]);
  }
  if (s_err) {
    if (tid == 0) status_error(status, (s_err & 2) ? ARBOR_ENONFINITE : ARBOR_EINVAL);
    return;
  }
  const int64_t b_off = budget - path_tok;

  if (sum_F <= b_off) {
    // ---- budget mode: alpha from the price order statistic ---------------
    const int64_t E = b_off - sum_F;
    if (total <= E) {
      for (int i = tid; i < V; i += AT)
        if (!(nd.path[i] && p.k_protect == 0)) k_out[i] = nd.F[i] + nd.cnt[i];
      return;
    }

    // -- few nodes: narrow on exact counts --------------------------------
    // Keys ka < kb with count(<= ka) <= E < count(<= kb), from ka = the
    // smallest price's key - 1 (-1 when that price is 0: below every
    // price) and kb = the largest one's.  Each round tests ka, kb and 62
    // keys between them, one key per lane; the waves split the blocks,
    // whose exact counts (last_le) are added in wave order.  It stops when
    // kb - ka = 1 (the answer is kb) or when at most 64 prices lie in
    // (ka, kb], which are then listed and ranked by one wave.
    int64_t ka = (int64_t)kmin - 1, kb = (int64_t)kmax;
    int64_t cA = 0, cB = 0;
    bool counted = false;
    uint64_t answer = 0;
    bool found = false;
    for (int round = 0;; ++round) {
      if (kb - ka <= 1) {
        answer = (uint64_t)kb;
        found = true;
        break;
      }
      if (counted && cB - cA <= kWave) break;
      const uint64_t span = (uint64_t)(kb - ka);
      const uint64_t m = (uint64_t)lane;
      const int64_t x = lane == kWave - 1
                            ? kb
                            : ka + (int64_t)((span / (kWave - 1)) * m +
                                             ((span % (kWave - 1)) * m) / (kWave - 1));
      double c = 0.0;
      if (x >= 0) {
        const double xv = key_value((uint64_t)x);
#pragma unroll 4
        for (int i = wave; i < V; i += AT / kWave) {
          const int cnt = nd.cnt[i];
          const int F = nd.F[i];
          const int mm = cnt > 0 ? last_le(xv, F, cnt, nd.W[i]) : F;
          c += (double)(mm - F);
        }
      }
      s_part[tid] = c;
      __syncthreads();
      if (tid < kWave) {
        double sum = 0.0;
        for (int w = 0; w < AT / kWave; ++w) sum += s_part[w * kWave + tid];
        s_cnt[round & 1][tid] = sum;
        s_x[round & 1][tid] = (uint64_t)x;
      }
      __syncthreads();
      // the keys ascend and their counts with them: the last one with
      // count <= E is the new ka (lane 0 at least), the first one above E
      // the new kb (lane 63 at least)
      const double cq = s_cnt[round & 1][lane];
      const int64_t xq = (int64_t)s_x[round & 1][lane];
      const uint64_t le = ballot(cq <= (double)E);
      const int qa = 63 - __builtin_clzll(le);
      const int qb = __builtin_ctzll(~le);
      ka = lane_value(xq, qa);
      kb = lane_value(xq, qb);
      cA = (int64_t)lane_value(cq, qa);
      cB = (int64_t)lane_value(cq, qb);
      counted = true;
    }
    if (!found) {
      // the cB - cA <= 64 prices in (ka, kb], placed by a block scan and
      // ranked by one wave
      uint64_t *const lst = cand_lds;
      const double av1 = ka >= 0 ? key_value((uint64_t)ka) : 0.0, bv1 = key_value((uint64_t)kb);
      int m_lo = 0, m_hi = 0;
      double Wt = 0.0;
      if (tid < V && nd.cnt[tid] > 0) {
        const int F = nd.F[tid], cnt = nd.cnt[tid];
        Wt = nd.W[tid];
        m_lo = ka >= 0 ? last_le(av1, F, cnt, Wt) : F;
        m_hi = last_le(bv1, F, cnt, Wt);
      }
      int64_t tot;
      const int64_t off = block_exclusive_scan<int64_t>((int64_t)(m_hi - m_lo), sm, &tot);
      for (int j = m_lo; j < m_hi; ++j)
        lst[off + (j - m_lo)] = (uint64_t)__double_as_longlong(price(j + 1, Wt));
      __syncthreads();
      if (wave == 0) {
        const int n = (int)tot;
        const int64_t r = E - cA;
        const uint64_t key = lane < n ? lst[lane] : ~0ull;
        int less = 0, leq = 0;
        for (int q = 0; q < n; ++q) {
          const uint64_t kq = lane_value(key, q);
          less += kq < key ? 1 : 0;
          leq += kq <= key ? 1 : 0;
        }
        if (lane < n && less <= r && r < leq) s_x[0][0] = key;
      }
      __syncthreads();
      answer = s_x[0][0];
    }
    const double cut = key_value(answer);
    for (int i = tid; i < V; i += AT) {
      if (nd.path[i] && p.k_protect == 0) continue;
      const int F = nd.F[i];
      const double W = nd.W[i];
      k_out[i] = W > 0.0 ? last_lt(cut, F, nd.cap[i] - F, W) : F;
    }
    return;
  }

  pressure_drain(p, V, nd.path, [&](int i) { return nd.F[i]; }, nd.w, nd.n_kept, sum_red,
                 sum_F - b_off, k_out, status, sm);
}

}  // namespace

size_t allocate_workspace(const arbor_sizes_t *sz) {
  const size_t V = (size_t)sz->num_nodes;
  return V * (4 + sizeof(NodeRec) + 8) + (V / kNodeThreads + 1) * sizeof(NodeSums) + 8192;
}

__global__ __launch_bounds__(AT) void walk_stats(Tree t, const int32_t *__restrict__ k,
                                                 const uint8_t *__restrict__ on_path,
                                                 int64_t budget, int transition, int rehydrate,
                                                 int64_t *__restrict__ row, int32_t *status) {
  walk_stats_body(t, k, on_path, budget, transition, rehydrate, row, status);
}

int launch_walk_stats(const arbor_tree_t *tree, const int32_t *k, const uint8_t *on_path,
                      int64_t budget, int transition, int rehydrate, int64_t *row,
                      int32_t *status, hipStream_t stream) {
  Tree t = make_tree(tree);
  if (t.V <= 0) return ARBOR_OK;
  hipLaunchKernelGGL(walk_stats, dim3(1), dim3(AT), 0, stream, t, k, on_path, budget, transition,
                     rehydrate, row, status);
  return hip_ok(hipGetLastError());
}

int launch_allocate(const arbor_tree_t *tree, const int32_t *active, int32_t n_active,
                    int64_t budget_tokens, const float *s, const arbor_params_t *params,
                    int32_t *k_out, int32_t *delta_out, uint8_t *on_path_out, int32_t *status,
                    void *workspace, size_t workspace_bytes, hipStream_t stream, int gate) {
  Tree t = make_tree(tree);
  if (t.V <= 0) return ARBOR_OK;
  // (a workspace too small is refused for trees of any size, also for those whose
  // state fits LDS)
  const int n_wg = (t.V + kNodeThreads - 1) / kNodeThreads;
  Carve cv(workspace, workspace_bytes);
  AllocWs ws;
  ws.down = cv.take<int32_t>(t.V);
  ws.rec = cv.take<NodeRec>(t.V);
  ws.w = cv.take<double>(t.V);
  ws.sums = cv.take<NodeSums>(n_wg);
  ws.gated = cv.take<int32_t>(1);
  if (!cv.ok) return ARBOR_EWORKSPACE;
  AllocParams p{params->alpha_max, params->gamma, params->lambda_d, params->lambda_delta,
                params->eta, params->r_min, params->k_min, params->l_tail,
                params->lazy_rehydration, params->k_protect, {}, {}};
  for (int i = 0; i < kDecay; ++i) {
    p.dexp[i] = exp(-params->lambda_d * (double)i);
    p.texp[i] = exp(-params->lambda_delta * (double)i);
  }
  if (t.V <= kLdsNodes) {
    const size_t lds = ((size_t)t.V * kNodeBytes + 15) / 16 * 16 + (kWave + AT) * 8;
    static_assert(kLdsNodes <= AT && kLdsNodes * kNodeBytes + (kWave + AT) * 8 + 16 <= 64 * 1024,
                  "one thread per node, and no more LDS than a launch may take unasked");
    hipLaunchKernelGGL(allocate_kernel, dim3(1), dim3(AT), lds, stream, t, active, n_active,
                       (int64_t)budget_tokens, s, p, k_out, delta_out, on_path_out, status, gate);
    return hip_ok(hipGetLastError());
  }
#define ARBOR_NODES_ARGS                                                                         \
  t, active, n_active, (int64_t)budget_tokens, s, p, k_out, delta_out, on_path_out, status, ws, gate
  if (t.V <= kGeoNodes) {
    const size_t lds = (size_t)t.V * 8;
    // more than 64 KiB of dynamic LDS has to be allowed explicitly
    static_assert(kGeoNodes * 8 <= 140 * 1024, "within the LDS of a CU");
    if (lds > 60 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(&alloc_nodes<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return ARBOR_EHIP;
    hipLaunchKernelGGL(alloc_nodes<true>, dim3(n_wg), dim3(kNodeThreads), lds, stream,
                       ARBOR_NODES_ARGS);
  } else {
    hipLaunchKernelGGL(alloc_path, dim3(1), dim3(AT), 0, stream, t, active, n_active, status, ws);
    hipLaunchKernelGGL(alloc_nodes<false>, dim3(n_wg), dim3(kNodeThreads), 0, stream,
                       ARBOR_NODES_ARGS);
  }
#undef ARBOR_NODES_ARGS
  if (t.V <= kCutThreads * kRegNodes)
    hipLaunchKernelGGL(alloc_cut<true>, dim3(1), dim3(kCutThreads), 0, stream, t,
                       (int64_t)budget_tokens, p, k_out, on_path_out, status, ws, n_wg);
  else
    hipLaunchKernelGGL(alloc_cut<false>, dim3(1), dim3(kCutThreads), 0, stream, t,
                       (int64_t)budget_tokens, p, k_out, on_path_out, status, ws, n_wg);
  return hip_ok(hipGetLastError());
}

}  // namespace arbor
