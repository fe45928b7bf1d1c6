// arbor_tree_decode_attn: decode attention of every active leaf over the
// resident tokens of its root-to-leaf chain (Sec. 1, Sec. 3: the next decoding
// step depends only on the ancestor chain).
//
// Tree-aware split-K: a work unit is (chain node a, chunk of a's slots, layer,
// kv head, up to 16 of the node's query rows).  The node's rows are the G query
// heads of every active leaf below a, so a shared ancestor is streamed from HBM
// once for all leaves that need it: the units of one chunk that differ only in
// their rows are neighbouring waves, whose loads meet in the caches.  A
// wave computes S = K Q^T with bf16 MFMA (keys along M, so each lane owns one
// query row), an online softmax per fragment of keys, and O += P V.  For
// bf16 pools P is split into a bf16 high part and a bf16 remainder, both
// multiplied with the exact bf16 V by bf16 MFMAs (fp32-level accuracy of P);
// fp32 pools use the fp32 MFMA (16x16x4).  The key order inside each MFMA
// step is permuted so P needs no cross-lane movement.  Each unit writes an
// unnormalised partial (max, sum, o); the merge kernel combines the partials of
// a leaf in root-to-leaf order, so results are bitwise reproducible.
//
// A wave holds 16 rows however many leaves there are.  Waves of 32 and 64 rows, of
// which one fits a SIMD, took 972 us for 64 leaves of the 70B shape and 8 layers
// (now 811), 3,415 for 256 of them (2,804), 824 for 64 leaves of the 8B shape and
// 32 layers (781) and 2,686 for 256 leaves of a 341-block tree (2,378).
#include <type_traits>

#include "arbor_internal.h"
#include "mfma_ops.h"

namespace arbor {

namespace {

constexpr int MAXD = ARBOR_MAX_DEPTH + 1;
static_assert(MAXD == kWave, "one wave covers a chain");
// Slots of a chain node that one work unit takes: the plan picks the largest of
// kChunks that is no longer than a wave's even share of the call, 1 / kWaves of the
// (slot, 16-row block, layer, kv head)s, so that no unit outlasts the others and
// few partials are written and merged; of four fifths of it where a node is
// shorter than the chunk, as uneven units fill the waves less well.  Times at
// this size / at half of it / at twice of it, us: the 8B shape under 4 leaves, 32
// layers 117 / - / 122, 16 layers 57.4 / 60.4 / -, 8 layers 37.0 / 41.2 / 37.6;
// the 70B shape under one leaf, 20 layers 117 / 129 / -, under 8 leaves 349 at
// 1,024, 373 at 512, 402 at 256, and for 4 layers 82 / 96 / -; 16 leaves of a
// 341-block tree, 8 layers 66.4 / 68.2 / 79.2, one layer 35 at 64, 91 at 256.
// Taking the largest size that gives 4,096 units instead cut the calls of few
// rows too finely (the second figures).
constexpr int kChunks[] = {1024, 512, 256, 128, 64};
constexpr int kNChunks = 5;
constexpr int kMinChunk = 64, kMaxChunk = 1024;
constexpr int kWaves = 2048;      // two for every SIMD, as the registers of d = 128 allow
constexpr int kWaves64 = 3072;    // bf16 pools of d = 64: three
constexpr int kPartSlots = 256;   // slots of a unit that share a reference max
// fp32 pools, whose slots are twice the bytes: units of at most 256 slots, so that
// none is summed in parts, whose second accumulator would leave two waves per
// SIMD instead of three (8 layers of the 70B shape: 306 us, in parts of longer
// units 390)
constexpr int kFirstChunkF32 = 2;
static_assert(kChunks[kFirstChunkF32] <= kPartSlots, "no parts");
constexpr int kPlanLds = 4096;    // trees up to this many nodes are walked from LDS
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// One chunk of a chain node and one block of 16 of its rows (for every layer
// and kv head): all a wave needs besides the page ids and its query rows.
struct __attribute__((aligned(16))) Unit {
  int32_t po;        // first page-table entry of the node
  int32_t s_begin;   // first slot
  int32_t n_slots;
  int32_t rowbase;   // partial row of the chunk's row 0
  int32_t R;         // rows of the node: G per leaf below it
  int32_t loff;      // its leaves in leaf_list
  int32_t first;     // unit of the chunk's row block 0
  int32_t zbase;     // its kept logits, [R][slots rounded up to 64]: first block of 64
  int32_t node;
  int32_t piece0;    // credit calls with a list of pieces: the chunk's first one
  int32_t pad[2];
};
static_assert(sizeof(Unit) == 48, "three 16-byte loads");

struct Meta {
  int32_t n_units, rows, chunk, z_total;
  int32_t max_np, n_pieces;
  int64_t parts;     // float offsets from `rest`: leaf_part entries, max_np per leaf,
  int64_t pieces;    //   the unit of each listed 64-slot piece (credit calls),
  int64_t ml;        //   (max, sum) of the partial rows,
  int64_t part;      //   their unnormalised outputs,
  int64_t z;         //   kept logits
};

struct DecArgs {
  Tree t;
  Pool pl;
  const int32_t *leaves;
  int n_leaves;
  int l0, Lr;
  const void *q;
  float sl2;
  // plan outputs
  Meta *meta;
  int32_t *leaf_list;   // leaves below each chain node, in leaf order
  int32_t *lanc;        // [n_leaves][MAXD] chain of each leaf, root first
  int32_t *ldepth;
  int32_t *leaf_np;     // partials of each leaf's chain
  int32_t *ent_p0;      // [n_leaves][MAXD]: first listed piece of an entry's node
  // units, leaf_part (first partial row of the leaf's heads, per partial), the
  // partials and the kept logits follow one another here
  float *rest;
  int64_t rest_cap;     // floats
  int zS;               // credit calls: distinct slice layers whose logits the units keep
  int zlr[8];           //   (relative to l0); zS = 0 otherwise
  int32_t *status;
};

__device__ __forceinline__ const Unit *units_of(const DecArgs &a) {
  return reinterpret_cast<const Unit *>(a.rest);
}

// The decode-time credit of accumulated attention: slice layers relative to
// the call's first layer, the crediting mode and the caller's A / rows_seen.
struct CreditArgs {
  int S;          // slice entries (a layer may be listed more than once)
  int U;          // distinct slice layers: the units keep logits for these
  int slice[8];   // distinct slice layers
  int mult[8];    //   and how often each is listed
  int self_window;
  float *A;
  int64_t *rows_seen;
};

// Plan of one call, in one workgroup.  Every (leaf, depth) entry of the active
// chains finds the other leaves below its node: the first of them stands for
// the node (its entry's rank is 0) and brings the node's units, the others
// only their place in its leaf list.  The work is O(leaves depth), not O(V):
// only the parent links are read for the whole tree (into LDS, for trees of up
// to kPlanLds nodes, so that the chain walks do not wait on global memory).
// There the leaves below a node are one 64-bit mask, set during the walks (up
// to kPlanLeaves leaves); otherwise an entry compares its node with the other
// leaves' nodes of its depth.  The units are written by all threads, each
// finding its unit's entry by a binary search.  SMALL / FEW are template
// arguments, so that every access compiles to an LDS or a global instruction
// rather than a flat one; WAVES and FIRST are the pool's rule of the
// chunk size.
// Bound by latency: 16 leaves of a 341-block tree take 8.0 us; with a
// comparison against every leaf and each node's thread writing its units
// 14.8, and 9.7 for the former plan, which scanned all V nodes.
constexpr int kPlanLeaves = 64;
constexpr int kCreditGroups = 256;   // workgroups that credit

// per-entry state, [n_leaves][MAXD] each (workspace for many leaves); entry
// e = leaf * ds + depth for chains of at most ds blocks
struct PlanEnt {
  int32_t *up;       // [n_leaves][MAXD]: the chain, leaf first
  int32_t *kept, *rbase, *loff, *np, *u0, *z0;
  uint64_t *place;   // rank | first << 21 | leaves below << 42
};
constexpr int kPlanEnts = 7;

struct Place {
  int rank, first, nl;
};

template <bool SMALL, bool FEW, int WAVES, int FIRST>
__global__ __launch_bounds__(1024) void decode_plan(DecArgs a, PlanEnt gent) {
  constexpr bool MASKS = SMALL && FEW;
  constexpr int kEnt = FEW ? kPlanLeaves * MAXD : 1;
  __shared__ int64_t sm[4 * 16];
  __shared__ unsigned s_work;
  __shared__ int s_least;
  __shared__ int s_err, s_maxd, s_maxnp;
  // the parent links are not needed once the chains are known: u0 takes their place
  static_assert(kPlanLds >= kPlanLeaves * MAXD, "u0 fits");
  __shared__ int32_t s_par[SMALL ? kPlanLds : kEnt];
  __shared__ uint64_t s_mask[MASKS ? kPlanLds : kEnt];   // or the entries' places
  __shared__ int32_t s_ent[kPlanEnts - 1][kEnt];
  __shared__ int32_t s_ldep[FEW ? kPlanLeaves : 1];
  const Tree &t = a.t;
  const int V = t.V, G = a.pl.G, nb = a.n_leaves;
  // (loaded here, not where they are used)
  const int zS = a.zS, planes = a.Lr * a.pl.Hkv;
  asm volatile("" : : "s"(zS), "s"(planes));
  const int nt = blockDim.x, tid = threadIdx.x;
  // each thread's first node and leaf are loaded together with the status word
  const int par0 = SMALL && tid < V ? t.parent[tid] : 0;
  const int leaf0 = tid < nb ? a.leaves[tid] : 0;
  if (status_failed(a.status)) {
    if (tid == 0) a.meta->n_units = 0;
    return;
  }
  PlanEnt en;
  if constexpr (FEW)
    en = PlanEnt{s_ent[0], s_ent[1], s_ent[2], s_ent[3], s_ent[4], s_par, s_ent[5], s_mask};
  else
    en = gent;
  int32_t *ldepp = FEW ? s_ldep : a.ldepth;
  if (tid == 0) {
    s_err = s_maxd = s_maxnp = 0;
    s_work = 0;
    s_least = INT32_MAX;
  }
  if constexpr (SMALL)
    for (int i = tid; i < V; i += nt) {
      s_par[i] = i == tid ? par0 : t.parent[i];
      if (MASKS) s_mask[i] = 0;
    }
  const int32_t *par = SMALL ? s_par : t.parent;
  __syncthreads();
  for (int b = tid; b < nb; b += nt) {
    const int l = b == tid ? leaf0 : a.leaves[b];
    int d = 0, bad = l < 0 || l >= V ? 1 : 0;
    // validate the chain and keep it, leaf first
    for (int x = l; x >= 0 && !bad;) {
      const int px = par[x];
      if (px >= x || px < (x > 0 ? 0 : -1)) bad = 1;
      else if (d == MAXD) bad = 2;
      else en.up[b * MAXD + d++] = x;
      if (MASKS)
        atomicOr(reinterpret_cast<unsigned long long *>(&s_mask[x]), 1ull << (b & 63));
      x = px;
    }
    if (bad) {
      atomicOr(&s_err, bad);
      d = 0;
    }
    ldepp[b] = d - 1;
    if (FEW) a.ldepth[b] = d - 1;
    atomicMax(&s_maxd, d - 1);
  }
  __syncthreads();
  if (s_err) {
    if (tid == 0) {
      status_error(a.status, (s_err & 1) ? ARBOR_EINVAL : ARBOR_EUNSUPPORTED);
      a.meta->n_units = 0;
    }
    return;
  }
  const int ds = s_maxd + 1;
  const int n_e = nb * ds;
  // the leaves below the node of entry e (node x of leaf b at depth d)
  auto place = [&](int e, int b, int x) __attribute__((always_inline)) -> Place {
    const uint64_t m = en.place[MASKS ? x : e];
    if constexpr (MASKS)
      return Place{popc(m & ((1ull << b) - 1)), (int)__builtin_ctzll(m), popc(m)};
    constexpr uint64_t k = (1ull << 21) - 1;
    return Place{(int)(m & k), (int)((m >> 21) & k), (int)(m >> 42)};
  };
  int64_t work = 0;          // slots times row blocks
  int least = INT32_MAX;     // the shortest node's slots
  for (int e = tid; e < n_e; e += nt) {
    const int b = e / ds, d = e - b * ds;
    const int dl = ldepp[b];
    if (d > dl) continue;
    const int x = en.up[b * MAXD + dl - d];
    const int c = t.n_kept[x];
    if constexpr (!MASKS) {
      int r = 0, cnt = 0, first = b;
#pragma unroll 4
      for (int b2 = 0; b2 < nb; ++b2) {
        const int d2 = ldepp[b2];
        const bool same = d2 >= d && en.up[b2 * MAXD + (d2 >= d ? d2 - d : 0)] == x;
        cnt += same ? 1 : 0;
        r += same && b2 < b ? 1 : 0;
        first = same && b2 < first ? b2 : first;
      }
      en.place[e] = (uint64_t)r | ((uint64_t)first << 21) | ((uint64_t)cnt << 42);
    }
    const Place pc = place(e, b, x);
    a.lanc[b * MAXD + d] = x;
    en.kept[e] = c;
    if (pc.rank == 0) {
      work += (int64_t)c * ((pc.nl * G + 15) / 16);
      if (c > 0) least = min(least, c);
    }
  }
  // the chunk size (a thread's work counts up to the largest one's need: the sum
  // of 1,024 threads fits 32 bits)
  int C = kMinChunk;
  {
    constexpr int64_t kMost = (int64_t)kMaxChunk * WAVES * 5 / 4;
    static_assert(kMost <= 1 << 22, "1,024 of them fit");
    const int64_t all = work * planes;
    if ((tid & ~(kWave - 1)) < n_e) {
      const unsigned v = wave_sum((unsigned)(all < kMost ? all : kMost));
      const int lo = wave_allreduce(least, [](int x, int y) { return min(x, y); });
      if (lane_id() == 0) {
        atomicAdd(&s_work, v);
        atomicMin(&s_least, lo);
      }
    }
    __syncthreads();
    const unsigned s = (unsigned)__builtin_amdgcn_readfirstlane((int)s_work);
    const int lo = __builtin_amdgcn_readfirstlane(s_least);
#pragma unroll
    for (int k = kNChunks - 2; k >= FIRST; --k) {
      const unsigned need = (unsigned)(kChunks[k] * WAVES);
      C = s >= (lo < kChunks[k] ? need / 4 * 5 : need) ? kChunks[k] : C;
    }
  }
  const int lc = 31 - __builtin_clz(C);      // chunks of c slots: (c + C - 1) >> lc
  // units, partial rows, leaf-list places and logit slots of every node, in
  // the order of its first leaf's chain; v[0] carries units (high half) and
  // leaf-list entries (low half)
  // (in a credit call whose chunks have several 64-slot pieces v[3] counts those,
  // for the list from which the credit's workgroups take them)
  const bool pieced = zS > 0 && C > kWave;
  int64_t run[4] = {0, 0, 0, 0};
  for (int base = 0; base < n_e; base += nt) {
    const int e = base + tid;
    const int b = e / ds, d = e - b * ds;
    int64_t v[4] = {0, 0, 0, 0};
    if (e < n_e && d <= ldepp[b]) {
      const int c = en.kept[e];
      const int chunks = (c + C - 1) >> lc;
      // the entry's place among its leaf's partials: the chunks above it
      int np = 0;
      for (int d2 = 0; d2 < d; ++d2) np += (en.kept[e - d + d2] + C - 1) >> lc;
      en.np[e] = np;
      if (d == ldepp[b]) {
        a.leaf_np[b] = np + chunks;
        atomicMax(&s_maxnp, np + chunks);
      }
      const Place pc = place(e, b, en.up[b * MAXD + ldepp[b] - d]);
      if (pc.rank == 0) {
        const int R = pc.nl * G;
        v[0] = ((int64_t)chunks * ((R + 15) / 16) << 32) | pc.nl;
        v[1] = (int64_t)chunks * R;
        v[2] = (int64_t)R * ((c + 63) / 64);
        v[3] = (c + 63) / 64;
      }
    }
    int64_t ex[4], tot[4];
    if (pieced) {
      block_exclusive_scan_n<4>(v, ex, tot, sm, n_e - base);
      if (e < n_e) a.ent_p0[e] = (int)(run[3] + ex[3]);
    } else {
      const int64_t v3[3] = {v[0], v[1], v[2]};
      int64_t ex3[3], tot3[3];
      block_exclusive_scan_n<3>(v3, ex3, tot3, sm, n_e - base);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        ex[k] = ex3[k];
        tot[k] = tot3[k];
      }
      tot[3] = 0;
    }
    if (e < n_e) {
      en.u0[e] = (int)((run[0] + ex[0]) >> 32);
      en.loff[e] = (int)(uint32_t)(run[0] + ex[0]);
      en.rbase[e] = (int)(run[1] + ex[1]);
      en.z0[e] = (int)(run[2] + ex[2]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) run[k] += tot[k];
  }
  __syncthreads();
  const int64_t n_units = run[0] >> 32;
  const int max_np = s_maxnp;
  // no list where every place of every unit has a workgroup of its own anyway
  // (building one took 0.9 us)
  const bool listed = pieced && n_units * (C / kWave) > kCreditGroups;
  if (!listed) run[3] = 0;
  const int64_t parts = n_units * (int64_t)(sizeof(Unit) / 4);
  const int64_t pieces = parts + (int64_t)nb * max_np;
  if (tid == 0) {
    // the units, the partial and piece lists, the partials, then (credit calls) the
    // slice-layer logits of every node's rows and slots, in blocks
    // of 64 floats: [slice][kv head][z_total]
    Meta m;
    m.n_units = (int32_t)n_units;
    m.rows = (int32_t)run[1];
    m.chunk = C;
    m.z_total = (int32_t)run[2];
    m.max_np = max_np;
    m.n_pieces = (int32_t)run[3];
    m.parts = parts;
    m.pieces = pieces;
    m.ml = (pieces + run[3] + 3) & ~(int64_t)3;
    m.part = (m.ml + run[1] * planes * 2 + 3) & ~(int64_t)3;
    m.z = m.part + run[1] * planes * a.pl.D;
    const int64_t need = m.z + (int64_t)a.zS * a.pl.Hkv * run[2] * 64;
    if (need > a.rest_cap || run[1] > INT32_MAX || run[2] > INT32_MAX) {
      status_error(a.status, ARBOR_EWORKSPACE);
      m.n_units = 0;
    }
    *a.meta = m;
  }
  // the units
  Unit *units = reinterpret_cast<Unit *>(a.rest);
  int32_t *piece_unit = reinterpret_cast<int32_t *>(a.rest) + pieces;
  const int64_t piece_cap = a.rest_cap - pieces;
  const int64_t unit_cap = a.rest_cap / (int64_t)(sizeof(Unit) / 4);
  for (int64_t i = tid; i < n_units && i < unit_cap; i += nt) {
    int lo = 0, hi = n_e - 1;                 // the last entry with u0 <= i
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (en.u0[mid] <= (int)i) lo = mid;
      else hi = mid - 1;
    }
    const int b = lo / ds, d = lo - b * ds;
    const int x = en.up[b * MAXD + ldepp[b] - d];
    const int po = (int)t.page_off[x];
    const int p0 = listed ? a.ent_p0[lo] : 0;
    const int c = en.kept[lo];
    const int R = place(lo, b, x).nl * G;
    const int nbr = (R + 15) / 16;
    const int q = ((int)i - en.u0[lo]) / nbr;
    Unit u;
    u.po = po;
    u.s_begin = q << lc;
    u.n_slots = min(C, c - (q << lc));
    u.rowbase = en.rbase[lo] + q * R;
    u.R = R;
    u.loff = en.loff[lo];
    u.first = en.u0[lo] + q * nbr;
    u.zbase = en.z0[lo] + R * (q << (lc - 6));
    u.node = x;
    u.piece0 = p0 + (q << (lc - 6));
    u.pad[0] = u.pad[1] = 0;
    units[i] = u;
    if (listed && u.first == (int)i)
      for (int j = 0; j * kWave < u.n_slots; ++j)
        if (u.piece0 + j < piece_cap) piece_unit[u.piece0 + j] = (int32_t)i;
  }
  // the leaves below each node, and each leaf's partials, root first (so the
  // merge needs no chain walk)
  int32_t *leaf_part = reinterpret_cast<int32_t *>(a.rest) + parts;
  const int64_t parts_cap = a.rest_cap - parts;
  for (int e = tid; e < n_e; e += nt) {
    const int b = e / ds, d = e - b * ds;
    if (d > ldepp[b]) continue;
    const Place pc = place(e, b, en.up[b * MAXD + ldepp[b] - d]);
    const int f = pc.first * ds + d;
    a.leaf_list[en.loff[f] + pc.rank] = b;
    const int nch = (en.kept[e] + C - 1) >> lc;
    const int rb = en.rbase[f] + pc.rank * G, rows = pc.nl * G;
    const int64_t o = (int64_t)b * max_np + en.np[e];
    for (int q = 0; q < nch; ++q)
      if (o + q < parts_cap) leaf_part[o + q] = rb + q * rows;
  }
}

// K and V of GSP consecutive 16-slot sub-pages of one unit, in MFMA operand
// layout: lane (rr, g4) holds key row rr of each sub-page (S = K Q^T), and
// value rows 4 g4 + e, columns NC rr .. NC rr + NC - 1 (O += P V).
template <class T, int D, int GSP>
struct KVFrag {
  typedef typename std::conditional<sizeof(T) == 2, __bf16, float>::type VT;
  static constexpr int KS = D / 4 / Op<T>::kPerStep;
  static constexpr int NC = D / 16;
  typename Op<T>::reg k[GSP][KS];
  VT v[GSP][4][NC];
  int nval[GSP];  // valid slots of each sub-page (0: padding, never counted); wave-uniform
};

// Where a unit's rows live: the (layer, kv head) plane of K and V at page 0,
// the bytes between pages, and this lane's offsets within a 16-row sub-page.
struct UnitAddr {
  const char *k, *v;
  int64_t page_bytes;
  int row_bytes;
  uint32_t koff, voff;
};

template <class T, int D, int GSP>
__device__ __forceinline__ KVFrag<T, D, GSP> fetch_kv(const UnitAddr &ua, int pg, int s_begin,
                                                      int s_end, int n_sub, int sub0, int P) {
  typedef KVFrag<T, D, GSP> F;
  F f;
#pragma unroll
  for (int sp = 0; sp < GSP; ++sp) {
    // clamped to a valid sub-page so that every load is unconditional
    const int sub = min(sub0 + sp, n_sub - 1);
    const int q0 = s_begin + sub * 16;
    f.nval[sp] = sub0 + sp < n_sub ? min(16, s_end - q0) : 0;
    // lane j holds sub-page j's page; the page base is wave-uniform
    const int page = __builtin_amdgcn_readlane(pg, sub);
    const int64_t base = (int64_t)page * ua.page_bytes + (int64_t)(q0 % P) * ua.row_bytes;
    const char *kp = ua.k + base + ua.koff;
    const char *vp = ua.v + base + ua.voff;
#pragma unroll
    for (int ks = 0; ks < F::KS; ++ks)
      f.k[sp][ks] = Op<T>::load(reinterpret_cast<const T *>(kp + frag_col<T>(ks, 0) * (int)sizeof(T)));
    // fp32 rows of 512 bytes: all loads of K go out before those of V, and none is
    // held back to its use (the compiler otherwise waits for each 16 bytes of K
    // in turn: 121 us for 16 layers of the 8B shape instead of 110)
    if constexpr (sizeof(T) == 4 && D == 128) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const typename F::VT *vr = reinterpret_cast<const typename F::VT *>(vp + e * ua.row_bytes);
#pragma unroll
      for (int cc = 0; cc < F::NC; ++cc) f.v[sp][e][cc] = vr[cc];
    }
  }
  return f;
}

// Online-softmax update of one wave's rows with one fragment.  Slots past a
// sub-page's resident count may hold anything: only a ragged sub-page (the
// last of a node) masks its logits and zeroes its value rows.  The output is
// rescaled only when some row's running max moved.  A logit is scaled and
// taken relative to the max in one fused step, so it is rounded once.
// zs (when keep_z) receives the fragment's masked products of query and key,
// which the decode-time credit turns into weights later; the caller stores them.
template <class T, int D, int GSP>
__device__ __forceinline__ void attend(KVFrag<T, D, GSP> &f,
                                       const typename Op<T>::reg (&q)[KVFrag<T, D, GSP>::KS],
                                       float sl2, int g4, float &m_run, float &l_run,
                                       f32x4 (&o)[D / 16], bool keep_z, float (&zs)[GSP][4]) {
  typedef KVFrag<T, D, GSP> F;
  constexpr int NC = F::NC;
  float sv[GSP][4];
  float gmax = -__builtin_inff();
#pragma unroll
  for (int sp = 0; sp < GSP; ++sp) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < F::KS; ++ks) acc = Op<T>::mma(f.k[sp][ks], q[ks], acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) sv[sp][e] = acc[e];
    if (f.nval[sp] < 16) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sv[sp][e] = 4 * g4 + e < f.nval[sp] ? sv[sp][e] : -__builtin_inff();
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cc = 0; cc < NC; ++cc)
          f.v[sp][e][cc] = 4 * g4 + e < f.nval[sp] ? f.v[sp][e][cc] : (typename F::VT)0.f;
    }
    gmax = fmaxf(gmax, fmaxf(fmaxf(sv[sp][0], sv[sp][1]), fmaxf(sv[sp][2], sv[sp][3])));
    if (keep_z) {
#pragma unroll
      for (int e = 0; e < 4; ++e) zs[sp][e] = sv[sp][e];
    }
  }
  gmax = across_rows(gmax, [](float x, float y) { return fmaxf(x, y); });
  const float mn = fmaxf(m_run, gmax * sl2);
  const bool moved = mn != m_run;
  const float alpha = m_run > -__builtin_inff() ? __builtin_amdgcn_exp2f(m_run - mn) : 0.f;
  m_run = mn;
  if (__builtin_amdgcn_ballot_w64(moved) != 0) {
    l_run *= alpha;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float fe = __shfl(alpha, 4 * g4 + e, kWave);
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) o[cc][e] *= fe;
    }
  }
  const float nm = m_run > -__builtin_inff() ? -m_run : 0.f;
  if constexpr (sizeof(T) == 2) {
    // bf16 values: O += P V as bf16 MFMAs (16x16x32), one per 16 output
    // columns and pair of sub-pages sp0, sp0 + 1 of the fragment, element t =
    // 4 (sp - sp0) + e of a lane's k-slice being key 4 g4 + e of sub-page sp
    // (zero past GSP sub-pages).  P is split into a bf16 high part and a bf16
    // remainder, p = hi + lo to about 2^-17 relative, and both are multiplied
    // by the exact bf16 V, so the product keeps fp32-level accuracy at a
    // quarter of the fp32 MFMA's issue time.
#pragma unroll
    for (int sp0 = 0; sp0 < GSP; sp0 += 2) {
      bf16x8 ph, pl;
      float p[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int sp = sp0 + t / 4, e = t % 4;
        p[t] = sp < GSP ? __builtin_amdgcn_exp2f(
                              __builtin_fmaf(sv[sp < GSP ? sp : 0][e], sl2, nm))
                        : 0.f;
        const __bf16 hi = (__bf16)p[t];
        ph[t] = hi;
        pl[t] = (__bf16)(p[t] - (float)hi);
      }
      // (pairwise: the running sum of 256 slots takes 8 terms, not 64)
      l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) {
        bf16x8 vv;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int sp = sp0 + t / 4;
          vv[t] = sp < GSP ? (__bf16)f.v[sp < GSP ? sp : 0][t % 4][cc] : (__bf16)0.f;
        }
        o[cc] = Op<__bf16>::mma(ph, vv, o[cc]);
        o[cc] = Op<__bf16>::mma(pl, vv, o[cc]);
      }
    }
  } else {
#pragma unroll
    for (int sp = 0; sp < GSP; ++sp) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[sp][e], sl2, nm));
      l_run += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int cc = 0; cc < NC; ++cc) o[cc] = mma_f32(p[ks], (float)f.v[sp][ks][cc], o[cc]);
    }
  }
}

// Sub-pages a wave loads at once: 16 KB of K and V in flight per wave, one
// fragment at a time.  With a single buffer two waves fit a SIMD for bf16
// pools of d = 128 (195 registers, scored 206) and three or four (plain fp32, d = 64)
// otherwise, and their loads overlap one another's work.  Double-buffered
// fragments, or larger ones, leave one wave per SIMD (two where there were
// three) and stream HBM more slowly, measured on the llama8b and dpts trees.
template <class T, int D>
constexpr int sub_pages_per_fetch() {
  constexpr int per = 32 * D * (int)sizeof(T);   // K and V of one 16-slot sub-page
  return (16 << 10) / per < 1 ? 1 : (16 << 10) / per;
}

// One wave: one unit (a chunk of a chain node's slots, one layer, one kv
// head), rows [rbase, rbase + 16).  The unit's sub-pages are taken GSP at
// a time (the last fragment of a unit re-reads its last sub-page in the
// unused places, which the cache serves); other waves of the SIMD attend
// while one waits for its fragment.
// KZ: the call credits (some slice layers keep their logits); a plain call
// compiles without that path and its registers.
template <class T, int D, bool KZ>
__device__ __forceinline__ void decode_unit(const DecArgs &a, const Meta &mt, const Unit &un,
                                            int lr, int g, int rbase) {
  using O = Op<T>;
  constexpr int GSP = sub_pages_per_fetch<T, D>();
  typedef KVFrag<T, D, GSP> F;
  constexpr int KS = F::KS;
  constexpr int NC = F::NC;
  const Tree &t = a.t;
  const Pool &pl = a.pl;
  const int lane = lane_id();
  const int rr = lane & 15;
  const int g4 = lane >> 4;
  const int G = pl.G;
  const int R = un.R;
  const int s_begin = un.s_begin, s_end = un.s_begin + un.n_slots;
  const int layer = a.l0 + lr;
  const int Hq = pl.Hkv * G;
  const int n_sub = (un.n_slots + 15) / 16;
  const int n_grp = (n_sub + GSP - 1) / GSP;
  // page ids of all sub-pages up front: a dependent load inside the pipeline
  // would make every wait cover the fragment still in flight
  static_assert(kMaxChunk / 16 <= kWave, "one lane per sub-page");
  const int pg = lane < n_sub ? t.page_table[un.po + (s_begin + 16 * lane) / pl.P] : 0;

  const int r = rbase + rr;
  typename O::reg q[KS];
  if (r < R) {
    const int b = a.leaf_list[un.loff + r / G];
    const int h = g * G + r % G;
    const T *qp = static_cast<const T *>(a.q) + (((int64_t)b * a.Lr + lr) * Hq + h) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = O::load(qp + frag_col<T>(ks, g4));
  } else {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = O::zero();
  }
  UnitAddr ua;
  {
    const int esz = (int)sizeof(T);
    ua.row_bytes = D * esz;
    ua.page_bytes = (int64_t)pl.Hkv * pl.P * D * esz;
    const int64_t plane = ((int64_t)layer * pl.num_pages * pl.Hkv + g) * pl.P * D * esz;
    ua.k = static_cast<const char *>(pl.k) + plane;
    ua.v = static_cast<const char *>(pl.v) + plane;
    ua.koff = (uint32_t)(rr * D * esz + frag_col<T>(0, g4) * esz);
    ua.voff = (uint32_t)(4 * g4 * D * esz + F::NC * rr * esz);
  }
  // a credited slice layer keeps its logits: [slice][kv head][unit row][slot]
  float *zrow = nullptr;
  const int zstride = (un.n_slots + 63) & ~63;
  for (int z = 0; KZ && z < a.zS; ++z)
    if (a.zlr[z] == lr) {
      zrow = a.rest + mt.z + (((int64_t)z * pl.Hkv + g) * mt.z_total + un.zbase) * 64 +
             (int64_t)r * zstride;
      break;
    }
  F cur = fetch_kv<T, D, GSP>(ua, pg, s_begin, s_end, n_sub, 0, pl.P);
  float m_run = -__builtin_inff(), l_run = 0.f;
  f32x4 o[NC];
#pragma unroll
  for (int cc = 0; cc < NC; ++cc) o[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
  // A longer unit is summed in parts of kPartSlots, each against its own max, and
  // the parts are merged as partials of units of that size would be: weights far
  // below the max carry the rounding of their distance to it, so one max for
  // 1,024 slots lost accuracy (fp32 outputs of the 70B shape, nodes of 512
  // slots: 4.4e-7 from 64 bits, in parts 3.6e-7).
  constexpr int kPart = kPartSlots / (16 * GSP);
  constexpr bool PARTS = sizeof(T) == 2;
  float m_tot, l_tot;               // (set by the first part)
  f32x4 ot[NC];
  auto first_part = [&]() __attribute__((always_inline)) {
    m_tot = m_run;
    l_tot = l_run;
    m_run = -__builtin_inff();
    l_run = 0.f;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      ot[cc] = o[cc];
      o[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto merge_part = [&]() __attribute__((always_inline)) {
    const float mn = fmaxf(m_tot, m_run);
    const float ft = m_tot > -__builtin_inff() ? __builtin_amdgcn_exp2f(m_tot - mn) : 0.f;
    const float fr = m_run > -__builtin_inff() ? __builtin_amdgcn_exp2f(m_run - mn) : 0.f;
    l_tot = __builtin_fmaf(l_tot, ft, l_run * fr);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float te = __shfl(ft, 4 * g4 + e, kWave), re = __shfl(fr, 4 * g4 + e, kWave);
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) {
        ot[cc][e] = __builtin_fmaf(ot[cc][e], te, o[cc][e] * re);
        o[cc][e] = 0.f;
      }
    }
    m_tot = mn;
    m_run = -__builtin_inff();
    l_run = 0.f;
  };
  // the logits of fragment gi are stored after fragment gi + 1's loads are
  // issued: a wave's loads and stores share one counter, so a wait for loads
  // issued after the stores would wait for the stores as well
  float zs[GSP][4];
  auto store_z = [&](int gz) __attribute__((always_inline)) {
    // lane (rr, g4) holds keys 4 g4 .. 4 g4 + 3 of each sub-page for row rr
#pragma unroll
    for (int sp = 0; sp < GSP; ++sp)
      if (gz * GSP + sp < n_sub && r < R)
        *reinterpret_cast<float4 *>(zrow + 16 * (gz * GSP + sp) + 4 * g4) =
            make_float4(zs[sp][0], zs[sp][1], zs[sp][2], zs[sp][3]);
  };
  for (int gi = 0; gi < n_grp; ++gi) {
    if (gi > 0) {
      cur = fetch_kv<T, D, GSP>(ua, pg, s_begin, s_end, n_sub, gi * GSP, pl.P);
      if (KZ && zrow) store_z(gi - 1);
    }
    attend<T, D, GSP>(cur, q, a.sl2, g4, m_run, l_run, o, KZ && zrow != nullptr, zs);
    if (PARTS && gi % kPart == kPart - 1 && gi + 1 < n_grp) {
      if (gi < kPart) first_part();
      else merge_part();
    }
  }
  if (PARTS && n_grp > kPart) {
    merge_part();
    m_run = m_tot;
    l_run = l_tot;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) o[cc] = ot[cc];
  }
  if (KZ && zrow && n_grp > 0) store_z(n_grp - 1);
  // partial rows of this unit: (max, sum) pairs and outputs
  const int64_t prow = ((int64_t)lr * pl.Hkv + g) * mt.rows + un.rowbase;
  const float l = across_rows(l_run, [](float x, float y) { return x + y; });
  if (g4 == 0 && r < R)
    reinterpret_cast<float2 *>(a.rest + mt.ml)[prow + r] = make_float2(m_run, l);
  float *outp = a.rest + mt.part + prow * D + NC * rr;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int orow = rbase + 4 * g4 + e;
    if (orow < R) {
#pragma unroll
      for (int cc = 0; cc < NC; cc += 4)
        *reinterpret_cast<float4 *>(outp + (int64_t)orow * D + cc) =
            make_float4(o[cc][e], o[cc + 1][e], o[cc + 2][e], o[cc + 3][e]);
    }
  }
}

// Waves take (unit, layer, kv head) in turn: chunk by chunk, over its planes
// (whose rows of a page lie side by side), the chunk's row blocks innermost.
// In a plain call every other workgroup takes them from the end: the shared blocks
// near the root (many rows, so bound by the matrix cores) come first in the plan's
// order, and run beside the leaves' (bound by HBM): 344 us against 355 in order on
// 8 leaves of the 70B shape.  A credit call takes them in order: 132.3 us against
// 135.4 on the 8B shape after an eviction, 185 / 196 for 16 leaves of the dpts
// shape, 2,308 / 2,587 for 256, and 387 / 400 on 8 leaves of the 70B shape.
template <class T, int D, bool KZ>
__global__ __launch_bounds__(256) void decode_attn(DecArgs a) {
  const int planes = a.Lr * a.pl.Hkv;
  // the wave index is wave-uniform: keep the unit's bookkeeping scalar
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (loaded together with the status word)
  const Meta mt = *a.meta;
  if (status_failed(a.status)) return;
  const int64_t total = (int64_t)mt.n_units * planes;
  const int64_t nblk = (total + 3) / 4;
  for (int64_t vb = blockIdx.x; vb < nblk; vb += gridDim.x) {
    const int64_t blk = KZ ? vb : (vb & 1) ? nblk - 1 - vb / 2 : vb / 2;
    const int64_t w = blk * 4 + wave;
    if (w >= total) continue;
    const Unit un = units_of(a)[w / planes];
    const int p = (int)(w - (int64_t)un.first * planes);
    const int nbr = (un.R + 15) / 16;
    const int plane = p / nbr;
    decode_unit<T, D, KZ>(a, mt, un, plane / a.pl.Hkv, plane % a.pl.Hkv, 16 * (p % nbr));
  }
}

// One wave per (leaf, layer, query head): merge the partials of the leaf's
// chain.  Lane k holds partial k's (max, sum); the running max and the weights
// come from fixed-order wave reductions, and o is accumulated in partial order,
// so the result does not depend on scheduling.  Workgroups blk of nblk take
// the rows in turn.
template <int D>
__device__ __forceinline__ void merge_rows(const DecArgs &a, const Meta &mt, void *out,
                                           int out_dtype, float *lse_out, int blk, int nblk) {
  constexpr int EPL = D / 64;  // output columns per lane
  constexpr int U = 8;         // partial rows loaded together
  constexpr int kPreO = 8;     // partial rows read ahead of the max
  const Pool &pl = a.pl;
  const int lane = lane_id();
  const int G = pl.G;
  const int Hq = pl.Hkv * G;
  const int64_t total = (int64_t)a.n_leaves * a.Lr * Hq;
  const int wpb = blockDim.x / kWave;
  for (int64_t w = (int64_t)blk * wpb + threadIdx.x / kWave; w < total;
       w += (int64_t)nblk * wpb) {
    const int b = (int)(w / (a.Lr * Hq));
    const int rem = (int)(w % (a.Lr * Hq));
    const int lr = rem / Hq;
    const int h = rem % Hq;
    const int g = h / G;
    const int hl = h % G;
    const int64_t row0 = ((int64_t)lr * pl.Hkv + g) * mt.rows + hl;
    const float2 *ml = reinterpret_cast<const float2 *>(a.rest + mt.ml) + row0;
    const float *base = a.rest + mt.part + row0 * D + EPL * lane;
    const int np = a.leaf_np[b];
    const int32_t *lp = reinterpret_cast<const int32_t *>(a.rest) + mt.parts +
                        (int64_t)b * mt.max_np;
    // global max over the chain's partials; the first kWave partials'
    // rows, maxima and sums stay in registers for the second pass (longer
    // chains reload the rest there)
    int off0 = 0;
    float m0 = -__builtin_inff(), l0 = 0.f;
    if (lane < np) {
      off0 = lp[lane];
      const float2 v = ml[off0];
      m0 = v.x;
      l0 = v.y;
    }
    // the output rows of the first kPreO partials are read together with
    // their (max, sum), before the max is known
    float xv0[kPreO][EPL];
    auto load_row = [&](float (&x)[EPL], int row) __attribute__((always_inline)) {
      const float *p = base + (int64_t)row * D;
      if constexpr (EPL == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(p);
        x[0] = v.x;
        x[1] = v.y;
      } else {
        x[0] = p[0];
      }
    };
    static_assert(EPL == 1 || EPL == 2, "head_dim 64 or 128");
#pragma unroll
    for (int u = 0; u < kPreO; ++u) {
      const int oj = lane_value(off0, u < np ? u : 0);
      if (u < np) {
        load_row(xv0[u], oj);
      } else {
#pragma unroll
        for (int e = 0; e < EPL; ++e) xv0[u][e] = 0.f;
      }
    }
    float M = m0;
    for (int k0 = kWave; k0 < np; k0 += kWave) {
      const int k = k0 + lane;
      const float m = k < np ? ml[lp[k]].x : -__builtin_inff();
      M = fmaxf(M, m);
    }
    M = wave_allreduce(M, [](float x, float y) { return fmaxf(x, y); });
    float L = 0.f, ov[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) ov[e] = 0.f;
    if (M > -__builtin_inff()) {
      for (int k0 = 0; k0 < np; k0 += kWave) {
        const int k = k0 + lane;
        int off = 0;
        float f = 0.f, lk = 0.f;
        if (k < np) {
          float m = m0;
          off = off0;
          lk = l0;
          if (k0 > 0) {
            off = lp[k];
            const float2 v = ml[off];
            m = v.x;
            lk = v.y;
          }
          f = m > -__builtin_inff() ? __builtin_amdgcn_exp2f(m - M) : 0.f;
        }
        L += wave_sum(lk * f);
        const int nk = min(kWave, np - k0);
        int jstart = 0;
        if (k0 == 0) {
#pragma unroll
          for (int u = 0; u < kPreO; ++u) {
            const float fu = u < nk ? lane_value(f, u) : 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) ov[e] += (fu > 0.f ? xv0[u][e] * fu : 0.f);
          }
          jstart = kPreO;
        }
        for (int j0 = jstart; j0 < nk; j0 += U) {
          float xv[U][EPL], fj[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = min(j0 + u, nk - 1);
            fj[u] = j0 + u < nk ? lane_value(f, j) : 0.f;
            load_row(xv[u], lane_value(off, j));
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < EPL; ++e) ov[e] += (fj[u] > 0.f ? xv[u][e] * fj[u] : 0.f);
        }
      }
    }
    const int64_t oi = (((int64_t)b * a.Lr + lr) * Hq + h) * D + EPL * lane;
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    if (out_dtype == ARBOR_BF16) {
      __bf16 *op = static_cast<__bf16 *>(out) + oi;
#pragma unroll
      for (int e = 0; e < EPL; ++e) op[e] = (__bf16)(ov[e] * inv);
    } else {
      float *op = static_cast<float *>(out) + oi;
#pragma unroll
      for (int e = 0; e < EPL; ++e) op[e] = ov[e] * inv;
    }
    if (lane == 0) {
      const float l2 = L > 0.f ? M + __log2f(L) : -__builtin_inff();
      const int64_t li = ((int64_t)b * a.Lr + lr) * Hq + h;
      if (lse_out) lse_out[li] = L > 0.f ? l2 * kLn2 : -__builtin_inff();
    }
  }
}

// Decode-time credit (Sec. 4 Execution (iii)): the softmax weight exp2(c z - M)
// / L of every decode query row on every key of a unit, from the products z of
// query and key that the attention units kept for the credited slice layers (c
// the softmax scale in log2 units), summed over the rows whose leaf lies
// strictly below the unit's node (and, in the self-window mode, the leaf's own
// rows on keys before its newest position) and over the slice layers (a layer
// listed m times counts m times) and kv heads, and added to A at the key's
// token.  A row's max M and sum L = sum_k l_k exp2(m_k - M) over the (max m_k,
// sum l_k) of the partials of its leaf's chain are formed here from those
// partials, so the credit does not wait for the merge and runs beside it in the
// same launch.
// One workgroup of kCreditWaves waves per 64 slots of a chunk, one lane per
// slot.  The unit's (row, distinct slice layer, kv head) triples, in
// the order (z * Hkv + g) * R + r, are staged in LDS up to kCreditTile at a
// time: each triple's M and its weight, the layer's multiplicity over L, in one of
// two tables, for the rows of other leaves and for the node's own.  Rows are
// innermost because the (max, sum) pairs of a partial's rows lie side by side,
// so that the lanes of a load share cache lines (with the kv heads innermost
// each lane read a line of its own: 16.8 us for the launch against 13.3, one
// layer under 16 leaves).  Several threads share a triple's partials where there
// are fewer triples than threads.  Wave v takes the triples v, v + kCreditWaves,
// ... in order, kCreditBatch loads at a time, the next batch in flight while one
// is summed; the first batch is issued before the tables are built, and for up to
// kCreditWaves * kCreditBatch triples it is the only one.  A batch's table entries
// come with one LDS read per table (lane u holds entry u).  The two sums of a wave
// are added in wave order, so each token's sum has one owner and a fixed order.
// Workgroup 0 also adds the row counts to rows_seen (integer atomics: order-free).
constexpr int kCreditWaves = 16;
constexpr int kCreditThreads = kCreditWaves * kWave;
constexpr int kCreditTile = 1024;
constexpr int kCreditBatch = 16;
constexpr int kLsePar = 12;           // partials of a chain that a thread loads together
constexpr int kLseThreads = 32;       // most threads of one triple's LSE
static_assert(kMinChunk % kWave == 0, "a chunk is a whole number of 64-slot pieces");
static_assert(kCreditTile % (kCreditWaves * kCreditBatch) == 0, "batches do not straddle tiles");
static_assert(kCreditTile == kCreditThreads, "one thread per triple of a full tile");

// a triple as (row r, zg = z * Hkv + g); dr, dzg: the step of kCreditWaves
struct Triple {
  int r, zg, dr, dzg;
  __device__ __forceinline__ Triple(int e, int R)
      : r(e % R), zg(e / R), dr(kCreditWaves % R), dzg(kCreditWaves / R) {}
  __device__ __forceinline__ void step(int R) {
    r += dr;
    zg += dzg;
    if (r >= R) {
      r -= R;
      ++zg;
    }
  }
};

// logits of the batch of triples it, it + kCreditWaves, ... (it is left at
// the next batch's first triple): zb points at the unit's first logit row and
// the lane's slot; triples past the last one are not read
__device__ __forceinline__ void credit_load(float (&zv)[kCreditBatch], const float *zb, Triple &it,
                                            int R, int per, int64_t z_slab, int zstride) {
#pragma unroll
  for (int u = 0; u < kCreditBatch; ++u) {
    zv[u] = it.zg < per ? zb[it.zg * z_slab + (int64_t)it.r * zstride] : 0.f;
    it.step(R);
  }
}

// (max, sum) of two sets of partials
__device__ __forceinline__ float2 ml_merge(float2 x, float2 y) {
  const float m = fmaxf(x.x, y.x);
  if (m == -__builtin_inff()) return make_float2(m, 0.f);
  const float sx = x.x > -__builtin_inff() ? x.y * __builtin_amdgcn_exp2f(x.x - m) : 0.f;
  const float sy = y.x > -__builtin_inff() ? y.y * __builtin_amdgcn_exp2f(y.x - m) : 0.f;
  return make_float2(m, sx + sy);
}

// (max, sum) of query row (leaf b, layer lr, head g * G + hl) over the partials
// j, j + tpt, ... of b's chain, kLsePar of them loaded together
__device__ __forceinline__ float2 chain_ml(const DecArgs &a, const Meta &mt, int b, int lr, int g,
                                           int hl, int j, int tpt) {
  const float2 *ml = reinterpret_cast<const float2 *>(a.rest + mt.ml) +
                     ((int64_t)lr * a.pl.Hkv + g) * mt.rows + hl;
  const int np = a.leaf_np[b];
  const int32_t *lp = reinterpret_cast<const int32_t *>(a.rest) + mt.parts +
                      (int64_t)b * mt.max_np;
  float2 r = make_float2(-__builtin_inff(), 0.f);
  for (int k0 = j; k0 < np; k0 += kLsePar * tpt) {
    int row[kLsePar];
    float2 v[kLsePar];
#pragma unroll
    for (int u = 0; u < kLsePar; ++u) row[u] = k0 + u * tpt < np ? lp[k0 + u * tpt] : -1;
#pragma unroll
    for (int u = 0; u < kLsePar; ++u)
      v[u] = row[u] >= 0 ? ml[row[u]] : make_float2(-__builtin_inff(), 0.f);
    float m = r.x;
#pragma unroll
    for (int u = 0; u < kLsePar; ++u) m = fmaxf(m, v[u].x);
    if (m == -__builtin_inff()) continue;
    float s = r.x > -__builtin_inff() ? r.y * __builtin_amdgcn_exp2f(r.x - m) : 0.f;
#pragma unroll
    for (int u = 0; u < kLsePar; ++u)
      s += v[u].x > -__builtin_inff() ? v[u].y * __builtin_amdgcn_exp2f(v[u].x - m) : 0.f;
    r = make_float2(m, s);
  }
  return r;
}

// The credit of the 64-slot pieces blk, blk + nblk, ... of the plan's chunks.
// They are numbered as units and places in them, or taken from the plan's list of
// the live ones where there are more such places than workgroups: without it the
// live pieces fell on few of them (blocks of 128 slots in chunks of 1,024 have two
// of sixteen: the launch of 16 leaves and 32 layers took 43.8 us, now 24.2, and
// that of 64 leaves of the 70B shape and 8 layers 673, now 168).
__device__ __forceinline__ void credit_pieces(const DecArgs &a, const Meta &mt,
                                              const CreditArgs &cr, int blk, int nblk) {
  __shared__ float s_oth[kCreditWaves][kWave], s_own[kCreditWaves][kWave];
  __shared__ float s_m[kCreditTile], s_wo[kCreditTile], s_wn[kCreditTile];
  __shared__ float2 s_ml[kCreditThreads];
  const Tree &t = a.t;
  const Pool &pl = a.pl;
  const int G = pl.G, Hkv = pl.Hkv;
  const int Hq = Hkv * G;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (blk == 0) {
    const unsigned long long per = (unsigned long long)cr.S * Hq;
    for (int e = threadIdx.x; e < a.n_leaves * MAXD; e += blockDim.x) {
      const int b = e / MAXD, d = e % MAXD;
      const int dl = a.ldepth[b];
      if (d < dl || (d == dl && cr.self_window))
        atomicAdd(reinterpret_cast<unsigned long long *>(cr.rows_seen) +
                      a.lanc[(int64_t)b * MAXD + d],
                  per);
    }
  }
  const float *z0 = a.rest + mt.z;
  const int64_t z_slab = (int64_t)mt.z_total * 64;
  const int per = cr.U * Hkv;
  // (in a vector register: the fused step below reads one scalar register, M)
  float c2 = a.sl2;
  asm volatile("" : "+v"(c2));
  const bool listed = mt.n_pieces > 0;
  const int32_t *piece_unit = reinterpret_cast<const int32_t *>(a.rest) + mt.pieces;
  const int per_unit = mt.chunk / kWave;
  const int64_t n_w = listed ? mt.n_pieces : (int64_t)mt.n_units * per_unit;
  constexpr int kLast = kCreditWaves - 1;
  for (int64_t w = blk; w < n_w; w += nblk) {
    const int u = listed ? piece_unit[w] : (int)((unsigned)w / (unsigned)per_unit);
    const Unit un = units_of(a)[u];
    const int piece = (int)(w - (listed ? (int64_t)un.piece0 : (int64_t)u * per_unit)) * kWave;
    // (uniform over the workgroup) a chunk is credited once, by its first unit
    if (un.first != u || piece >= un.n_slots) continue;
    const int node = un.node;
    const int slot = un.s_begin + piece + lane;
    const bool key_ok = piece + lane < un.n_slots;
    const int R = un.R;
    const int loff = un.loff;
    const int n = R * per;
    const int zstride = (un.n_slots + 63) & ~63;
    // threads per triple: as many as there are for the unit's triples, but no
    // more than the longest list of partials
    int tpt = 1;
    while (2 * tpt <= kLseThreads && 2 * tpt * n <= kCreditThreads && tpt < mt.max_np) tpt *= 2;
    const int tri = min(n, kCreditTile);
    const int tj = (int)threadIdx.x / tri, ti = (int)threadIdx.x - tj * tri;
    // the leaf of this thread's first table entry, read before the logits so
    // that waiting for it does not wait for them
    const int b_first = tj < tpt ? a.leaf_list[loff + ti % R / G] : 0;
    // logit rows hold whole 64-slot pieces, so the lane's slot is in bounds for
    // every lane; lanes past the node's count are masked after the load
    const float *zb = z0 + (int64_t)un.zbase * 64 + piece + lane;
    float cur[kCreditBatch];
    Triple it(wv, R);
    credit_load(cur, zb, it, R, per, z_slab, zstride);
    // the last wave fetches the lane's token and its A entry meanwhile; each
    // token has one owner, so A is read before the sums
    int64_t tok = 0;
    float a_old = 0.f;
    bool own_ok = false;
    if (wv == kLast && key_ok) {
      const int page = t.page_table[t.page_off[node] + slot / pl.P];
      const int pos = pl.slot_pos[(int64_t)page * pl.P + slot % pl.P];
      tok = t.tok_off[node] + pos;
      a_old = cr.A[tok];
      // own rows (the node is the row's leaf) are credited only on earlier
      // keys in the self-window mode
      own_ok = cr.self_window && pos < t.n_full[node] - 1;
    }
    float oth = 0.f, own = 0.f;
    int e0 = wv;
    for (int t0 = 0; t0 < n; t0 += kCreditTile) {
      const int nt = min(kCreditTile, n - t0);
      const int e = t0 + ti;
      const int r = e % R, zg = e / R;
      const int z = zg / Hkv, g = zg - z * Hkv;
      const bool mine = tj < tpt && ti < nt;
      int b = 0;
      if (mine) {
        b = t0 == 0 ? b_first : a.leaf_list[loff + r / G];
        s_ml[tj * tri + ti] = chain_ml(a, mt, b, cr.slice[z], g, r % G, tj, tpt);
      }
      __syncthreads();
      if (mine && tj == 0) {
        float2 v = s_ml[ti];
        for (int j = 1; j < tpt; ++j) v = ml_merge(v, s_ml[j * tri + ti]);
        // (M + log2 L in one number would round M's distance to the logits)
        const float m = v.y > 0.f ? (float)cr.mult[z] / v.y : 0.f;
        const bool own_row = a.leaves[b] == node;
        s_m[ti] = v.y > 0.f ? v.x : __builtin_inff();
        s_wo[ti] = own_row ? 0.f : m;
        s_wn[ti] = own_row ? m : 0.f;
      } else if ((int)threadIdx.x >= nt) {
        s_m[threadIdx.x] = s_wo[threadIdx.x] = s_wn[threadIdx.x] = 0.f;
      }
      __syncthreads();
      for (; e0 < t0 + nt; e0 += kCreditWaves * kCreditBatch) {
        float nxt[kCreditBatch];
        const bool more = e0 + kCreditWaves * kCreditBatch < n;
        if (more) credit_load(nxt, zb, it, R, per, z_slab, zstride);
        static_assert(kCreditBatch == 16, "one row of lanes per batch");
        const int i = e0 - t0 + kCreditWaves * (lane & (kCreditBatch - 1));
        const float mx = s_m[i], wo = s_wo[i], wn = s_wn[i];
#pragma unroll
        for (int u = 0; u < kCreditBatch; ++u) {
          const float p = key_ok ? __builtin_amdgcn_exp2f(
                                       __builtin_fmaf(cur[u], c2, -lane_value(mx, u)))
                                 : 0.f;
          oth = __builtin_fmaf(lane_value(wo, u), p, oth);
          own = __builtin_fmaf(lane_value(wn, u), p, own);
        }
        if (more) {
#pragma unroll
          for (int u = 0; u < kCreditBatch; ++u) cur[u] = nxt[u];
        }
      }
      __syncthreads();                        // the tables are reused by the next tile
    }
    s_oth[wv][lane] = oth;
    s_own[wv][lane] = own;
    __syncthreads();
    if (wv == kLast && key_ok) {
      float tot = 0.f;
#pragma unroll
      for (int v = 0; v < kCreditWaves; ++v) tot += s_oth[v][lane];
      if (own_ok) {
#pragma unroll
        for (int v = 0; v < kCreditWaves; ++v) tot += s_own[v][lane];
      }
      cr.A[tok] = a_old + tot;
    }
    __syncthreads();                          // the sums are reused by the next piece
  }
}

template <int D>
__global__ __launch_bounds__(256) void decode_merge(DecArgs a, void *out, int out_dtype,
                                                    float *lse_out) {
  // (loaded together with the status word)
  const Meta mt = *a.meta;
  if (status_failed(a.status)) return;
  merge_rows<D>(a, mt, out, out_dtype, lse_out, blockIdx.x, gridDim.x);
}

// scored calls: the first credit_blocks workgroups credit (their chain of
// loads is the longer one, so they are dispatched first), the rest merge
template <int D>
__global__ __launch_bounds__(kCreditThreads) void decode_merge_credit(DecArgs a, CreditArgs cr,
                                                                      void *out, int out_dtype,
                                                                      float *lse_out,
                                                                      int credit_blocks) {
  // (loaded together with the status word)
  const Meta mt = *a.meta;
  if (status_failed(a.status)) return;
  if ((int)blockIdx.x < credit_blocks) {
    credit_pieces(a, mt, cr, blockIdx.x, credit_blocks);
    return;
  }
  merge_rows<D>(a, mt, out, out_dtype, lse_out, blockIdx.x - credit_blocks,
                gridDim.x - credit_blocks);
}

template <class T, int D>
void launch_decode_kernels(const arbor_geom_t *geom, const DecArgs &a, void *out, int out_dtype,
                           float *lse_out, const CreditArgs *cr, hipStream_t stream) {
  const int grid = 2048;
  timing_begin(geom, ARBOR_KERNEL_DECODE_ATTN, stream);
  if (cr)
    hipLaunchKernelGGL((decode_attn<T, D, true>), dim3(grid), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_attn<T, D, false>), dim3(grid), dim3(256), 0, stream, a);
  timing_end(geom, ARBOR_KERNEL_DECODE_ATTN, stream);
  const int64_t mw = (int64_t)a.n_leaves * a.Lr * a.pl.Hkv * a.pl.G;
  if (!cr) {
    const int mgrid = (int)((mw + 3) / 4 < 8192 ? (mw + 3) / 4 : 8192);
    hipLaunchKernelGGL((decode_merge<D>), dim3(mgrid), dim3(256), 0, stream, a, out, out_dtype,
                       lse_out);
    return;
  }
  // credit workgroups stride over the 64-slot pieces of the plan's chunks (at
  // most half the chip's wave slots, so that the merge workgroups start beside
  // them); merge workgroups hold kCreditWaves rows each
  const int cgrid = kCreditGroups;
  const int64_t mb = (mw + kCreditWaves - 1) / kCreditWaves;
  const int mgrid = (int)(mb < 2048 ? mb : 2048);
  timing_begin(geom, ARBOR_KERNEL_DECODE_CREDIT, stream);
  hipLaunchKernelGGL((decode_merge_credit<D>), dim3(cgrid + mgrid), dim3(kCreditThreads), 0,
                     stream, a, *cr, out, out_dtype, lse_out, cgrid);
  timing_end(geom, ARBOR_KERNEL_DECODE_CREDIT, stream);
}

}  // namespace

size_t decode_workspace(const arbor_geom_t *g, const arbor_sizes_t *sz) {
  const size_t nl = (size_t)(sz->max_leaves > 0 ? sz->max_leaves : 1);
  const size_t planes = (size_t)sz->max_layers * g->num_kv_heads;
  const size_t ctx = (size_t)sz->max_context, G = (size_t)g->q_per_kv;
  // chunks along one chain (at most one ragged chunk per chain node), at the
  // smallest chunk size; rows and units over all leaves
  const size_t per_leaf = ctx / kMinChunk + MAXD + 1;
  const size_t rows = nl * per_leaf * G;
  size_t b = 16 * 256;
  b += nl * (MAXD * (4 * (3 + kPlanEnts) + 8) + 12);
  b += (nl * per_leaf + rows / 16 + nl) * sizeof(Unit) + 2 * nl * per_leaf * 4;
  // partial rows over all planes.  A chunk size C below the longest is taken while
  // 2 C is more than an even share, or than four fifths of it, so the whole
  // chunks hold at most 5/2 kWaves64 units of 16 rows, beside one ragged chunk for
  // each row of each chain node.
  const int longest = g->dtype == ARBOR_BF16 ? kMaxChunk : kChunks[kFirstChunkF32];
  const size_t least = nl * (ctx / longest + MAXD + 1) * G * planes;
  const size_t most =
      std::min(rows * planes, (size_t)kWaves64 * 40 + nl * (MAXD + 1) * G * planes);
  b += std::max(least, most) * (g->head_dim + 2) * 4;
  // logits of the credited slice layers (scored decode)
  b += nl * G * (ctx + 64 * (MAXD + 1)) * (size_t)(sz->n_slice > 0 ? sz->n_slice : 0) *
           g->num_kv_heads * 4 +
       64;
  return b;
}

int launch_decode(const arbor_geom_t *geom, const arbor_tree_t *tree, const arbor_pool_t *pool,
                  const int32_t *leaves, int32_t n_leaves, int32_t layer_begin, int32_t layer_end,
                  const void *q, void *out, int32_t out_dtype, float *lse_out, float softmax_scale,
                  const arbor_decode_credit_t *credit, int32_t *status, void *workspace,
                  size_t workspace_bytes, hipStream_t stream) {
  Tree t = make_tree(tree);
  Pool pl = make_pool(geom, pool);
  if (t.V <= 0 || n_leaves <= 0 || layer_end <= layer_begin) return ARBOR_OK;
  DecArgs a;
  a.t = t;
  a.pl = pl;
  a.leaves = leaves;
  a.n_leaves = n_leaves;
  a.l0 = layer_begin;
  a.Lr = layer_end - layer_begin;
  a.q = q;
  const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)geom->head_dim);
  a.sl2 = scale * kLog2e;
  a.status = status;
  const bool small = t.V <= kPlanLds, few = n_leaves <= kPlanLeaves;
  const size_t ne = (size_t)n_leaves * MAXD;
  Carve cv(workspace, workspace_bytes);
  a.meta = cv.take<Meta>(1);
  a.leaf_list = cv.take<int32_t>(ne);
  a.lanc = cv.take<int32_t>(ne);
  a.ldepth = cv.take<int32_t>(n_leaves);
  a.leaf_np = cv.take<int32_t>(n_leaves);
  a.ent_p0 = cv.take<int32_t>(ne);
  PlanEnt ent{};
  if (!few) {
    int32_t **f[kPlanEnts] = {&ent.up, &ent.kept, &ent.rbase, &ent.loff, &ent.np, &ent.u0, &ent.z0};
    for (int e = 0; e < kPlanEnts; ++e) *f[e] = cv.take<int32_t>(ne);
    ent.place = cv.take<uint64_t>(ne);
  }
  if (!cv.ok) return ARBOR_EWORKSPACE;
  CreditArgs cr{};
  if (credit) {
    cr.S = credit->n_slice;
    for (int e = 0; e < credit->n_slice; ++e) {
      const int lr = credit->slice_layers[e] - layer_begin;
      int u = 0;
      while (u < cr.U && cr.slice[u] != lr) ++u;
      if (u == cr.U) cr.slice[cr.U++] = lr;
      ++cr.mult[u];
    }
    cr.self_window = credit->self_window;
    cr.A = credit->A;
    cr.rows_seen = credit->rows_seen;
  }
  a.zS = credit ? cr.U : 0;
  for (int e = 0; e < 8; ++e) a.zlr[e] = credit && e < cr.U ? cr.slice[e] : -1;
  a.rest = reinterpret_cast<float *>(cv.rest());
  a.rest_cap = (int64_t)(cv.remaining() / 4);
  // one thread per node (whose parent links go to LDS) and per chain entry: a
  // small tree takes a smaller workgroup, whose barriers are cheaper
  const int64_t plan_need = std::max<int64_t>(small ? t.V : 0, (int64_t)n_leaves * 8);
  const int plan_threads = (int)std::min<int64_t>(1024, (plan_need + kWave - 1) / kWave * kWave);
#define ARBOR_PLAN_LAUNCH(S, F)                                                              \
  hipLaunchKernelGGL((decode_plan<S, F, decltype(waves)::value, decltype(first)::value>),    \
                     dim3(1), dim3(plan_threads), 0, stream, a, ent)
  auto plan = [&](auto waves, auto first) {
    if (small && few) ARBOR_PLAN_LAUNCH(true, true);
    else if (small) ARBOR_PLAN_LAUNCH(true, false);
    else if (few) ARBOR_PLAN_LAUNCH(false, true);
    else ARBOR_PLAN_LAUNCH(false, false);
  };
  using std::integral_constant;
  if (geom->dtype != ARBOR_BF16)
    plan(integral_constant<int, kWaves>{}, integral_constant<int, kFirstChunkF32>{});
  else if (geom->head_dim == 64)
    plan(integral_constant<int, kWaves64>{}, integral_constant<int, 0>{});
  else
    plan(integral_constant<int, kWaves>{}, integral_constant<int, 0>{});
#undef ARBOR_PLAN_LAUNCH
  const CreditArgs *crp = credit ? &cr : nullptr;
  if (geom->dtype == ARBOR_BF16) {
    if (geom->head_dim == 128)
      launch_decode_kernels<__bf16, 128>(geom, a, out, out_dtype, lse_out, crp, stream);
    else
      launch_decode_kernels<__bf16, 64>(geom, a, out, out_dtype, lse_out, crp, stream);
  } else {
    if (geom->head_dim == 128)
      launch_decode_kernels<float, 128>(geom, a, out, out_dtype, lse_out, crp, stream);
    else
      launch_decode_kernels<float, 64>(geom, a, out, out_dtype, lse_out, crp, stream);
  }
  return hip_ok(hipGetLastError());
}

}  // namespace arbor
