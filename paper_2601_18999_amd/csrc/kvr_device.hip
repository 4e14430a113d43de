// kvr_device.hip - gfx950 kernels of the batched KV-cache routing / eviction
// simulator.
//
// One workgroup owns one replica for a whole batch and walks the batch's
// queries in order (the simulation is sequential within a replica, Sec. 3.1:
// the state after query j-1 decides query j).  Per query, in two phases
// separated by workgroup barriers:
//   * phase A, wave 0: the LBGR score of every worker from its load,
//     residual model and h_ij, the longest cached prefix of the query (Sec.
//     3.2 "Cache Matching"); the argmin (lowest index on ties) and the commit
//     on the routed worker (Algorithm 2 routing thread, Eq. LBGR-score, Eq. 2
//     with the estimate), or a baseline router of Sec. 5.  The other waves
//     stage the next query in LDS.
//   * phase B, wave 0: the insertion into the routed worker's cache with RLT
//     (Algorithm 1: marks along the path, phase resets, a uniform draw over
//     the unmarked leaf tokens U for every token loaded into a full cache;
//     Eq. 3: no other cache changes) or L-LRU, then that worker's h for the
//     next query.  The other waves: the draw words of the insertion and the
//     new leaf's rank; completions and load decay at the next arrival, one
//     lane per worker (Algorithm 2, update and decay threads; Sec. 4.2); the
//     next query's h on every other worker, walking each compressed radix
//     tree from the point where the previous match on it can be resumed.

// The cache of a worker is a compressed radix tree: a node holds an edge of
// `len` tokens; its leaf token (when it has no children) is the last one.
// U is kept as an ordered list of candidate leaf nodes in lexicographic
// order of their root paths: rebuilt from the ordered list of all leaves
// when a phase starts, shortened when a candidate's leaf token is marked,
// and updated in place when an eviction exposes the parent as a new leaf
// (the parent inherits the rank of the leaf it replaces).  A draw takes
// index floor(r * |U| / 2^64), r = word 0 of Philox4x64-10 with key
// (seed, replica) and counter (query index, worker, draw index, 0).
//
// With cached responses a query is a complete token path q_j || a_j (Sec.
// 3.2 "Cache Matching and Arrival Model"): the match, the scores and the
// commit see the prompt q_j, the insertion takes the whole path.
//
// Floating point: double, left-to-right sums, built with -ffp-contract=off so
// no multiply-add is fused; the same expressions in the same order as the
// definition, so results are bit-identical to any IEEE implementation that
// evaluates them in that order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "kvr_trail.h"

namespace kvr {

// ---------------------------------------------------------------- kernels

// Paths recorded in LDS: entries of worker i at [i * kPathMax, (i+1) * kPathMax)
// of the node, start and end arrays, then one count per worker.
struct PathArea {
  int32_t* base;
  uint32_t W;
  __device__ PathRef of(uint32_t i) const {
    PathRef p;
    p.node = base + (size_t)i * kPathMax;
    p.start = base + (size_t)(W + i) * kPathMax;
    p.end = base + (size_t)(2 * W + i) * kPathMax;
    p.cnt = base + (size_t)3 * W * kPathMax + i;
    return p;
  }
};

__device__ __forceinline__ void count_matched(const Ptrs& P, int32_t h, int32_t* hslot) {
  if (lane_id() == 0) {
    *hslot = h;
    P.hdr->matched_tokens += (uint64_t)h;
  }
}

// Words in front of and behind each query buffer: staging writes whole 16-byte
// blocks of the stream, up to three words outside the query.
constexpr uint32_t kQueryPad = 4;
__host__ __device__ constexpr uint32_t query_words(uint32_t maxL) { return ((maxL + 3u) & ~3u) + 2u * kQueryPad; }

// Stage q_next[0, Ln) (threads t0, t0 + stride, ...) and fold each thread's
// first position where it differs from q_cur into *ell (LDS minimum), so
// that once all have staged, *ell = LCP(q_cur, q_next).  The stream is read in
// aligned 16-byte blocks, kU per thread in flight; threads past the end read
// the last block again.
template <int kU>
__device__ __forceinline__ void stage_query(const int32_t* tokens, uint64_t n0, int32_t Ln, int32_t* qn,
                                            const int32_t* qc, int32_t Lc, uint32_t wave0, uint32_t stride,
                                            int32_t* ell) {
  const int32_t* p = tokens + n0;
  const int32_t lead = (int32_t)((reinterpret_cast<uintptr_t>(p) >> 2) & 3u);
  const int4* base = reinterpret_cast<const int4*>(p - lead);
  const uint32_t nb = (uint32_t)((lead + Ln + 3) >> 2);
  int32_t m = Lc < Ln ? Lc : Ln;
  for (uint32_t b = wave0; b < nb; b += kU * stride) {
    int4 v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t k = b + (uint32_t)u * stride + (uint32_t)lane_id();
      if (u == 0 || b + (uint32_t)u * stride < nb) v[u] = base[k < nb ? k : nb - 1u];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (u != 0 && b + (uint32_t)u * stride >= nb) break;
      const uint32_t k = b + (uint32_t)u * stride + (uint32_t)lane_id();
      const int32_t x0 = (int32_t)(k < nb ? k : nb - 1u) * 4 - lead;
      const int32_t t4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
      const bool end = x0 < 0 || x0 + 4 > Ln;  // the first or last block
#pragma unroll
      for (int c = 3; c >= 0; --c) {
        const int32_t x = x0 + c;
        qn[x] = t4[c];
        if (qc[x] != t4[c] && x < m && (!end || x >= 0)) m = x;
      }
    }
  }
  // minimum over the wave (m >= 0), then one LDS atomic per wave
  m = (int32_t)wave_min_u64((uint64_t)(uint32_t)m);
  if (lane_id() == 0) atomicMin(ell, m);
}

// Lowest index among the minimal scores (lanes >= W hold +inf): the same
// result as scanning i = 0..W-1 with a strict less-than.  -0.0 is folded
// into +0.0 (they compare equal); a NaN makes the scan itself decide.
__device__ __forceinline__ uint32_t wave_argmin(double eh, uint32_t W, const double* eh_sh) {
  if (__ballot(eh != eh)) {
    uint32_t best = 0;
    for (uint32_t i = 1; i < W; ++i)
      if (eh_sh[i] < eh_sh[best]) best = i;
    return best;
  }
  const double z = eh + 0.0;
  uint64_t b = (uint64_t)__double_as_longlong(z);
  b = (b >> 63) ? ~b : (b | 0x8000000000000000ull);  // order-preserving key
  const uint64_t mn = wave_min_u64(b);
  return (uint32_t)first_lane(__ballot(b == mn));
}

// Lowest lane among the minima of v (lanes >= W excluded).
__device__ __forceinline__ uint32_t wave_argmin_u32(uint32_t v, uint32_t W) {
  const uint64_t key = (uint32_t)lane_id() < W ? (((uint64_t)v << 32) | (uint32_t)lane_id()) : ~0ull;
  return (uint32_t)(wave_min_u64(key) & 0xffffffffull);
}

// The baseline routers of Sec. 5.  One lane per worker.  In line: a call costs
// 0.2 to 0.4 us a step (27 workers, random router: 7.17 ms a simulation of 732
// queries instead of 6.91); the learned router of the pipelined kernel has a
// form without them.
__device__ __forceinline__ uint32_t route_baseline(int32_t router, uint64_t jg, uint64_t seed, uint32_t r, uint32_t W,
                                                uint32_t load, uint32_t size, uint32_t h, int32_t Lq, uint32_t abs,
                                                double rel, double threshold) {
  if (uni(router) == KVR_ROUTE_RANDOM) return (uint32_t)__umul64hi(philox_word0(jg, 0ull, 0ull, 1ull, seed, r), (uint64_t)W);
  if (uni(router) == KVR_ROUTE_ROUND_ROBIN) return (uint32_t)(jg % W);
  const uint32_t lo = wave_argmin_u32(load, W);
  const uint32_t hi = wave_argmin_u32(~load, W);
  const uint32_t hmax = wave_argmin_u32(~h, W);
  const uint32_t small = wave_argmin_u32(size, W);
  const uint32_t lmin = (uint32_t)__builtin_amdgcn_readlane((int)load, (int)lo);
  const uint32_t lmax = (uint32_t)__builtin_amdgcn_readlane((int)load, (int)hi);
  const int32_t hbest = __builtin_amdgcn_readlane((int)h, (int)hmax);
  if (lmax - lmin > abs && (double)lmax > rel * (double)lmin) return lo;
  if ((double)hbest > threshold * (double)Lq) return hmax;
  return small;
}

// The routed worker of query k (global index j0 + k): the LBGR argmin, or
// one of the baseline routers.  Wave-uniform; one lane per worker.
__device__ __forceinline__ uint32_t route_choice(const StepArgs& a, uint32_t r, uint32_t k, uint32_t W, double eh,
                                                 const int32_t* hrow, int32_t Lq, const double* eh_sh,
                                                 const RouteView& v) {
  if (a.C.router == KVR_ROUTE_LBGR) return wave_argmin(eh, W, eh_sh);
  const uint32_t h = (uint32_t)lane_id() < W ? (uint32_t)hrow[lane_id()] : 0u;
  return uni(route_baseline(a.C.router, a.j0 + k, a.C.seed, r, W, v.pend_count, v.size, h, Lq,
                            (uint32_t)a.C.ca_balance_abs, a.C.ca_balance_rel, a.C.ca_cache_threshold));
}

// Record a match length without counting it (the cache's own match when
// the router scores with its own tree).
__device__ __forceinline__ void store_h(int32_t h, int32_t* hslot) {
  if (lane_id() == 0) *hslot = h;
}

// The next query's h on the workers other than `best`, taken one item at a
// time from an LDS counter, so a wave that drew long matches takes fewer.
// Items 0..W-1 are the
// caches; with the approximate router, items W..2W-1 are the router's trees.
// The index is wave-uniform (lane 0's atomic, read back from lane 0) and the
// loop is bounded by the number of items.
__device__ __forceinline__ void take_matches(const StepArgs& a, uint32_t r, uint32_t W, uint32_t best,
                                             const int32_t* qn, int32_t Lnq, int32_t ell, const int32_t* h_cur,
                                             int32_t* h_next, const int32_t* g_cur, int32_t* g_next,
                                             const PathArea& paths, const PathArea& rpaths, bool rtree,
                                             uint32_t* next) {
  const uint32_t items = rtree ? 2u * W : W;
  for (uint32_t it = 0; it < items; ++it) {
    uint32_t got = 0;
    if (lane_id() == 0) got = atomicAdd(next, 1u);
    const uint32_t i = (uint32_t)__builtin_amdgcn_readlane((int)got, 0);
    if (i >= items) break;
    const uint32_t w = i < W ? i : i - W;
    if (w == best) continue;
    Ptrs Pw = worker_ptrs(a.ws, a.L, r, w);
    if (i < W) {
      const int32_t h = match_incremental(Pw, Pw.hdr->arena_sel, qn, Lnq, h_cur[w], ell, paths.of(w));
      if (rtree)
        store_h(h, &h_next[w]);
      else
        count_matched(Pw, h, &h_next[w]);
    } else {
      Ptrs Pr = router_ptrs(a.ws, a.L, r, w);
      count_matched(Pw, match_incremental(Pr, Pr.hdr->arena_sel, qn, Lnq, g_cur[w], ell, rpaths.of(w)), &g_next[w]);
    }
  }
}

// First device-side error of the run (check id and values for the message),
// then the sticky status bits; the workgroup stops after the next barrier.
__device__ __forceinline__ void report_error(GlobalHdr* g, uint32_t r, uint64_t jg, uint32_t err, const int64_t* dbg,
                                             uint32_t* abort_flag) {
  if (lane_id() != 0 || !err) return;
  if (atomicCAS(&g->err_taken, 0u, 1u) == 0u) {
    g->err_check = (uint32_t)dbg[0];
    g->err_replica = r;
    g->err_query = jg;
    g->err_val[0] = dbg[1];
    g->err_val[1] = dbg[2];
    g->err_val[2] = dbg[3];
  }
  atomicOr(&g->status, err);
  *abort_flag = 1;
}

// Approximate router: the router adds prompt q[0, Lq) to its tree of the
// routed worker (L-LRU; hr = the router's match of it), then matches the
// next prompt there, from the path just inserted.  Returns KVR_DEV_* bits.
__device__ __forceinline__ uint32_t router_admit(const StepArgs& a, uint32_t r, uint64_t jg, uint32_t best,
                                                 const int32_t* qs, int32_t Lq, int32_t hr, bool has_next,
                                                 const int32_t* qn, int32_t Lnq, int32_t ell, const PathArea& rpaths,
                                                 int32_t* g_next, int64_t* dbg) {
  Ptrs Pr = router_ptrs(a.ws, a.L, r, best);
  InsertArgs ia;
  ia.seed = a.C.seed;
  ia.jg = jg;
  ia.worker = best;
  ia.replica = r;
  ia.B = a.L.RB;
  ia.rn = 0;
  ia.rw = nullptr;
  ia.prog = nullptr;
  ia.nprog = 0;
  ia.round = 1;
  ia.rank = nullptr;
  ia.rank_ready = nullptr;
  const uint32_t err = lru_insert(Pr, ia, qs, Lq, hr, rpaths.of(best), dbg);
  if (!err && has_next)
    count_matched(worker_ptrs(a.ws, a.L, r, best),
                  match_incremental(Pr, Pr.hdr->arena_sel, qn, Lnq, Lq, ell, rpaths.of(best)), g_next);
  return err;
}

// Is the batch to be routed at all?  Called by a whole workgroup before it
// changes anything, with bad, a word of its LDS, at 0; after the next barrier
// `batch_ok` says.  The run must not have failed (a later part of a batch: this
// replica must have routed the parts before it) and, with a.check, the batch
// must be valid: lengths (with cached responses, a prompt of at least one token
// before the response) and arrival order, which every wave looks at for
// itself, and only then the tokens.  Every workgroup reads the same batch and
// its replica's own last arrival, so all come to the same verdict.
constexpr uint32_t kRunFailed = 1u << 31;
__device__ __forceinline__ void check_batch(const StepArgs& a, GlobalHdr* g, const ReplicaHdr* rh, int64_t tprev,
                                            uint32_t* bad) {
  if (threadIdx.x == 0 && (a.part ? rh->failed || rh->queries != a.j0 : __atomic_load_n(&g->status, __ATOMIC_RELAXED)))
    atomicOr(bad, kRunFailed);
  if (!a.check) return;
  uint32_t bits = 0;
  for (uint32_t j = (uint32_t)lane_id(); j < a.n; j += KVR_WAVE) {
    const uint64_t o0 = a.offsets[j], o1 = a.offsets[j + 1];
    if (o1 <= o0 || o1 - o0 > a.L.maxL) bits |= KVR_DEV_BAD_LENGTH;
    if (a.C.cache_responses && o1 - o0 <= (uint64_t)query_out_len(a.out_len, j)) bits |= KVR_DEV_BAD_LENGTH;
    if (a.arrival[j] < (j == 0 ? tprev : a.arrival[j - 1])) bits |= KVR_DEV_BAD_ARRIVAL;
  }
  if (__ballot(bits != 0u)) {
    if (bits) atomicOr(bad, bits);
    return;
  }
  const int32_t* p = a.tokens + a.offsets[0];
  const uint32_t m = (uint32_t)(a.offsets[a.n] - a.offsets[0]);
  constexpr int kU = 4;  // loads in flight per thread
  int32_t low = 0;
  for (uint32_t x = threadIdx.x; x < m; x += kU * blockDim.x) {
    int32_t v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t k = x + (uint32_t)u * blockDim.x;
      v[u] = p[k < m ? k : m - 1u];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) low |= v[u];
  }
  if (low < 0) atomicOr(bad, (uint32_t)KVR_DEV_BAD_TOKEN);
}

__device__ __forceinline__ bool batch_ok(GlobalHdr* g, uint32_t bad) {
  if (!bad) return true;
  if (threadIdx.x == 0 && !(bad & kRunFailed)) atomicOr(&g->status, bad);
  return false;
}

// One workgroup per replica walks the batch in order.  A worker's tree
// changes only when a query is routed to it, so while wave 0 inserts query k
// into the routed worker the other waves compute the draw words of that
// insertion, the completions and decay at the next arrival, and the next
// query's h on every other worker.  Matches are incremental: each worker
// keeps the path of its last match, and the next query follows it up to
// the longest common prefix of the two queries.  The routed worker's h for
// the next query is completed from the path of the inserted query.  With
// the approximate router every worker has two trees, the cache and the
// router's, each matched incrementally; the router's tree of the routed
// worker is updated by a helper wave.  The approximate router (RT) and
// continuous batching (BA) are template switches, so the kernel without
// them carries none of their registers.
template <bool RT, bool BA, bool PT>
__global__ void __launch_bounds__(512) step_kernel(StepArgs a) {
  // dynamic LDS: two query buffers (max_query_tokens entries each), the high
  // halves of the draw words, the match paths (the caches', then the router
  // trees'), then the staged candidate list
  extern __shared__ __align__(16) int32_t smem[];
  const uint32_t W = a.L.W;
  constexpr bool rtree = RT;
  const uint32_t qstride = query_words(a.L.maxL);
  uint32_t* rw = reinterpret_cast<uint32_t*>(smem + 2 * qstride);
  PathArea paths, rpaths;
  paths.base = reinterpret_cast<int32_t*>(rw + a.rcap);
  paths.W = W;
  rpaths.base = paths.base + (size_t)W * (3 * kPathMax + 1);
  rpaths.W = W;
  UStage ustage;
  {
    int32_t* ub = paths.base + (size_t)(rtree ? 2 : 1) * W * (3 * kPathMax + 1);
    ustage.node = ub;
    ustage.len = ub + a.ucap;
    ustage.top = ub + 2 * a.ucap;
    ustage.par = ub + 3 * a.ucap;
    ustage.cap = a.ucap;
  }
  __shared__ int32_t h_sh[2][kMaxWorkers];  // h of the current and of the next query (the caches)
  __shared__ int32_t g_sh[2][kMaxWorkers];  // the same on the router's trees (approximate router)
  __shared__ double eh_sh[kMaxWorkers];
  __shared__ int32_t ell_sh[2];  // LCP(q_k, q_k+1) in slot k & 1
  __shared__ int32_t best_sh;
  __shared__ int32_t hins_sh;  // cached length of the inserted path (>= h of the prompt)
  __shared__ uint32_t abort_sh;
  __shared__ uint32_t nev_sh;
  __shared__ uint32_t prog_sh[16];  // rounds of draw words each drawing wave has written
  __shared__ uint32_t next_sh;    // next item for the helpers' matches
  __shared__ int32_t rank_sh;     // the new leaf's rank, from the last helper wave
  __shared__ uint32_t rank_ready_sh;
  // the hits the router scores with: the caches' own, or its trees'
  int32_t(*est)[kMaxWorkers] = rtree ? g_sh : h_sh;

  const uint32_t r = blockIdx.x;
  const bool resp = a.C.cache_responses != 0;
  const int lane = lane_id();
  const uint32_t wave = threadIdx.x / KVR_WAVE;
  const uint32_t nwaves = blockDim.x / KVR_WAVE;
  const uint32_t nh = nwaves - 1;  // helper waves
  GlobalHdr* g = reinterpret_cast<GlobalHdr*>(a.ws + a.L.off_global);
  ReplicaHdr* rh = reinterpret_cast<ReplicaHdr*>(a.ws + a.L.off_rhdr) + r;

  if (threadIdx.x == 0) {
    abort_sh = 0;
    ell_sh[0] = 0x7fffffff;
  }
  __syncthreads();
  check_batch(a, g, rh, rh->tprev, &abort_sh);
  __syncthreads();
  if (!batch_ok(g, abort_sh)) return;
  // the replica's route digest and query count, kept by the routing wave
  uint64_t chain = 0, routed = 0;
  if (wave == 0) {
    chain = rh->route_digest;
    routed = rh->queries;
  }
  PhaseClock clk;
  clock_start<PT>(&clk);

  // query 0: stage its path; completions and decay at its arrival; full
  // matches of its prompt
  {
    const uint64_t o0 = a.offsets[0];
    const int32_t L0 = (int32_t)(a.offsets[1] - o0);
    const int32_t L0q = resp ? L0 - query_out_len(a.out_len, 0) : L0;
    for (int32_t x = (int32_t)threadIdx.x; x < L0; x += (int32_t)blockDim.x) smem[kQueryPad + x] = a.tokens[o0 + x];
    if (wave == 0 && (uint32_t)lane < W)
      complete_and_decay(a.C, worker_ptrs(a.ws, a.L, r, (uint32_t)lane), a.arrival[0], rh->tprev);
    __syncthreads();
    for (uint32_t i = wave; i < W; i += nwaves) {
      Ptrs P = worker_ptrs(a.ws, a.L, r, i);
      const int32_t h = match_lcp(P, P.hdr->arena_sel, smem + kQueryPad, L0q, paths.of(i));
      if (rtree) {
        store_h(h, &h_sh[0][i]);
        Ptrs Pr = router_ptrs(a.ws, a.L, r, i);
        count_matched(P, match_lcp(Pr, Pr.hdr->arena_sel, smem + kQueryPad, L0q, rpaths.of(i)), &g_sh[0][i]);
      } else {
        count_matched(P, h, &h_sh[0][i]);
      }
    }
  }
  for (uint32_t k = 0; k < a.n; ++k) {
    const uint64_t o0 = a.offsets[k];
    const int32_t Lp = (int32_t)(a.offsets[k + 1] - o0);  // the path inserted
    const int64_t t = a.arrival[k];
    const int32_t olen = query_out_len(a.out_len, k);
    const int32_t Lq = resp ? Lp - olen : Lp;  // the prompt
    const uint32_t cur = k & 1u;
    int32_t* qs = smem + cur * qstride + kQueryPad;
    int32_t* qn = smem + (cur ^ 1u) * qstride + kQueryPad;
    const bool has_next = k + 1 < a.n;
    int32_t Ln = 0, Lnq = 0;  // path and prompt of the next query
    uint64_t n0 = 0;
    if (has_next) {
      n0 = a.offsets[k + 1];
      Ln = (int32_t)(a.offsets[k + 2] - n0);
      Lnq = resp ? Ln - query_out_len(a.out_len, k + 1) : Ln;
    }
    __syncthreads();

    // ---- phase A.  Wave 0: scores, argmin, commit.  Helpers: stage the
    // next query.
    if (wave == 0) {
      double eh = __builtin_huge_val(), ch = 0.0;
      RouteView v{};
      if ((uint32_t)lane < W) {
        v = load_view(worker_ptrs(a.ws, a.L, r, (uint32_t)lane).hdr);
        eh = lbgr_score(a.C, v, est[cur][lane], Lq, &ch);
        eh_sh[lane] = eh;
      }
      __builtin_amdgcn_wave_barrier();
      const uint32_t best = route_choice(a, r, k, W, eh, est[cur], Lq, eh_sh, v);
      Ptrs P = worker_ptrs(a.ws, a.L, r, best);
      const int32_t hb = h_sh[cur][best];  // the worker's true hit
      // a cached prompt may continue into a cached response: the insertion
      // needs the cached length of the whole path, continued from the
      // prompt's recorded match
      int32_t hins = hb;
      if (resp && hb == Lq && Lp > Lq) hins = match_incremental(P, P.hdr->arena_sel, qs, Lp, Lq, Lq, paths.of(best));
      // the routed worker's lane commits from the header fields it holds
      uint32_t cerr = 0;
      if ((uint32_t)lane == best) cerr = commit_route(a.C, P, v, ch, hb, est[cur][best], Lq, t, olen);
      const uint32_t err = (uint32_t)__builtin_amdgcn_readlane((int)cerr, (int)best);
      const uint32_t size = (uint32_t)__builtin_amdgcn_readlane((int)v.size, (int)best);
      if ((uint32_t)lane < 16u) prog_sh[lane] = 0u;
      if (lane == 0) {
        best_sh = (int32_t)best;
        hins_sh = hins;
        next_sh = 0;
        rank_ready_sh = 0;
        const uint64_t orow = (uint64_t)r * a.rows + k;
        if (a.route) a.route[orow] = (int32_t)best;
        if (a.hits) a.hits[orow] = hb;
        if (!err) {
          chain = route_chain(chain, a.j0 + k, best, hb);
          routed += 1;
        }
        // draws this insertion will take: one per token loaded into a full cache
        const uint32_t nload = (uint32_t)(Lp - hins);
        const uint32_t nfree = a.L.B - size;
        nev_sh = err ? 0u : (nload > nfree ? nload - nfree : 0u);
        if (err) {
          atomicOr(&g->status, err);
          abort_sh = 1;
        }
      }
      if (a.all_hits && (uint32_t)lane < W)
        a.all_hits[((uint64_t)r * a.rows + k) * W + (uint32_t)lane] = est[cur][lane];
      if (nh == 0 && has_next) stage_query<8>(a.tokens, n0, Ln, qn, qs, Lp, 0u, KVR_WAVE, &ell_sh[cur]);
    } else if (has_next) {
      stage_query<8>(a.tokens, n0, Ln, qn, qs, Lp, uni(wave - 1u) * KVR_WAVE, blockDim.x - KVR_WAVE, &ell_sh[cur]);
    }
    if (wave == 0) clock_mark<PT>(&clk, KVR_PHASE_ROUTE);
    __syncthreads();
    if (wave == 0) clock_mark<PT>(&clk, KVR_PHASE_STAGE_WAIT);
    if (abort_sh) break;
    const uint32_t best = (uint32_t)best_sh;
    const uint32_t nev = nev_sh;
    // draw words: RLT only
    const uint32_t rn = a.C.evict == KVR_EVICT_RLT ? (nev < a.rcap ? nev : a.rcap) : 0u;
    const int32_t hins = hins_sh;
    // LCP of the two paths, then of what the next match needs: the next
    // prompt against the inserted path (the routed cache) or against this
    // prompt (every other cache, whose recorded match is of this prompt, and
    // every router tree, which holds prompts only)
    const int32_t ellp = ell_sh[cur];
    const int32_t ell_r = ellp < Lnq ? ellp : Lnq;
    const int32_t ell = ell_r < Lq ? ell_r : Lq;
    const uint64_t jg = a.j0 + k;
    // with two or more helpers, the last one ranks the new leaf of an RLT
    // insertion while the others compute its draw words
    const bool ranker = nh >= 2 && a.C.evict == KVR_EVICT_RLT && hins < Lp;

    // ---- phase B.  Wave 0: the insertion, then the routed worker's h for
    // the next query.  Helpers: the insertion's draw words first, then
    // completions and decay at the next arrival (and the router's tree of
    // the routed worker), and the next query's h on the other workers.
    if (wave == 0) {
      if (nh == 0)
        for (uint32_t d = (uint32_t)lane; d < rn; d += KVR_WAVE)
          rw[d] = (uint32_t)(philox_word0(jg, best, d, 0ull, a.C.seed, r) >> 32);
      Ptrs P = worker_ptrs(a.ws, a.L, r, best);
      InsertArgs ia;
      ia.seed = a.C.seed;
      ia.jg = jg;
      ia.worker = best;
      ia.replica = r;
      ia.B = a.L.B;
      ia.rn = rn;
      ia.rw = rw;
      ia.prog = nh && rn ? prog_sh : nullptr;
      ia.nprog = ranker ? nh - 1u : nh;
      ia.round = 2u * (blockDim.x - (ranker ? 2u : 1u) * KVR_WAVE);
      ia.rank = ranker ? &rank_sh : nullptr;
      ia.rank_ready = &rank_ready_sh;
      int64_t dbg[4] = {0, 0, 0, 0};
      uint32_t err = a.C.evict == KVR_EVICT_RLT ? rlt_insert<PT>(P, ia, qs, Lp, hins, ustage, paths.of(best), dbg, &clk)
                                                : lru_insert(P, ia, qs, Lp, hins, paths.of(best), dbg);
      // continuous batching: the path joins the worker's running batch
      if (BA && !err && P.beta > 1) err = batch_admit(P, paths.of(best), qs, Lp, dbg);
      report_error(g, r, jg, err, dbg, &abort_sh);
      // the routed worker's h for the next query, from the path of the
      // query just inserted (all of it is cached now: the old h is Lp)
      if (has_next && !err) {
        Ptrs Pb = worker_ptrs(a.ws, a.L, r, best);
        const int32_t h = match_incremental(Pb, Pb.hdr->arena_sel, qn, Lnq, Lp, ell_r, paths.of(best));
        if (rtree)
          store_h(h, &h_sh[cur ^ 1u][best]);
        else
          count_matched(Pb, h, &h_sh[cur ^ 1u][best]);
      }
      clock_mark<PT>(&clk, KVR_PHASE_MATCH);
      if (nh == 0 && !err) {
        if (has_next) {
          if ((uint32_t)lane < W)
            complete_and_decay(a.C, worker_ptrs(a.ws, a.L, r, (uint32_t)lane), a.arrival[k + 1], t);
          if (lane == 0) ell_sh[cur ^ 1u] = 0x7fffffff;
        }
        if (rtree) {
          int64_t rdbg[4] = {0, 0, 0, 0};
          const uint32_t rerr = router_admit(a, r, jg, best, qs, Lq, g_sh[cur][best], has_next, qn, Lnq, ell, rpaths,
                                             &g_sh[cur ^ 1u][best], rdbg);
          report_error(g, r, jg, rerr, rdbg, &abort_sh);
        }
        if (has_next)
          take_matches(a, r, W, best, qn, Lnq, ell, h_sh[cur], h_sh[cur ^ 1u], g_sh[cur], g_sh[cur ^ 1u], paths,
                       rpaths, rtree, &next_sh);
      }
    } else {
      if (ranker && wave == nwaves - 1) {
        // the last helper ranks the insertion's new leaf
        rank_for_insertion(worker_ptrs(a.ws, a.L, r, best), paths.of(best), qs, hins, &rank_sh, &rank_ready_sh);
      } else {
        // the others compute the draw words, a round of 2*nd words at a
        // time (two independent words per lane), and publish each round
        // they complete
        const uint32_t nd = blockDim.x - (ranker ? 2u : 1u) * KVR_WAVE;
        uint32_t rounds = 0;
        for (uint32_t base = 0; base < rn; base += 2u * nd) {
          const uint32_t d0 = base + threadIdx.x - KVR_WAVE, d1 = d0 + nd;
          const uint64_t w0 = philox_word0(jg, best, d0, 0ull, a.C.seed, r);
          const uint64_t w1 = philox_word0(jg, best, d1, 0ull, a.C.seed, r);
          if (d0 < rn) rw[d0] = (uint32_t)(w0 >> 32);
          if (d1 < rn) rw[d1] = (uint32_t)(w1 >> 32);
          ++rounds;
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
          if (lane == 0)
            __hip_atomic_store(&prog_sh[wave - 1u], rounds, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
      if (wave == 1) {
        if (has_next) {
          if ((uint32_t)lane < W)
            complete_and_decay(a.C, worker_ptrs(a.ws, a.L, r, (uint32_t)lane), a.arrival[k + 1], t);
          if (lane == 0) ell_sh[cur ^ 1u] = 0x7fffffff;
        }
        if (rtree) {
          int64_t rdbg[4] = {0, 0, 0, 0};
          const uint32_t rerr = router_admit(a, r, jg, best, qs, Lq, g_sh[cur][best], has_next, qn, Lnq, ell, rpaths,
                                             &g_sh[cur ^ 1u][best], rdbg);
          report_error(g, r, jg, rerr, rdbg, &abort_sh);
        }
      }
      if (has_next)
        take_matches(a, r, W, best, qn, Lnq, ell, h_sh[cur], h_sh[cur ^ 1u], g_sh[cur], g_sh[cur ^ 1u], paths,
                     rpaths, rtree, &next_sh);
    }
    __syncthreads();
    if (wave == 0) clock_mark<PT>(&clk, KVR_PHASE_JOIN);
    if (abort_sh) break;
  }
  if (threadIdx.x == 0) {
    if constexpr (PT)
      for (int p = 0; p < KVR_PHASES; ++p) rh->phase_ticks[p] += clk.acc[p];
    rh->route_digest = chain;
    rh->queries = routed;
    if (!abort_sh && a.n > 0) {
      rh->tprev = a.arrival[a.n - 1];
      if (r == 0) g->last_arrival = a.arrival[a.n - 1];
    }
  }
}

// ---------------------------------------------------------------- pipelined step kernel
//
// RLT with prompts only, LBGR or a baseline router, no approximate router
// and single-query processing (the benchmark's path).  A step is bound by
// latency: the route of a query needs its h on every worker, and the routed
// worker's h needs the insertion of the query before it.  So everything that
// need not lie on that chain is taken off it:
//   * the next queries are matched on every worker before this one is routed.  A
//     worker's tree changes only when a query is routed to it, so only the
//     routed worker's match is looked at again after the load, and it follows
//     from the one before;
//   * the routing wave only scores, commits and plans the insertion; the load of
//     the new leaf, the marks, the leaf list and the evictions follow on an
//     evicting wave, several insertions (of different workers) at a time;
//   * LBGR state, tree state and query data live in LDS for the launch.
// What is left on the chain is about 2.5 us of one wave's instructions a query
// (route 1.4, owning the worker and planning 0.6; a wave issues an instruction
// every 5 cycles or so, and raising its priority changes nothing), the wait for
// matches that are late (1.5 to 3.5) and for a worker that is routed to twice in
// a row (2 to 3).
//
// Waves: 0 routes, 1..NE insert and evict, the rest are helpers: they stage
// queries, match, compute draw words, rank new leaves and apply completions and
// decay, whichever is due first.
//
// The order of a worker's matches and insertions: kvr_trail.h.  Waves
// synchronise through the workers' state words and the counters below (LDS,
// workgroup scope, release/acquire); every wait is bounded and sees the stop
// flag, so an error ends every loop.

struct PipeFlags {
  uint32_t routed;   // queries routed
  uint32_t fronts;   // leaves loaded: the buffer of query fronts - 1 is free
  uint32_t staged;   // helpers done staging, over all queries
  uint32_t decayed;  // arrivals whose completions and decay are applied
  uint32_t handed;   // insertions handed to the evicting waves
  uint32_t ticket;   // insertions they have taken
  uint32_t end;      // every query is routed and handed
  uint32_t stop;     // an error stopped the replica
  uint32_t bad;      // the verdict on the batch
  uint32_t err, err_query, err_check;  // the first error
  uint32_t pad[4];
  int64_t err_val[3];
  int64_t pad2;
};
constexpr int kFlagWords = 16;  // the counters, a word per lane of a row
static_assert(sizeof(PipeFlags) == 4 * kFlagWords + 32, "counters, then the error's values");

// 16-byte compare loads in flight per lane in the pipelined kernel's matches
#ifndef KVR_PIPE_MATCH_UNROLL
#define KVR_PIPE_MATCH_UNROLL 8
#endif
constexpr int kPipeMatchUnroll = KVR_PIPE_MATCH_UNROLL;
constexpr uint32_t kSpinLimit = 1u << 24;
// Waves per workgroup: 12 (three per SIMD, 150 registers a lane; against 8,
// multi-turn 51.0 ms a simulation instead of 55.3, the paper's groups in
// round-robin order 67.9 instead of 77.8, the rest within 3%), and 16 for
// replicas of many workers, whose matches of one query keep more helpers busy
// (128 registers and some scratch), and whose lanes take the matches that are zero
// (take_zero_match; in the 12-wave form it costs 1 to 2%).  16 against 12 waves, in
// ms a simulation of long prompts, of conversations and of short prompts:
//   12 workers: 15.83 / 15.60, 15.77 / 15.44, 12.10 / 12.06
//   16 workers: 14.46 / 14.50, 15.33 / 15.18, 11.72 / 12.13
//   18 workers: 13.45 / 13.83, 15.10 / 15.09, 11.81 / 12.63
//   22 workers: 12.26 / 13.49, 14.86 / 15.44, 10.72 / 13.00
// and the line lies between 16 and 18.
#ifndef KVR_PIPE_WAVES
#define KVR_PIPE_WAVES 12
#endif
#ifndef KVR_PIPE_WAVES_WIDE
#define KVR_PIPE_WAVES_WIDE 16
#endif
#ifndef KVR_PIPE_WIDE_WORKERS
#define KVR_PIPE_WIDE_WORKERS 17
#endif
constexpr uint32_t kPipeWaves = KVR_PIPE_WAVES;
constexpr uint32_t kPipeWavesWide = KVR_PIPE_WAVES_WIDE;
constexpr uint32_t kPipeWideWorkers = KVR_PIPE_WIDE_WORKERS;
// Evicting waves.  One insertion takes 9 to 13 us of a wave, a step 8 to 10 us,
// so one wave would be the step's bound.  A third (one helper fewer) gains 2 to
// 3% on the drift and two-level workloads and loses 5% on the long-prompt one,
// 2% on the smallest and on the ensemble.
#ifndef KVR_PIPE_EVICTORS
#define KVR_PIPE_EVICTORS 2
#endif
constexpr uint32_t kPipeEvictors = KVR_PIPE_EVICTORS;

__device__ __forceinline__ uint32_t ld_acq(const uint32_t* p) {
  return uni(__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
}

// Publish v (lane 0, after every lane's earlier writes).
__device__ __forceinline__ void st_rel(uint32_t* p, uint32_t v) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane_id() == 0) __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void add_rel(uint32_t* p, uint32_t v) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane_id() == 0) __hip_atomic_fetch_add(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Stop the replica: its first error is noted in LDS (bits, the query, check id,
// values), to be reported when the workgroup ends, and every wave's waits end.
__device__ __forceinline__ void pipe_stop(PipeFlags* f, uint32_t k, uint32_t err, const int64_t* dbg) {
  if (lane_id() == 0) {
    if (atomicCAS(&f->err, 0u, err) == 0u) {
      f->err_query = k;
      f->err_check = (uint32_t)dbg[0];
      f->err_val[0] = dbg[1];
      f->err_val[1] = dbg[2];
      f->err_val[2] = dbg[3];
    }
    __hip_atomic_store(&f->stop, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// One poll of a wait: false once the replica was stopped; a wait that has
// run out stops it (check id 90 + site, an internal error).
__device__ __forceinline__ bool pipe_poll(uint32_t& spins, PipeFlags* f, uint32_t k, int site) {
  if (ld_acq(&f->stop)) return false;
  if (++spins > kSpinLimit) {
    const int64_t dbg[4] = {90 + site, (int64_t)f->routed, (int64_t)f->handed, (int64_t)f->staged};
    pipe_stop(f, k, KVR_DEV_INTERNAL, dbg);
    return false;
  }
  __builtin_amdgcn_s_sleep(1);
  return true;
}

// Wait until *p >= target.  False when the replica was stopped.
__device__ __forceinline__ bool pipe_wait(const uint32_t* p, uint32_t target, PipeFlags* f, uint32_t k, int site) {
  uint32_t spins = 0;
  while (ld_acq(p) < target)
    if (!pipe_poll(spins, f, k, site)) return false;
  return true;
}

// The leaf list and the worker state of an evicting wave: the new leaf's rank
// comes from a helper, and is waited for only when something needs the list;
// the state goes back to LDS.
struct PipeHook {
  bool todo;
  PipeJob job;
  const uint32_t* ready;  // rank_ready of the job's slot
  const int32_t* rank;
  uint32_t* state;        // the worker's state words
  const uint32_t* stop;
  __device__ __forceinline__ void before_list(const Ptrs& P, St& s) {
    if (!todo) return;
    todo = false;
    const uint32_t want = ((job.k + 1u) << 2) | 3u;
    uint32_t spins = 0;
    while (ld_acq(ready) != want) {
      if (ld_acq(stop) || ++spins > kSpinLimit) {
        KVR_FAIL_CHECK(s, 5, job.k, job.worker, spins);
        return;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    const int32_t pos = uni(*rank);
    if (pos < 0 || (uint32_t)pos > s.nleaves) {
      KVR_FAIL_CHECK(s, 4, pos, s.nleaves, job.a);
      return;
    }
    if (job.replace) {
      if (lane_id() == 0) P.leaf[pos] = job.l;
    } else {
      arr_insert(P.leaf, s.nleaves, (uint32_t)pos, job.l, false);
      s.nleaves += 1;
    }
    wave_mem_sync();
  }
  __device__ __forceinline__ void keep(const Ptrs&, const St& s) { store_st_lds(state, s); }
  // the ring and the rounds' counts go to later insertions once this one ends: a
  // wave that still draws would write into theirs
  static constexpr bool kWordsMustCome = true;
  __device__ __forceinline__ void words_late(St& s) { KVR_FAIL_CHECK(s, 7, job.k, job.worker, job.rn); }
};

// NW waves, NE of them evicting; kLbgr: the learned router only (the baselines'
// code would lengthen every step).
template <bool PT, uint32_t NW, uint32_t NE, bool kLbgr>
__global__ void __launch_bounds__(64 * NW) step_kernel_pipe(StepArgs a) {
  constexpr uint32_t nh = NW - 1u - NE;  // helper waves
  // half of the helpers compute draw words, from the second on (the first
  // applies completions and decay)
  constexpr uint32_t ndraw = nh / 2u;
  static_assert(nh >= 2u && ndraw >= 1u && ndraw < nh && ndraw <= 16u, "too few or too many waves");
  constexpr uint32_t nd = ndraw * KVR_WAVE;  // drawing threads
  extern __shared__ __align__(16) int32_t smem[];
  const uint32_t W = a.L.W;
  // dynamic LDS: nbuf query buffers, the LBGR state, the workers' tree states,
  // the trails of nbuf queries, the root filters, the ring of draw words, the
  // evicting waves' staged candidates
  const uint32_t qwords = query_words(a.L.maxL);
  LbgrLds lb;
  lb.W = W;
  lb.P = reinterpret_cast<double*>(smem + a.nbuf * qwords);
  lb.theta = lb.P + W;
  lb.Wb = reinterpret_cast<int64_t*>(lb.theta + 4 * W);
  lb.done_at = lb.Wb + W;
  lb.head = reinterpret_cast<uint32_t*>(lb.done_at + W);
  lb.count = lb.head + W;
  lb.size = lb.count + W;
  uint32_t* st_sh = lb.size + W;                   // state words
  uint32_t* tree_sh = st_sh + W;                   // kStWords per worker
  int32_t* trail_sh = reinterpret_cast<int32_t*>(tree_sh + kStWords * W);  // [nbuf][W][kTrailWords]
  uint32_t* rootf = reinterpret_cast<uint32_t*>(trail_sh + a.nbuf * kTrailWords * W);
  uint32_t* ring = rootf + kRootFilterWords * W;   // rcap draw words
  int32_t* stage_base = reinterpret_cast<int32_t*>(ring + a.rcap);

  __shared__ PipeFlags f;
  __shared__ int32_t h_sh[kMaxBuf][kMaxWorkers];  // h of q_k in slot query_slot(k)
  __shared__ double eh_sh[kMaxWorkers];
  __shared__ int32_t ell_sh[8];             // LCP(q_k, q_k+1) in slot k & 7
  __shared__ int32_t len_sh[8], olen_sh[8]; // length and output length of q_k
  __shared__ int64_t arr_sh[8];             // its arrival
  __shared__ PipeJob job_sh[kJobs];         // insertion k in slot k % kJobs
  __shared__ uint32_t jdone_sh[kJobs];      // k + 1 once it is finished
  __shared__ uint32_t owner_sh[kMaxWorkers]; // the insertion that owns a worker
  __shared__ uint32_t best_sh[kJobs], r0_sh[kJobs];
  __shared__ int32_t hit_sh[kJobs];         // h of the routed worker
  __shared__ uint64_t rn_sh[kJobs];         // ((k + 1) << 32) | its precomputed draw words
  __shared__ uint32_t prog_sh[kJobs][16];   // rounds of them each drawing wave has written
  __shared__ int32_t rank_sh[kJobs];        // the new leaf's rank
  __shared__ uint32_t rank_ready_sh[kJobs]; // 0, or ((k + 1) << 2) | 1 wanted, 2 being computed, 3 there
  __shared__ unsigned long long eticks_sh[KVR_PHASES];  // evicting and helper waves' ticks
  // matched tokens per worker over the batch (added to the headers at the end)
  __shared__ unsigned long long mtok_sh[kMaxWorkers];

  const uint32_t r = blockIdx.x;
  const int lane = lane_id();
  const uint32_t wave = uni((uint32_t)(threadIdx.x / KVR_WAVE));
  GlobalHdr* g = reinterpret_cast<GlobalHdr*>(a.ws + a.L.off_global);
  ReplicaHdr* rh = reinterpret_cast<ReplicaHdr*>(a.ws + a.L.off_rhdr) + r;

  // ---- the launch's state: nothing here depends on anything else but the
  // root filters on the tree state, so its loads are under way together; what
  // changes the replica's state (the decay to the first arrival with the rest)
  // comes after the verdict on the batch
  const int64_t tprev = rh->tprev;
  if (threadIdx.x < kFlagWords) reinterpret_cast<uint32_t*>(&f)[threadIdx.x] = 0u;
  if (threadIdx.x < KVR_PHASES) eticks_sh[threadIdx.x] = 0ull;
  if (threadIdx.x < kMaxWorkers) {
    mtok_sh[threadIdx.x] = 0ull;
    for (uint32_t b = 0; b < kMaxBuf; ++b) h_sh[b][threadIdx.x] = 0;
  }
  if (threadIdx.x < 8u) ell_sh[threadIdx.x] = 0x7fffffff;
  if (threadIdx.x < kJobs) {
    jdone_sh[threadIdx.x] = 0u;
    rank_ready_sh[threadIdx.x] = 0u;
    rn_sh[threadIdx.x] = 0ull;
  }
  for (uint32_t x = threadIdx.x; x < W * kRootFilterWords; x += 64 * NW) rootf[x] = 0u;
  __syncthreads();
  for (uint32_t x = threadIdx.x; x < W * (uint32_t)kStWords; x += 64 * NW) {
    const uint32_t* hw = reinterpret_cast<const uint32_t*>(worker_ptrs(a.ws, a.L, r, x / kStWords).hdr);
    tree_sh[x] = hw[x % kStWords];
  }
  if (threadIdx.x < W) {
    const uint32_t w = threadIdx.x;
    const Ptrs P = worker_ptrs(a.ws, a.L, r, w);
    const WorkerHdr* h = P.hdr;
    lb.P[w] = h->P;
    for (int k = 0; k < 4; ++k) lb.theta[k * W + w] = h->theta[k];
    lb.Wb[w] = h->Wb;
    lb.head[w] = h->pend_head;
    lb.count[w] = h->pend_count;
    lb.done_at[w] = h->pend_count > 0 ? P.pend[h->pend_head].t_done : kNever;
    lb.size[w] = h->size;
    st_sh[w] = 0u;
    for (uint32_t b = 0; b < a.nbuf; ++b) trail_sh[(b * W + w) * kTrailWords] = 0;
  }
  // the root filters: the first token of every child of every root
  for (uint32_t i = wave; i < W; i += NW) {
    const Ptrs P = worker_ptrs(a.ws, a.L, r, i);
    const NodeRec root = load_node(P.nodes, 0);
    const int32_t* ar = arena_of(P, uni(P.hdr->arena_sel));
    for (int32_t c = lane; c < root.nchild; c += KVR_WAVE) rf_add(rootf + i * kRootFilterWords, ar[root.coff + 2 * c]);
  }
  check_batch(a, g, rh, tprev, &f.bad);
  __syncthreads();
  if (!batch_ok(g, f.bad)) return;

  const uint32_t n = a.n;
  PhaseClock clk;
  clock_start<PT>(&clk);
  // progress of this wave: the next query to route (routing wave); the
  // insertion taken (evicting waves); the next query to stage and to serve once
  // routed (helpers)
  uint32_t kq = 0, sN = 0, dN = 0;
  uint32_t spins = 0, seen = 0;
  uint32_t ring_head = 0;
  bool ticket = false;
  uint64_t chain = 0, routed_total = 0;
  int64_t tick_prev = 0;
  if (wave == NE + 1u) {
    chain = rh->route_digest;
    routed_total = rh->queries;
    // completions and decay at the first arrival
    const int64_t t = a.arrival[0], tick = t / a.C.dt_us;
    if ((uint32_t)lane < W) {
      const Ptrs P = worker_ptrs(a.ws, a.L, r, (uint32_t)lane);
      decay_lds(a.C, lb, (uint32_t)lane, P.hdr, P.pend, P.PC, t, tprev, tick, tprev / a.C.dt_us);
    }
    tick_prev = tick;
    st_rel(&f.decayed, 1u);
  }
  MatchArea ma;
  ma.W = W;
  ma.nbuf = a.nbuf;
  ma.q = smem + kQueryPad;
  ma.qstride = qwords;
  ma.len = len_sh;
  ma.ell = ell_sh;
  ma.h = &h_sh[0][0];
  ma.trail = trail_sh;
  ma.tree = tree_sh;
  ma.rootf = rootf;
  ma.state = st_sh;
  ma.owner = owner_sh;
  ma.jobs = job_sh;
  ma.mtok = mtok_sh;

  if (wave == 0) {
    for (;;) {
      // -------------------------------------------------------- routing wave
      // h of q_kq on every worker
      if (kq == n) break;
      // the match to take this round, if any: query mm on worker mw, whose state
      // was msv
      uint32_t msv = 0, mm = 0, mw = 0;
      const uint32_t sv =
          (uint32_t)lane < W ? __hip_atomic_load(&st_sh[lane], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
      const uint64_t open = __ballot((uint32_t)lane < W && (sv >> kCountShift) == (kq & kCountMask));
      if (open) {
        const uint64_t can = __ballot((uint32_t)lane < W && can_match(sv, kq, owner_sh[lane], a.nbuf));
        if (can && ld_acq(&f.staged) >= (kq + 1u) * nh) {
          mw = (uint32_t)first_lane(can);
          mm = kq;
          msv = (uint32_t)__builtin_amdgcn_readlane((int)sv, (int)mw);
          if (!claim_match(&st_sh[mw], msv)) continue;
        } else {
          if (!pipe_poll(spins, &f, kq, 0)) break;
          continue;
        }
      } else {
        {
          // ---- route q_kq
          spins = 0;
          const uint32_t k = kq, cur = query_slot(k, a.nbuf), nxt = query_slot(k + 1u, a.nbuf), slot = k % kJobs;
          const uint64_t jg = a.j0 + k;
          clock_mark<PT>(&clk, KVR_PHASE_JOIN);
          if (!pipe_wait(&f.decayed, k + 1u, &f, k, 1)) break;
          clock_mark<PT>(&clk, KVR_PHASE_STAGE_WAIT);
          // the slot of insertion k - kJobs is reused
          if (k >= kJobs) {
            bool ok = true;
            while (ld_acq(&jdone_sh[slot]) != k - kJobs + 1u)
              if (!(ok = pipe_poll(spins, &f, k, 2))) break;
            if (!ok) break;
          }
          clock_mark<PT>(&clk, KVR_PHASE_EVICTOR_WAIT);
          const int32_t Lp = uni(len_sh[k & 7u]);
          double eh = __builtin_huge_val(), ch = 0.0;
          RouteView v{};
          if ((uint32_t)lane < W) {
            v.P = lb.P[lane];
            for (int x = 0; x < 4; ++x) v.theta[x] = lb.theta[x * W + lane];
            v.Wb = lb.Wb[lane];
            v.pend_head = lb.head[lane];
            v.pend_count = lb.count[lane];
            v.size = lb.size[lane];
            eh = lbgr_score(a.C, v, h_sh[cur][lane], Lp, &ch);
            eh_sh[lane] = eh;
          }
          __builtin_amdgcn_wave_barrier();
          const uint32_t best =
              uni(kLbgr ? wave_argmin(eh, W, eh_sh) : route_choice(a, r, k, W, eh, h_sh[cur], Lp, eh_sh, v));
          const Ptrs P = worker_ptrs(a.ws, a.L, r, best);
          const int32_t hb = uni(h_sh[cur][best]);
          const uint32_t size = (uint32_t)__builtin_amdgcn_readlane((int)v.size, (int)best);
          const uint32_t nload = (uint32_t)(Lp - hb);
          const uint32_t nfree = a.L.B - size;
          const uint32_t nev = nload > nfree ? nload - nfree : 0u;
          // commit: the routed worker's lane
          uint32_t err0 = 0;
          if ((uint32_t)lane == best) {
            err0 = commit_lds(a.C, P, lb, best, v, ch, hb, Lp, arr_sh[k & 7u], olen_sh[k & 7u]);
            lb.size[best] = size + nload - nev;
          }
          err0 = (uint32_t)__builtin_amdgcn_readlane((int)err0, (int)best);
          // draw words: a stretch of the ring that no unfinished insertion uses
          uint32_t rn = nev, r0 = 0;
          if (nev > 0) {
            uint32_t jd = 0, j0 = 0, jn = 0;
            // lane i looks at insertion k - kJobs + 1 + i (the oldest first)
            const uint32_t ji = k - kJobs + 1u + (uint32_t)lane;
            bool used = false;
            if ((uint32_t)lane < kJobs - 1u && ji < k) {
              const uint32_t js = ji % kJobs;
              jd = jdone_sh[js];
              j0 = r0_sh[js];
              jn = (uint32_t)rn_sh[js];
              used = jd != ji + 1u && jn > 0u;
            }
            const uint64_t um = __ballot(used);
            uint32_t room = a.rcap;
            if (um) {
              const uint32_t tail = (uint32_t)__builtin_amdgcn_readlane((int)j0, first_lane(um));
              if (ring_head > tail) {
                const uint32_t after = a.rcap - ring_head;
                r0 = after >= nev || after >= tail ? ring_head : 0u;
                room = r0 ? after : tail;
              } else {
                r0 = ring_head;
                room = tail - ring_head;
              }
            }
            rn = nev < room ? nev : room;
            ring_head = r0 + rn;
          }
          if ((uint32_t)lane < 16u) prog_sh[slot][lane] = 0u;
          if (lane == 0) {
            best_sh[slot] = best;
            hit_sh[slot] = hb;
            r0_sh[slot] = r0;
            rn_sh[slot] = ((uint64_t)(k + 1u) << 32) | rn;
            rank_ready_sh[slot] = 0u;
          }
          if (err0) {
            if (lane == 0) {
              const uint64_t orow = (uint64_t)r * a.rows + k;
              if (a.route) a.route[orow] = (int32_t)best;
              if (a.hits) a.hits[orow] = hb;
            }
            const int64_t dbg[4] = {0, 0, 0, 0};
            pipe_stop(&f, k, err0, dbg);
            break;
          }
          st_rel(&f.routed, k + 1u);
          clock_mark<PT>(&clk, KVR_PHASE_ROUTE);
          // ---- own the worker: its earlier insertion first finishes, and so does
          // a match of a later query on it
          uint32_t pre;  // matches of later queries taken on it
          {
            bool ok = true;
            uint32_t sb = 0;
            for (;;) {
              if (lane == 0) sb = __hip_atomic_fetch_or(&st_sh[best], kOwner, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
              sb = uni(sb);
              if (!(sb & kOwner)) break;
              if (!(ok = pipe_poll(spins, &f, k, 3))) break;
            }
            if (!ok) break;
            while (sb & kReader) {
              sb = ld_acq(&st_sh[best]);
              if ((sb & kReader) && !(ok = pipe_poll(spins, &f, k, 4))) break;
            }
            if (!ok) break;
            pre = ((sb >> kCountShift) - (k + 1u)) & kCountMask;
            spins = 0;
          }
          clock_mark<PT>(&clk, KVR_PHASE_EVICTOR_WAIT);
          // ---- plan the insertion, and what it makes of the match of q_k+1 taken
          // before it; those of later ones are taken again
          PipeJob job;
          plan_insertion(job, tree_sh + best * kStWords, a.L.B, a.L.maxL, hb, Lp);
          job.pre = -1;
          uint32_t state = 0;
          if (pre) {
            const int32_t h_pre = uni(h_sh[nxt][best]);
            bool stays;
            const int32_t h = match_before_load(P.nodes, job, h_pre, uni(ell_sh[k & 7u]),
                                                trail_sh + (nxt * W + best) * kTrailWords, stays);
            int32_t diff = (stays ? h : 0) - h_pre;
            for (uint32_t x = 2; x <= pre; ++x) {
              diff -= uni(h_sh[query_slot(k + x, a.nbuf)][best]);
              state -= 1u << kCountShift;
            }
            if (lane == 0) {
              h_sh[nxt][best] = h;
              atomicAdd(&mtok_sh[best], (unsigned long long)(int64_t)diff);
            }
            if (stays)
              job.pre = h_pre;
            else  // put off: one match fewer, to be taken after the evictions
              state += kDeferred - (1u << kCountShift);
          }
          if (lane == 0) {
            PipeJob& j = job_sh[slot];
            j.k = k;
            j.worker = best;
            j.h = job.h;
            j.L = job.L;
            j.nfree = job.nfree;
            j.nev = job.nev;
            j.rn = rn;
            j.r0 = r0;
            j.calm = job.calm;
            j.phase = job.phase;
            j.pre = job.pre;
            owner_sh[best] = k;
            h_sh[cur][best] = Lp;  // all of q_k is cached here from the load on
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
          if (lane == 0) {
            __hip_atomic_fetch_add(&st_sh[best], state, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(&f.handed, k + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          kq = k + 1u;
          clock_mark<PT>(&clk, KVR_PHASE_LOAD);
          continue;
        }
      }
      take_match<kPipeMatchUnroll>(ma, worker_ptrs(a.ws, a.L, r, mw), mm, mw, msv);
      clock_mark<PT>(&clk, KVR_PHASE_MATCH);
    }
  } else if (wave <= NE) {
    // ---------------------------------------------------------- evicting wave
    for (;;) {
      if (!ticket) {
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(&f.ticket, 1u);
        kq = uni(t);
        ticket = true;
        spins = 0;
      }
      const uint32_t ended = ld_acq(&f.end);  // (read first: set once every insertion has been handed)
      if (ld_acq(&f.handed) <= kq) {  // wait for that insertion
        if (ended) break;
        const uint32_t now = ld_acq(&f.routed);
        if (now != seen) {
          seen = now;
          spins = 0;
        }
        if (!pipe_poll(spins, &f, kq, 6)) break;
        continue;
      }
      clock_mark<PT>(&clk, KVR_PHASE_E_IDLE);
      ticket = false;
      {
        // ---- the load of the new leaf
        PipeHook hook;
        const uint32_t slot = kq % kJobs;
        PipeJob job = load_job(&job_sh[slot]);
        const Ptrs P = worker_ptrs(a.ws, a.L, r, job.worker);
        uint32_t* tree = tree_sh + job.worker * kStWords;
        const uint32_t buf = query_slot(kq, a.nbuf);
        int32_t* tr = trail_sh + (buf * W + job.worker) * kTrailWords;
        EvictJob ej;
        ej.s = load_st_lds(tree);
        int32_t split;
        const uint32_t lerr = load_leaf(P, ej.s, tree, a.L.B, smem + buf * qwords + kQueryPad, tr, job, split);
        store_st_lds(tree, ej.s);
        if (lerr) {
          const int64_t dbg[4] = {ej.s.dbg_check, ej.s.dbg_val[0], ej.s.dbg_val[1], ej.s.dbg_val[2]};
          pipe_stop(&f, kq, lerr, dbg);
          break;
        }
        if (job.pre >= 0)
          trail_after_load(job, split, job.pre, uni(ell_sh[kq & 7u]), tr,
                           trail_sh + (query_slot(kq + 1u, a.nbuf) * W + job.worker) * kTrailWords);
        // loads are published in order: q_kq's buffer is free then, and so is the
        // slot of the LCP of the query that will be staged there with the one
        // before it
        spins = 0;
        {
          bool ok = true;
          while (ld_acq(&f.fronts) != kq)
            if (!(ok = pipe_poll(spins, &f, kq, 7))) break;
          if (!ok) break;
        }
        if (lane == 0) {
          // a new child of the root: its first token joins the root filter
          if (job.h == 0) rf_add(rootf + job.worker * kRootFilterWords, job.tok);
          PipeJob& j = job_sh[slot];
          j.l = job.l;
          j.a = job.a;
          j.tok = job.tok;
          j.replace = job.replace;
          j.marked = job.marked;
          ell_sh[(kq + a.nbuf - 1u) & 7u] = 0x7fffffff;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane == 0) {
          __hip_atomic_fetch_or(&st_sh[job.worker], kLoaded, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (job.h < job.L)
            __hip_atomic_store(&rank_ready_sh[slot], ((kq + 1u) << 2) | 1u, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_store(&f.fronts, kq + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        clock_mark<PT>(&clk, KVR_PHASE_E_MATCH);
        // ---- marks, leaf list, evictions
        if (!job.marked) mark_cached(P, ej.s, a.L.B, job, tr);
        // the trail has been read
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane == 0) atomicOr(&st_sh[job.worker], kMarked);
        clock_mark<PT>(&clk, KVR_PHASE_E_FINISH);
        hook.todo = job.h < job.L;
        hook.job = job;
        hook.ready = &rank_ready_sh[slot];
        hook.rank = &rank_sh[slot];
        hook.state = tree;
        hook.stop = &f.stop;
        ej.ia.seed = a.C.seed;
        ej.ia.jg = a.j0 + kq;
        ej.ia.worker = job.worker;
        ej.ia.replica = r;
        ej.ia.B = a.L.B;
        ej.ia.rn = job.rn;
        ej.ia.rw = ring + job.r0;
        ej.ia.prog = job.rn ? prog_sh[slot] : nullptr;
        ej.ia.nprog = ndraw;
        ej.ia.round = 2u * nd;
        ej.ia.rank = nullptr;
        ej.ia.rank_ready = nullptr;
        ej.h = job.h;
        ej.L = job.L;
        ej.l = job.l;
        ej.nfree = job.nfree;
        ej.nev = job.nev;
        ej.c0 = ej.s.cnt;
        ej.reset_at = job.h < job.L && ej.c0 + (uint32_t)(job.L - job.h) >= a.L.B + 1u ? job.h + (int32_t)(a.L.B - ej.c0)
                                                                                       : -1;
        ej.worker = job.worker;
        ej.final_size = 0;
        UStage us;
        us.node = stage_base + (wave - 1u) * 4u * a.ucap;
        us.len = us.node + a.ucap;
        us.top = us.len + a.ucap;
        us.par = us.top + a.ucap;
        us.cap = a.ucap;
        int64_t dbg[4] = {0, 0, 0, 0};
        uint32_t err = ej.s.err;
        if (err) {
          dbg[0] = ej.s.dbg_check;
          dbg[1] = ej.s.dbg_val[0];
          dbg[2] = ej.s.dbg_val[1];
          dbg[3] = ej.s.dbg_val[2];
        } else {
          err = rlt_evict<PT>(P, ej, us, dbg, &clk, KVR_PHASE_E_EVICT, KVR_PHASE_E_FINISH, hook);
        }
        if (err) {
          pipe_stop(&f, kq, err, dbg);
          break;
        }
        // finished: the worker is free again
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane == 0) {
          __hip_atomic_fetch_and(&st_sh[job.worker], ~(kOwner | kLoaded | kMarked | kDeferred), __ATOMIC_RELEASE,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_store(&jdone_sh[slot], kq + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        continue;
      }
    }
  } else {
    // ---------------------------------------------------------- helper wave
    for (;;) {
      // the match to take this round, if any: query mm on worker mw, whose state
      // was msv
      uint32_t msv = 0, mm = 0, mw = 0;
      bool take = false;
      const uint32_t hw = wave - NE - 1u;
      const uint32_t fv = __hip_atomic_load(reinterpret_cast<uint32_t*>(&f) + (lane & (kFlagWords - 1)),
                                            __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
      const uint32_t routed = (uint32_t)__builtin_amdgcn_readlane((int)fv, 0);
      const uint32_t fronts = (uint32_t)__builtin_amdgcn_readlane((int)fv, 1);
      const uint32_t staged = (uint32_t)__builtin_amdgcn_readlane((int)fv, 2);
      const uint32_t ended = (uint32_t)__builtin_amdgcn_readlane((int)fv, 6);
      const uint32_t stopped = (uint32_t)__builtin_amdgcn_readlane((int)fv, 7);
      if (dN < routed && (hw > 0 || stopped || sN > dN + 1u || dN + 1u == n)) {
        // ---- what a routed query needs from this wave (the first helper
        // needs the next arrival, which it puts down when it stages the query)
        clock_mark<PT>(&clk, KVR_PHASE_H_WAIT);
        const uint32_t k = dN, slot = k % kJobs;
        dN += 1;
        spins = 0;
        if (hw == 0) {
          // its outputs, then completions and decay at the next arrival
          const uint32_t best = uni(best_sh[slot]);
          const int32_t hb = uni(hit_sh[slot]);
          const uint64_t orow = (uint64_t)r * a.rows + k;
          if (lane == 0) {
            if (a.route) a.route[orow] = (int32_t)best;
            if (a.hits) a.hits[orow] = hb;
          }
          if (a.all_hits && (uint32_t)lane < W) a.all_hits[orow * W + (uint32_t)lane] = (uint32_t)lane == best ? hb : h_sh[query_slot(k, a.nbuf)][lane];
          if (k + 1u < n && !stopped) {
            const int64_t t = arr_sh[(k + 1u) & 7u], tp = arr_sh[k & 7u];
            const int64_t tick = t / a.C.dt_us;
            if ((uint32_t)lane < W) {
              const Ptrs P = worker_ptrs(a.ws, a.L, r, (uint32_t)lane);
              decay_lds(a.C, lb, (uint32_t)lane, P.hdr, P.pend, P.PC, t, tp, tick, tick_prev);
            }
            tick_prev = tick;
            st_rel(&f.decayed, k + 2u);
          }
          chain = route_chain(chain, a.j0 + k, best, hb);
          routed_total += 1;
          clock_mark<PT>(&clk, KVR_PHASE_H_OTHER);
        } else if (hw <= ndraw && !stopped) {
          // draw words, a round of 2 nd words at a time; each round written is
          // published
          const uint64_t info = rn_sh[slot];
          const uint32_t rn = uni((uint32_t)info);
          if (uni((uint32_t)(info >> 32)) == k + 1u && rn > 0u) {
            const uint32_t best = uni(best_sh[slot]);
            uint32_t* rw = ring + uni(r0_sh[slot]);
            uint32_t rounds = 0;
            for (uint32_t base = 0; base < rn; base += 2u * nd) {
              const uint32_t d0 = base + (hw - 1u) * KVR_WAVE + (uint32_t)lane, d1 = d0 + nd;
              const uint64_t w0 = philox_word0(a.j0 + k, best, d0, 0ull, a.C.seed, r);
              const uint64_t w1 = philox_word0(a.j0 + k, best, d1, 0ull, a.C.seed, r);
              if (d0 < rn) rw[d0] = (uint32_t)(w0 >> 32);
              if (d1 < rn) rw[d1] = (uint32_t)(w1 >> 32);
              ++rounds;
              st_rel(&prog_sh[slot][hw - 1u], rounds);
            }
          }
          clock_mark<PT>(&clk, KVR_PHASE_H_DRAW);
        }
        continue;
      }
      if (stopped) break;
      // ---- a new leaf's rank that nobody has taken
      const uint32_t rv = (uint32_t)lane < kJobs ? __hip_atomic_load(&rank_ready_sh[lane], __ATOMIC_ACQUIRE,
                                                                     __HIP_MEMORY_SCOPE_WORKGROUP)
                                                 : 0u;
      const uint64_t rm = __ballot((rv & 3u) == 1u);
      if (rm) {
        clock_mark<PT>(&clk, KVR_PHASE_H_WAIT);
        const int slot = first_lane(rm);
        const uint32_t want = (uint32_t)__builtin_amdgcn_readlane((int)rv, slot);
        uint32_t old = 0;
        if (lane == 0) old = atomicCAS(&rank_ready_sh[slot], want, want + 1u);
        if (uni(old) == want) {
          const PipeJob job = load_job(&job_sh[slot]);
          const St s = load_st_lds(tree_sh + job.worker * kStWords);
          const Ptrs P = worker_ptrs(a.ws, a.L, r, job.worker);
          const int32_t pos = rank_of_leaf(P, s.hwm, s.nleaves, arena_of(P, s.arena_sel), job);
          if (lane == 0) rank_sh[slot] = pos;
          st_rel(&rank_ready_sh[slot], want + 2u);
          clock_mark<PT>(&clk, KVR_PHASE_H_OTHER);
        }
        spins = 0;
        continue;
      }
      // ---- stage the next query whose buffer is free
      if (sN < n && sN < fronts + a.nbuf && staged >= sN * nh) {
        clock_mark<PT>(&clk, KVR_PHASE_H_WAIT);
        const uint64_t o0 = a.offsets[sN];
        const int32_t Ln = (int32_t)(a.offsets[sN + 1u] - o0);
        const int32_t Lc = sN > 0u ? uni(len_sh[(sN - 1u) & 7u]) : 0;
        if (hw == 0 && lane == 0) {
          len_sh[sN & 7u] = Ln;
          olen_sh[sN & 7u] = query_out_len(a.out_len, sN);
          arr_sh[sN & 7u] = a.arrival[sN];
        }
        int32_t* qn = smem + query_slot(sN, a.nbuf) * qwords + kQueryPad;
        const int32_t* qc = smem + query_slot(sN + a.nbuf - 1u, a.nbuf) * qwords + kQueryPad;
        stage_query<4>(a.tokens, o0, Ln, qn, qc, Lc, hw * KVR_WAVE, nh * KVR_WAVE, &ell_sh[(sN - 1u) & 7u]);
        add_rel(&f.staged, 1u);
        sN += 1;
        spins = 0;
        clock_mark<PT>(&clk, KVR_PHASE_H_STAGE);
        continue;
      }
      // ---- a match: on each worker the next query not matched there, as far
      // as queries are staged and their trails' slots are free (q_m takes that
      // of q_m-nbuf, whose leaf must be loaded); the earliest query first, and
      // each helper from another worker on
      if (routed < n) {
        const uint32_t whole = staged / nh;  // queries staged
        uint32_t lim = fronts + a.nbuf;
        if (lim > whole) lim = whole;        // matches of queries below this
        const uint32_t sv = (uint32_t)lane < W ? __hip_atomic_load(&st_sh[lane], __ATOMIC_ACQUIRE,
                                                                   __HIP_MEMORY_SCOPE_WORKGROUP)
                                               : 0u;
        const uint32_t m = routed + (((sv >> kCountShift) - routed) & kCountMask);
        const bool ok = (uint32_t)lane < W && m < lim && can_match(sv, m, owner_sh[lane & (kMaxWorkers - 1u)], a.nbuf);
        // all that are zero, a worker per lane (in the form for many workers)
        if constexpr (NW > kPipeWaves) {
          const bool took = ok && take_zero_match(ma, m, (uint32_t)lane, sv);
          if (__ballot(took)) {
            spins = 0;
            clock_mark<PT>(&clk, KVR_PHASE_H_MATCH);
            continue;
          }
        }
        uint64_t can = __ballot(ok && m == routed);
        if (!can) can = __ballot(ok && m == routed + 1u);
        if (!can) can = __ballot(ok);
        if (can) {
          clock_mark<PT>(&clk, KVR_PHASE_H_WAIT);
          const uint64_t hi = can & (~0ull << (hw * W / nh));
          if (hi) can = hi;
          mw = (uint32_t)first_lane(can);
          mm = (uint32_t)__builtin_amdgcn_readlane((int)m, (int)mw);
          msv = (uint32_t)__builtin_amdgcn_readlane((int)sv, (int)mw);
          if (!claim_match(&st_sh[mw], msv)) continue;
          take = true;
          spins = 0;
        }
      }
      if (!take) {
        if (ended && dN >= routed && fronts == n) break;  // (and no rank is wanted)
        const uint32_t now = routed + fronts + staged;
        if (now != seen) {
          seen = now;
          spins = 0;
        }
        if (!pipe_poll(spins, &f, routed, 9)) continue;  // (the duties of routed queries first)
        continue;
      }
      take_match<kPipeMatchUnroll>(ma, worker_ptrs(a.ws, a.L, r, mw), mm, mw, msv);
      clock_mark<PT>(&clk, KVR_PHASE_H_MATCH);
    }
  }
  if (wave == 0) {
    st_rel(&f.end, 1u);
    if constexpr (PT)
      if (lane == 0)
        for (int p = 0; p < KVR_PHASES; ++p) rh->phase_ticks[p] += clk.acc[p];
  } else {
    if constexpr (PT)
      if (lane == 0)
        for (int p = KVR_PHASE_E_EVICT; p < KVR_PHASES; ++p) atomicAdd(&eticks_sh[p], (unsigned long long)clk.acc[p]);
    if (wave == NE + 1u && lane == 0) {
      rh->route_digest = chain;
      rh->queries = routed_total;
    }
  }
  __syncthreads();
  // ---- the launch's state back to the headers
  for (uint32_t x = threadIdx.x; x < W * (uint32_t)kStWords; x += 64 * NW)
    if (x % kStWords < (uint32_t)kStWords - 1u)
      reinterpret_cast<uint32_t*>(worker_ptrs(a.ws, a.L, r, x / kStWords).hdr)[x % kStWords] = tree_sh[x];
  if (threadIdx.x < W) {
    const uint32_t w = threadIdx.x;
    WorkerHdr* h = worker_ptrs(a.ws, a.L, r, w).hdr;
    h->P = lb.P[w];
    for (int k = 0; k < 4; ++k) h->theta[k] = lb.theta[k * W + w];
    h->Wb = lb.Wb[w];
    if (f.decayed > 0u) h->tl = a.arrival[f.decayed - 1u];
    h->pend_head = lb.head[w];
    h->pend_count = lb.count[w];
    h->matched_tokens += mtok_sh[w];
  }
  if (threadIdx.x == 0) {
    if constexpr (PT)
      for (int p = KVR_PHASE_E_EVICT; p < KVR_PHASES; ++p) rh->phase_ticks[p] += eticks_sh[p];
    if (f.err) {
      rh->failed = 1;
      if (atomicCAS(&g->err_taken, 0u, 1u) == 0u) {
        g->err_check = f.err_check;
        g->err_replica = r;
        g->err_query = a.j0 + f.err_query;
        g->err_val[0] = f.err_val[0];
        g->err_val[1] = f.err_val[1];
        g->err_val[2] = f.err_val[2];
      }
      atomicOr(&g->status, f.err);
    }
    if (!f.stop) {
      rh->tprev = a.arrival[n - 1u];
      if (r == 0) g->last_arrival = a.arrival[n - 1u];
    }
  }
}

// Zero n 32-bit words (in-progress counts of continuous batching).
__global__ void zero_words_kernel(uint32_t* p, uint64_t n) {
  for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x)
    p[x] = 0u;
}

__global__ void init_kernel(char* ws, Layout L, double rls_p0) {
  const uint64_t RW = (uint64_t)L.R * L.W;
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid == 0) {
    GlobalHdr* g = reinterpret_cast<GlobalHdr*>(ws + L.off_global);
    g->status = 0;
    g->err_taken = 0;
    g->last_arrival = 0;
    g->err_check = 0;
    g->err_replica = 0;
    g->err_query = 0;
    g->err_val[0] = g->err_val[1] = g->err_val[2] = 0;
  }
  if (tid < L.R) {
    ReplicaHdr h;
    h.tprev = 0;
    h.queries = 0;
    h.route_digest = 0;
    for (int k = 0; k < KVR_PHASES; ++k) h.phase_ticks[k] = 0;
    h.failed = 0;
    for (uint64_t& x : h.pad) x = 0;
    reinterpret_cast<ReplicaHdr*>(ws + L.off_rhdr)[tid] = h;
  }
  if (tid < RW) {
    init_worker(worker_ptrs(ws, L, (uint32_t)(tid / L.W), (uint32_t)(tid % L.W)), rls_p0);
    if (L.has_router) init_worker(router_ptrs(ws, L, (uint32_t)(tid / L.W), (uint32_t)(tid % L.W)), rls_p0);
  }
}

// Batch checks before any state changes: lengths (with cached responses, a
// prompt of at least one token before the response) and arrival order.
__global__ void validate_kernel(char* ws, Layout L, const uint64_t* offsets, const int64_t* arrival,
                                const uint16_t* out_len, int32_t resp, uint32_t n) {
  GlobalHdr* g = reinterpret_cast<GlobalHdr*>(ws + L.off_global);
  uint32_t bits = 0;
  for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
       j += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t o0 = offsets[j], o1 = offsets[j + 1];
    if (o1 <= o0 || o1 - o0 > L.maxL) bits |= KVR_DEV_BAD_LENGTH;
    if (resp && o1 - o0 <= (uint64_t)query_out_len(out_len, j)) bits |= KVR_DEV_BAD_LENGTH;
    const int64_t prev = j == 0 ? g->last_arrival : arrival[j - 1];
    if (arrival[j] < prev) bits |= KVR_DEV_BAD_ARRIVAL;
  }
  if (bits) atomicOr(&g->status, bits);
}

// Token ids must be >= 0 (checked only when the offsets passed).
__global__ void validate_tokens_kernel(char* ws, Layout L, const int32_t* tokens,
                                       const uint64_t* offsets, uint32_t n) {
  GlobalHdr* g = reinterpret_cast<GlobalHdr*>(ws + L.off_global);
  if (__atomic_load_n(&g->status, __ATOMIC_RELAXED)) return;
  const uint64_t b = offsets[0], e = offsets[n];
  uint32_t bad = 0;
  for (uint64_t x = b + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < e;
       x += (uint64_t)gridDim.x * blockDim.x)
    if (tokens[x] < 0) bad = 1;
  if (__ballot(bad != 0) && lane_id() == 0) atomicOr(&g->status, (uint32_t)KVR_DEV_BAD_TOKEN);
}

// Final state of every (replica, worker): one wave each, for the workers
// w0 .. w0 + gridDim.x - 1 (index r * W + i).  The digest walk's FIFO is
// fifo + (widx - w0) * fifo_words (fifo_words / 2 entries), or the worker's
// scratch region when fifo is null; the records go to out[widx - w0].  An
// inconsistent tree or a FIFO too short raises KVR_DEV_INTERNAL.
__global__ void __launch_bounds__(64) stats_kernel(char* ws, Layout L, uint64_t w0, uint64_t* fifo,
                                                   uint64_t fifo_words, kvr_worker_stats* out) {
  const uint64_t widx = w0 + blockIdx.x;
  const uint32_t r = (uint32_t)(widx / L.W), i = (uint32_t)(widx % L.W);
  kvr_worker_stats* o = out + blockIdx.x;
  uint64_t* q = fifo ? fifo + (uint64_t)blockIdx.x * fifo_words : nullptr;
  bool ok = worker_stats(worker_ptrs(ws, L, r, i), o, q, fifo_words / 2);
  if (L.has_router) {
    // the router's tree of the worker (its walk reuses the same FIFO once
    // the cache's is done): contents digest and evictions
    wave_mem_sync();
    Ptrs Pr = router_ptrs(ws, L, r, i);
    kvr_worker_stats t;
    ok = worker_stats(Pr, &t, q, fifo_words / 2) && ok;
    if (lane_id() == 0) {
      o->router_resident = t.resident;
      o->router_digest_sum = t.digest_sum;
      o->router_digest_xor = t.digest_xor;
      o->router_evictions = Pr.hdr->evictions;
    }
  }
  if (!ok && lane_id() == 0) atomicOr(&reinterpret_cast<GlobalHdr*>(ws + L.off_global)->status, (uint32_t)KVR_DEV_INTERNAL);
}

// ---------------------------------------------------------------- launchers (host)

size_t step_lds_bytes(uint32_t maxL, uint32_t W, uint32_t ucap, uint32_t rcap, uint32_t path_sets) {
  return 2 * (size_t)query_words(maxL) * sizeof(int32_t) + (size_t)rcap * sizeof(uint32_t) +
         (size_t)path_sets * W * (3 * kPathMax + 1) * sizeof(int32_t) + (size_t)ucap * 4u * sizeof(int32_t);
}


// Dynamic LDS of the pipelined step kernel: nbuf query buffers; per worker the
// LBGR and tree state, the state word, nbuf trails and the root filter; rcap
// draw words; ucap staged candidates per evicting wave.
size_t step_lds_bytes_pipe(uint32_t maxL, uint32_t W, uint32_t nbuf, uint32_t ucap, uint32_t rcap) {
  return (size_t)nbuf * query_words(maxL) * 4u +
         (size_t)W * (kLbgrBytes + 4u * (1u + (uint32_t)kStWords + nbuf * (uint32_t)kTrailWords + kRootFilterWords)) +
         (size_t)rcap * 4u + (size_t)kPipeEvictors * ucap * 16u;
}

uint32_t step_pipe_evictors() { return kPipeEvictors; }

hipError_t launch_init(char* ws, const Layout& L, double rls_p0, hipStream_t st) {
  const uint64_t work = (uint64_t)L.R * L.W > L.R ? (uint64_t)L.R * L.W : L.R;
  const uint32_t blocks = (uint32_t)((work + 255) / 256);
  hipLaunchKernelGGL(init_kernel, dim3(blocks), dim3(256), 0, st, ws, L, rls_p0);
  if (L.pin_stride) {
    const uint64_t words = (uint64_t)L.R * L.W * L.pin_stride / 4u;
    hipLaunchKernelGGL(zero_words_kernel, dim3(1024), dim3(256), 0, st, reinterpret_cast<uint32_t*>(ws + L.off_pin),
                       words);
  }
  return hipGetLastError();
}

// Batches of at most this many tokens (at the longest) are checked by the step
// kernel itself, each workgroup for itself, instead of by two kernels before it:
// 3 us less a call (26.7 to 22.4 us for one short query).  At 33,000 tokens the two
// are equal (217 us), above it the kernels are ahead.  With one query a call, the
// time of 96 calls is 5.29 instead of 5.55 ms for 512 replicas, 10.05 instead of
// 10.23 for 1,024, and 38.1 instead of 37.7 for 4,096, where each compute unit checks
// the batch 16 times.
#ifndef KVR_CHECK_TOKENS
#define KVR_CHECK_TOKENS 8192
#endif
constexpr uint64_t kCheckTokens = KVR_CHECK_TOKENS;
constexpr uint32_t kCheckQueries = 256;  // (four rounds of a wave's lanes over their lengths)
constexpr uint32_t kCheckReplicas = 1024;

// A launch of the pipelined kernel takes at most this many queries: its counters
// run up to (queries + 4) x helper waves in 32 bits, and a launch more costs
// about 10 us, 0.1% of the time of this many steps.
constexpr uint32_t kLaunchQueries = 2048;

void launch_pipe(const StepArgs& a, size_t lds, hipStream_t st) {
  const bool lbgr = a.C.router == KVR_ROUTE_LBGR;
#define KVR_PIPE_LAUNCH(PT, NW, LB) \
  hipLaunchKernelGGL((step_kernel_pipe<PT, NW, kPipeEvictors, LB>), dim3(a.L.R), dim3(64 * NW), lds, st, a)
  if (a.L.W >= kPipeWideWorkers) {
    if (a.C.phase_timers)
      KVR_PIPE_LAUNCH(true, kPipeWavesWide, false);
    else if (lbgr)
      KVR_PIPE_LAUNCH(false, kPipeWavesWide, true);
    else
      KVR_PIPE_LAUNCH(false, kPipeWavesWide, false);
  } else {
    if (a.C.phase_timers)
      KVR_PIPE_LAUNCH(true, kPipeWaves, false);
    else if (lbgr)
      KVR_PIPE_LAUNCH(false, kPipeWaves, true);
    else
      KVR_PIPE_LAUNCH(false, kPipeWaves, false);
  }
#undef KVR_PIPE_LAUNCH
}

hipError_t launch_step(const StepArgs& args, hipStream_t st) {
  StepArgs a = args;
  a.check = a.n <= kCheckQueries && (uint64_t)a.n * a.L.maxL <= kCheckTokens && a.L.R <= kCheckReplicas ? 1u : 0u;
  if (!a.check) {
    const uint32_t blocks_v = (a.n + 255) / 256 < 1024 ? (a.n + 255) / 256 : 1024;
    hipLaunchKernelGGL(validate_kernel, dim3(blocks_v ? blocks_v : 1), dim3(256), 0, st, a.ws, a.L,
                       a.offsets, a.arrival, a.out_len, a.C.cache_responses, a.n);
    hipLaunchKernelGGL(validate_tokens_kernel, dim3(1024), dim3(256), 0, st, a.ws, a.L, a.tokens,
                       a.offsets, a.n);
  }
  const uint32_t waves = a.L.W < kMaxWavesPerBlock ? a.L.W : kMaxWavesPerBlock;
  const size_t lds = step_lds_bytes(a.L.maxL, a.L.W, a.ucap, a.rcap, a.L.has_router ? 2u : 1u);
  const bool rt = a.L.has_router != 0, ba = a.L.beta > 1;
  if (a.pipe) {
    const size_t lds_p = step_lds_bytes_pipe(a.L.maxL, a.L.W, a.nbuf, a.ucap, a.rcap);
    for (uint32_t k0 = 0; k0 < args.n; k0 += kLaunchQueries) {
      a.n = args.n - k0 < kLaunchQueries ? args.n - k0 : kLaunchQueries;
      a.offsets = args.offsets + k0;
      a.arrival = args.arrival + k0;
      a.out_len = args.out_len ? args.out_len + k0 : nullptr;
      a.route = args.route ? args.route + k0 : nullptr;
      a.hits = args.hits ? args.hits + k0 : nullptr;
      a.all_hits = args.all_hits ? args.all_hits + (uint64_t)k0 * a.L.W : nullptr;
      a.j0 = args.j0 + k0;
      a.part = k0 > 0 ? 1u : 0u;
      launch_pipe(a, lds_p, st);
    }
  } else if (rt && ba)
    hipLaunchKernelGGL((step_kernel<true, true, false>), dim3(a.L.R), dim3(64 * waves), lds, st, a);
  else if (rt)
    hipLaunchKernelGGL((step_kernel<true, false, false>), dim3(a.L.R), dim3(64 * waves), lds, st, a);
  else if (ba)
    hipLaunchKernelGGL((step_kernel<false, true, false>), dim3(a.L.R), dim3(64 * waves), lds, st, a);
  else if (a.C.phase_timers)
    hipLaunchKernelGGL((step_kernel<false, false, true>), dim3(a.L.R), dim3(64 * waves), lds, st, a);
  else
    hipLaunchKernelGGL((step_kernel<false, false, false>), dim3(a.L.R), dim3(64 * waves), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_stats(char* ws, const Layout& L, hipStream_t st) {
  hipLaunchKernelGGL(stats_kernel, dim3(L.R * L.W), dim3(64), 0, st, ws, L, 0ull, nullptr, 0ull,
                     reinterpret_cast<kvr_worker_stats*>(ws + L.off_stats));
  return hipGetLastError();
}

// ---------------------------------------------------------------- allocation-free statistics
//
// kvr_stats_noalloc keeps the digest walk's FIFO and the staged records in
// this array instead of the workspace; one copy per device, for the life of
// the process.  Host code uses its address from hipGetSymbolAddress, never
// its name.
constexpr size_t kScratchBytes = 32ull << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// The device address of `scratch` on the current device (looked up once per
// device).
hipError_t noalloc_scratch(int device, void** ptr, size_t* bytes) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = p;
  }
  *ptr = g_scratch_ptr[device];
  *bytes = kScratchBytes;
  return hipSuccess;
}

// Workers w0 .. w0 + n - 1 with their FIFOs (fifo_words each) and records
// in caller-given device memory.
hipError_t launch_stats_into(char* ws, const Layout& L, uint64_t w0, uint32_t n, uint64_t* fifo, uint64_t fifo_words,
                             kvr_worker_stats* out, hipStream_t st) {
  hipLaunchKernelGGL(stats_kernel, dim3(n), dim3(64), 0, st, ws, L, w0, fifo, fifo_words, out);
  return hipGetLastError();
}

static const void* const kStepKernels[11] = {
    reinterpret_cast<const void*>(step_kernel_pipe<false, kPipeWaves, kPipeEvictors, true>),
    reinterpret_cast<const void*>(step_kernel_pipe<false, kPipeWaves, kPipeEvictors, false>),
    reinterpret_cast<const void*>(step_kernel_pipe<true, kPipeWaves, kPipeEvictors, false>),
    reinterpret_cast<const void*>(step_kernel_pipe<false, kPipeWavesWide, kPipeEvictors, true>),
    reinterpret_cast<const void*>(step_kernel_pipe<false, kPipeWavesWide, kPipeEvictors, false>),
    reinterpret_cast<const void*>(step_kernel_pipe<true, kPipeWavesWide, kPipeEvictors, false>),
    reinterpret_cast<const void*>(step_kernel<false, false, false>),
    reinterpret_cast<const void*>(step_kernel<false, true, false>),
    reinterpret_cast<const void*>(step_kernel<true, false, false>),
    reinterpret_cast<const void*>(step_kernel<true, true, false>),
    reinterpret_cast<const void*>(step_kernel<false, false, true>)};

// Static LDS of the step kernels (their __shared__ variables, the largest),
// from the compiled kernels' attributes.
hipError_t step_static_lds(size_t* bytes) {
  size_t mx = 0;
  for (const void* f : kStepKernels) {
    hipFuncAttributes fa;
    const hipError_t e = hipFuncGetAttributes(&fa, f);
    if (e != hipSuccess) return e;
    if (fa.sharedSizeBytes > mx) mx = fa.sharedSizeBytes;
  }
  *bytes = mx;
  return hipSuccess;
}

hipError_t set_step_lds_limit(size_t bytes) {
  for (const void* f : kStepKernels) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace kvr
