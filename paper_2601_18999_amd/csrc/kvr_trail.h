// kvr_trail.h - per-wave tree logic of the pipelined step kernel (included by
// kvr_device.hip and by the single-lane replay): matches taken a query ahead
// along recorded trails, the order of a worker's matches and insertions, the two
// halves of an insertion (the load of the new leaf; marks, leaf list and
// evictions, both on an evicting wave), and completions and decay on state kept
// in LDS.
//
// Everything a wave decides on is wave-uniform and is read as such: a node
// record, a worker's state and a job are each read with one load, a word per
// lane, and taken to scalar registers with readlane.  The matching code is in the
// kernel twice, in the routing wave's loop and in the helpers'.
#ifndef KVR_TRAIL_H
#define KVR_TRAIL_H

#include "kvr_core.h"

namespace kvr {

// ---------------------------------------------------------------- a worker's tree state in LDS

constexpr int kStWords = 16;  // the words of St that a header holds, padded

__device__ __forceinline__ St load_st_lds(const uint32_t* p) {
  uint32_t f[kStWords - 1];
  if (KVR_WAVE == 1) {
    for (int k = 0; k < kStWords - 1; ++k) f[k] = p[k];
  } else {
    const uint32_t v = p[lane_id() & (kStWords - 1)];
#pragma unroll
    for (int k = 0; k < kStWords - 1; ++k) f[k] = (uint32_t)__builtin_amdgcn_readlane((int)v, k);
  }
  St s;
  s.phase = f[0];
  s.cnt = f[1];
  s.size = f[2];
  s.hwm = f[3];
  s.free_head = (int32_t)f[4];
  s.nleaves = f[5];
  s.nU = f[6];
  s.U_valid = f[7];
  s.rnode = (int32_t)f[8];
  s.rlo = (int32_t)f[9];
  s.rhi = (int32_t)f[10];
  s.rphase = f[11];
  s.arena_sel = f[12];
  s.arena_top = f[13];
  s.nnodes = f[14];
  s.err = 0;
  s.dbg_check = 0;
  s.dbg_val[0] = s.dbg_val[1] = s.dbg_val[2] = 0;
  return s;
}

__device__ __forceinline__ void store_st_lds(uint32_t* p, const St& s) {
  if (lane_id() != 0) return;
  p[0] = s.phase;
  p[1] = s.cnt;
  p[2] = s.size;
  p[3] = s.hwm;
  p[4] = (uint32_t)s.free_head;
  p[5] = s.nleaves;
  p[6] = s.nU;
  p[7] = s.U_valid;
  p[8] = (uint32_t)s.rnode;
  p[9] = (uint32_t)s.rlo;
  p[10] = (uint32_t)s.rhi;
  p[11] = s.rphase;
  p[12] = s.arena_sel;
  p[13] = s.arena_top;
  p[14] = s.nnodes;
}

// ---------------------------------------------------------------- root filters
// Per worker a 256-bit Bloom filter (in LDS) of the first tokens of its
// root's children, two bits per token, built when the kernel starts and
// extended when an insertion adds a child to the root.  A clear bit proves
// that no cached path starts with the token, so a match that starts at the
// root is 0 without a memory access; a set bit (also one left by a child
// evicted since) only means the tree is walked.  (512- and 1,024-bit filters
// measured within 1% of this.)
#ifndef KVR_ROOT_FILTER_LOG2_BITS
#define KVR_ROOT_FILTER_LOG2_BITS 8
#endif
constexpr uint32_t kRootFilterBits = 1u << KVR_ROOT_FILTER_LOG2_BITS;
constexpr uint32_t kRootFilterWords = kRootFilterBits / 32u;

__device__ __forceinline__ uint32_t rf_bit1(int32_t t) {
  return ((uint32_t)t * 0x9E3779B1u) >> (32 - KVR_ROOT_FILTER_LOG2_BITS);
}
__device__ __forceinline__ uint32_t rf_bit2(int32_t t) {
  return ((uint32_t)t * 0x85EBCA6Bu + 0x632BE5ABu) >> (32 - KVR_ROOT_FILTER_LOG2_BITS);
}

__device__ __forceinline__ void rf_add(uint32_t* rf, int32_t t) {
  atomicOr(&rf[rf_bit1(t) >> 5], 1u << (rf_bit1(t) & 31u));
  atomicOr(&rf[rf_bit2(t) >> 5], 1u << (rf_bit2(t) & 31u));
}

__device__ __forceinline__ bool rf_may(const uint32_t* rf, int32_t t) {
  return ((rf[rf_bit1(t) >> 5] >> (rf_bit1(t) & 31u)) & 1u) && ((rf[rf_bit2(t) >> 5] >> (rf_bit2(t) & 31u)) & 1u);
}

// The buffer of query k (nbuf = 2, 3 or 4).
__device__ __forceinline__ uint32_t query_slot(uint32_t k, uint32_t nbuf) {
  return nbuf == 3u ? k % 3u : k & (nbuf - 1u);
}

// ---------------------------------------------------------------- trails
// The trail of a match: the nodes it entered, [0] = their number (kPathMax + 1
// when there were more or they are unknown), then the nodes, then the depth
// after each node's edge (entry e starts where entry e - 1 ends).  A worker
// has as many as there are query buffers (nbuf, two to four; query k's in slot
// query_slot(k)), so that the next queries can be matched while the insertion of
// this one still needs its trail.
constexpr int32_t kTrailWords = 2 * kPathMax + 1;

__device__ __forceinline__ int32_t* trail_node(int32_t* t) { return t + 1; }
__device__ __forceinline__ const int32_t* trail_node(const int32_t* t) { return t + 1; }
__device__ __forceinline__ int32_t* trail_end(int32_t* t) { return t + 1 + kPathMax; }
__device__ __forceinline__ const int32_t* trail_end(const int32_t* t) { return t + 1 + kPathMax; }

__device__ __forceinline__ void trail_add(int32_t* t, int32_t& pc, int32_t node, int32_t end) {
  if (pc < kPathMax && lane_id() == 0) {
    trail_node(t)[pc] = node;
    trail_end(t)[pc] = end;
  }
  pc = pc < kPathMax ? pc + 1 : kPathMax + 1;
}

// A trail as a wave reads it: an entry per lane, so that everything looked up
// in it is one round of LDS reads.
struct TrailView {
  int32_t count, vnode, vend;
  const int32_t* t;
  __device__ __forceinline__ int32_t node(int32_t e) const {
    return KVR_WAVE == 1 ? t[1 + e] : __builtin_amdgcn_readlane(vnode, e);
  }
  __device__ __forceinline__ int32_t end(int32_t e) const {
    return KVR_WAVE == 1 ? t[1 + kPathMax + e] : __builtin_amdgcn_readlane(vend, e);
  }
  __device__ __forceinline__ int32_t start(int32_t e) const { return e > 0 ? end(e - 1) : 0; }
  // the last entry that starts above depth d > 0 (it holds depth d if any
  // does); -1 when there is none
  __device__ __forceinline__ int32_t at(int32_t d) const {
    if (KVR_WAVE == 1) {
      int32_t e = count - 1;
      while (e > 0 && end(e - 1) >= d) --e;
      return e;
    }
    return count > 0 ? (int32_t)__popcll(__ballot(lane_id() < count - 1 && vend < d)) : -1;
  }
  // the first n entries into another trail
  __device__ __forceinline__ void copy_to(int32_t* dst, int32_t n) const {
    if (KVR_WAVE == 1) {
      for (int32_t e = 0; e < n; ++e) {
        dst[1 + e] = t[1 + e];
        dst[1 + kPathMax + e] = t[1 + kPathMax + e];
      }
    } else if (lane_id() < n) {
      dst[1 + lane_id()] = vnode;
      dst[1 + kPathMax + lane_id()] = vend;
    }
  }
};
static_assert(KVR_WAVE == 1 || KVR_WAVE >= kPathMax, "a trail's entries fit a wave's lanes");

__device__ __forceinline__ TrailView view_trail(const int32_t* t) {
  TrailView v;
  v.t = t;
  const int32_t c = t[0];
  v.vnode = t[1 + (lane_id() & (kPathMax - 1))];
  v.vend = t[1 + kPathMax + (lane_id() & (kPathMax - 1))];
  v.count = uni(c);
  return v;
}

// ---------------------------------------------------------------- matching

// Where a match ended: `pos` tokens into the edge of `node` (0: at the root).
struct MatchEnd {
  int32_t node, pos;
};

// h = length of the longest prefix of q[0, L) in a worker's tree, whose match
// of the previous query is recorded in src (h_old = its h; ell = LCP of the
// two queries).  Up to depth min(h_old, ell) both walks are the same.  If the
// old match stopped first, the new one stops there; else the new one leaves
// the old query's path at depth ell: inside an edge that the old match
// followed further it stops, otherwise it goes on from there.  The new trail
// is written to dst (another array).  `walked` is false when no node was read,
// and me is then unset.  The tree may be one whose evictions are under way (see
// match_stays): a node freed meanwhile holds the free list's next entry in
// place of its offset, so offsets are checked against the semispace's size A.
template <int kU>
__device__ __forceinline__ int32_t match_ahead(const NodeRec* nodes, const int32_t* ar, const uint32_t* rf,
                                               uint32_t A, const int32_t* q, int32_t L, int32_t h_old, int32_t ell,
                                               const int32_t* src, int32_t* dst, bool& walked, MatchEnd& me) {
  const TrailView v = view_trail(src);
  int32_t x = 0, off = 0, d = 0, pc = 0;
  bool walk = true;
  if (ell > 0 && v.count <= kPathMax) {
    if (h_old < ell) {
      pc = v.count;
      d = h_old;
      walk = false;
    } else {
      const int32_t e = v.at(ell);
      if (e >= 0 && v.end(e) >= ell) {  // (always, for a consistent record)
        pc = e + 1;
        d = ell;
        if (ell == L || (ell < v.end(e) && h_old > ell)) {
          walk = false;
        } else {
          x = v.node(e);
          off = ell - v.start(e);
        }
      }
    }
  }
  if (walk && x == 0 && !rf_may(rf, uni(q[0]))) walk = false;
  v.copy_to(dst, pc);
  walked = walk;
  if (walk) {
    NodeRec nx = load_node(nodes, x);
    while (d < L) {
      if (off < nx.len) {  // the rest of this edge
        const int32_t rest = nx.len - off;
        const int32_t n = rest < L - d ? rest : L - d;
        const int32_t k = same_words<kU>(ar, nx.off + (uint32_t)off, q, d, n);
        d += k;
        off += k;
        if (k < rest) break;
        continue;
      }
      const int32_t c = child_find(ar, nx, uni(q[d]));
      if (c < 0) break;
      x = c;
      off = 0;
      nx = load_node(nodes, c);
      if (nx.len <= 0 || (uint64_t)nx.off + (uint32_t)nx.len > A) break;  // freed meanwhile
      trail_add(dst, pc, c, d + nx.len);
      d += 1;  // the child entry holds the edge's first token
      off = 1;
    }
    me.node = x;
    me.pos = off;
  }
  if (lane_id() == 0) dst[0] = pc;
  return d;
}

// ---------------------------------------------------------------- insertion

// An insertion: what the routing wave plans (k, worker, h, L, nfree, nev, rn, r0,
// calm, phase, pre) and what its load adds (LDS, one word per lane).
struct PipeJob {
  uint32_t k;       // query index in the batch
  uint32_t worker;
  int32_t h, L;     // cached length and length of the path
  int32_t l, a;     // the new leaf holding q[h, L) and the node it hangs from (h < L)
  int32_t tok;      // q[h]
  uint32_t nfree;   // free token slots before the load
  uint32_t nev;     // evictions the load needs
  uint32_t rn, r0;  // its draw words: how many, and where in the ring
  uint32_t replace; // a was a leaf
  uint32_t marked;  // the cached part is marked already
  uint32_t calm;    // no new phase can start in this insertion (match_stays)
  uint32_t phase;   // the phase before it
  int32_t pre;      // h of the next query's match taken before the load and final, else -1
};
constexpr int kJobWords = sizeof(PipeJob) / 4;
static_assert(kJobWords == 16, "a job is one word per lane of a row");

__device__ __forceinline__ PipeJob load_job(const PipeJob* p) {
  if (KVR_WAVE == 1) return *p;
  const uint32_t v = reinterpret_cast<const uint32_t*>(p)[lane_id() & (kJobWords - 1)];
  PipeJob j;
  uint32_t f[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) f[k] = (uint32_t)__builtin_amdgcn_readlane((int)v, k);
  j.k = f[0];
  j.worker = f[1];
  j.h = (int32_t)f[2];
  j.L = (int32_t)f[3];
  j.l = (int32_t)f[4];
  j.a = (int32_t)f[5];
  j.tok = (int32_t)f[6];
  j.nfree = f[7];
  j.nev = f[8];
  j.rn = f[9];
  j.r0 = f[10];
  j.replace = f[11];
  j.marked = f[12];
  j.calm = f[13];
  j.phase = f[14];
  j.pre = (int32_t)f[15];
  return j;
}

// A node id, its free list's next entry read by the caller (fh, fh_next).
__device__ __forceinline__ int32_t take_node(const Ptrs& P, St& s, int32_t fh, uint32_t fh_next) {
  if (fh >= 0 && s.free_head == fh) {
    s.free_head = (int32_t)fh_next;
    s.nnodes += 1;
    return fh;
  }
  return node_alloc(P, s);
}

// Prefix marks of node c: phase and length in one store (a match may read
// them meanwhile).
__device__ __forceinline__ void put_marks(const Ptrs& P, int32_t c, uint32_t phase, int32_t ma) {
  if (lane_id() == 0)
    __hip_atomic_store(reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(P.nodes + c) + offsetof(NodeRec, mphase)), ((uint64_t)(uint32_t)ma << 32) | phase,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One edge of Algorithm 1's marking walk: the first cov tokens of node c's
// edge (record nc) join the marking set, with the reset to the current token
// when it would exceed B; a candidate whose leaf token is marked leaves U.
// `leaf`: c is (or, before this insertion, was) a leaf.
__device__ __forceinline__ void mark_edge(const Ptrs& P, St& s, uint32_t B, int32_t c, const NodeRec& nc, int32_t cov,
                                          bool leaf) {
  const bool was_cand = leaf && !is_marked(s, nc, c, nc.len - 1);
  int32_t ma = (nc.mphase == s.phase) ? nc.ma : 0;
  bool rv = (s.rphase == s.phase) && (s.rnode == c);
  const int32_t rlo = s.rlo, rhi = s.rhi;
  if (rv && rlo <= ma) {  // the reset interval touches the prefix: merge
    ma = ma > rhi ? ma : rhi;
    rv = false;
    s.rphase = 0;
  }
  const int32_t m1 = ma < cov ? ma : cov;
  int32_t m2 = 0;
  if (rv) {
    const int32_t e = rhi < cov ? rhi : cov;
    m2 = e - rlo > 0 ? e - rlo : 0;
  }
  const int32_t newly = cov - m1 - m2;
  if (s.cnt + (uint32_t)newly <= B) {
    s.cnt += (uint32_t)newly;
    int32_t nma = ma > cov ? ma : cov;
    if (rv && rlo <= nma) {
      nma = nma > rhi ? nma : rhi;
      s.rphase = 0;
    }
    put_marks(P, c, s.phase, nma);
  } else {
    // |T| reaches B+1 at the `need`-th newly marked position of this edge
    const int32_t need = (int32_t)(B + 1u - s.cnt);
    int32_t rp;
    if (!rv) {
      rp = ma + need - 1;
    } else {
      const int32_t e1 = rlo < cov ? rlo : cov;
      const int32_t s1 = e1 - ma > 0 ? e1 - ma : 0;
      rp = need <= s1 ? ma + need - 1 : rhi + (need - s1) - 1;
    }
    s.phase += 1;
    s.U_valid = 0;
    s.cnt = (uint32_t)(cov - rp);
    if (rp == 0) {
      put_marks(P, c, s.phase, cov);
    } else {
      s.rnode = c;
      s.rlo = rp;
      s.rhi = cov;
      s.rphase = s.phase;
    }
  }
  if (was_cand && s.U_valid && cov == nc.len) {
    const int32_t pos = arr_find(P.U, s.nU, c);
    if (pos >= 0) {
      arr_erase(P.U, s.nU, (uint32_t)pos);
      s.nU -= 1;
    }
  }
}

// Split node x (record nx, read in semispace sel_read) at edge offset k: a new
// head node takes positions [0, k) and x keeps the rest below it, so every
// leaf keeps its id.  The head's child array, with room for the leaf that
// the insertion adds, and its record are returned; the head's id, or -1.
__device__ __forceinline__ int32_t split_for_leaf(const Ptrs& P, St& s, int32_t x, NodeRec nx, int32_t k, int32_t fh,
                                                  uint32_t fh_next, NodeRec& nh) {
  const uint32_t sel_read = s.arena_sel;
  uint32_t coff;
  if (!arena_alloc(P, s, 4u, true, coff)) return -1;
  const int32_t hd = take_node(P, s, fh, fh_next);
  if (hd < 0) return -1;
  if (s.arena_sel != sel_read) nx = load_node(P.nodes, x);  // a collection has moved it
  int32_t* ar = arena_of(P, s.arena_sel);
  const int32_t tail_tok = uni(ar[nx.off + (uint32_t)k]);
  const NodeRec np = load_node(P.nodes, nx.parent);
  nh.parent = nx.parent;
  nh.off = nx.off;
  nh.len = k;
  nh.nchild = 1;
  nh.coff = coff;
  nh.ccap = 2;
  nh.mphase = nx.mphase;
  nh.ma = nx.ma < k ? nx.ma : k;
  uint32_t tphase = nx.mphase;
  int32_t tma = nx.ma - k > 0 ? nx.ma - k : 0;
  if (s.rnode == x) {
    if (s.rphase != s.phase) {
      s.rphase = 0;
    } else if (s.rhi <= k) {
      s.rnode = hd;
    } else if (s.rlo >= k) {
      s.rlo -= k;
      s.rhi -= k;
    } else {
      const int32_t t = s.rhi - k;
      s.rnode = hd;
      s.rhi = k;
      if (tphase == s.phase) {
        tma = tma > t ? tma : t;
      } else {
        tphase = s.phase;
        tma = t;
      }
    }
  }
  const int32_t pos = child_slot(ar, np, x);
  if (pos < 0) {
    KVR_FAIL_CHECK(s, 3, x, nx.parent, hd);
    return -1;
  }
  if (lane_id() == 0) {
    ar[coff] = tail_tok;
    ar[coff + 1] = x;
    ar[np.coff + 2 * pos + 1] = hd;
    P.nodes[hd] = nh;
    P.nodes[x].parent = hd;
    P.nodes[x].off = nx.off + (uint32_t)k;
    P.nodes[x].len = nx.len - k;
    P.nodes[x].mphase = tphase;
    P.nodes[x].ma = tma;
  }
  return hd;
}

// The rare ways of a load, out of line so that the common
// one keeps its state in registers; St goes through the worker's words in LDS.

// A path too deep for a trail: walk it by child lookups and mark it; the node
// its cached part ends in and that node's start, or -1.
__device__ __noinline__ int32_t mark_by_lookup(Ptrs P, uint32_t* state, uint32_t B, const int32_t* q, int32_t h,
                                               int32_t* start, int64_t* fail) {
  St s = load_st_lds(state);
  const int32_t* ar = arena_of(P, s.arena_sel);
  int32_t d = 0, last = 0;
  NodeRec nx = load_node(P.nodes, 0);
  while (d < h) {
    const int32_t c = uni(child_find(ar, nx, uni(q[d])));
    if (c <= 0 || (uint32_t)c >= s.hwm) {
      KVR_FAIL_CHECK(s, 1, last, d, h);
      last = -1;
      break;
    }
    nx = load_node(P.nodes, c);
    const int32_t cov = nx.len < h - d ? nx.len : h - d;
    if (cov <= 0) {
      KVR_FAIL_CHECK(s, 2, c, nx.len, d);
      last = -1;
      break;
    }
    mark_edge(P, s, B, c, nx, cov, nx.nchild == 0);
    last = c;
    *start = d;
    d += cov;
  }
  wave_mem_sync();  // the marks above are read again below
  store_st_lds(state, s);
  fail[0] = s.dbg_check;
  fail[1] = s.dbg_val[0];
  fail[2] = s.dbg_val[1];
  fail[3] = s.dbg_val[2];
  return last;
}

// Split the edge of node x (split_for_leaf), with its head's child array at
// *coff; the head, or -1.
__device__ __noinline__ int32_t split_out_of_line(Ptrs P, uint32_t* state, int32_t x, int32_t k, uint32_t* coff,
                                                  uint32_t* err, int64_t* fail) {
  St s = load_st_lds(state);
  NodeRec nh;
  nh.coff = 0;
  const int32_t fh = s.free_head;
  uint32_t fh_next = 0;
  if (fh >= 0) fh_next = uni(P.nodes[fh].off);
  const int32_t hd = split_for_leaf(P, s, x, load_node(P.nodes, x), k, fh, fh_next, nh);
  wave_mem_sync();
  store_st_lds(state, s);
  *coff = nh.coff;
  *err = s.err;
  fail[0] = s.dbg_check;
  fail[1] = s.dbg_val[0];
  fail[2] = s.dbg_val[1];
  fail[3] = s.dbg_val[2];
  return hd;
}

// Where an insertion's cached part ends: entry e of the trail (-1: at the root),
// node `last`, whose edge starts at `start`; and what the load needs from memory
// in one read (lanes 0-7: that node's record, lane 8: the free list's next
// entry).
struct LeafPlace {
  int32_t count, e, last, start, end, fh;
  int32_t words;
};

__device__ __forceinline__ LeafPlace find_place(const Ptrs& P, const uint32_t* state, const int32_t* t, int32_t h) {
  LeafPlace w;
  const TrailView v = view_trail(t);
  w.fh = uni((int32_t)state[4]);
  w.count = v.count;
  w.e = -1;
  w.last = w.start = w.end = 0;
  if (h > 0 && v.count <= kPathMax) {
    w.e = v.at(h);
    if (w.e >= 0) {
      w.last = v.node(w.e);
      w.start = v.start(w.e);
      w.end = v.end(w.e);
    }
  }
  const bool fl = lane_id() >= 8 && w.fh >= 0;
  const int32_t* p = reinterpret_cast<const int32_t*>(P.nodes + (fl ? w.fh : w.last));
  w.words = p[fl ? 1 : (lane_id() & 7)];
  return w;
}

// The load of the planned insertion of q[0, job.L) (in LDS) into the worker's
// cache (job.h = LCP(q, cache), t = the trail of that match, s = the worker's
// state, of which `state` holds a copy): the split of the edge the match ends in
// and q[h, L) as one new leaf.  t then holds q's trail in the updated cache.
// The marks, the leaf list and the evictions are left, except that a path too
// deep for a trail is marked here.  Fills job's l, a, tok, replace and marked;
// split = the node whose edge was split (its head is job.a), or 0.  KVR_DEV_*
// bits (0: done).
__device__ __forceinline__ uint32_t load_leaf(const Ptrs& P, St& s, uint32_t* state, uint32_t B, const int32_t* q,
                                              int32_t* t, PipeJob& job, int32_t& split) {
  const int32_t h = job.h, L = job.L;
  const LeafPlace w = find_place(P, state, t, h);
  int32_t last = w.last, start = w.start;
  bool read = true;  // w.words are of the node the leaf hangs from
  split = 0;
  if (h > 0 && w.count <= kPathMax && (w.e < 0 || w.end < h || last <= 0 || (uint32_t)last >= s.hwm)) {
    KVR_FAIL_CHECK(s, 1, w.e, h, last);
    return s.err;
  }
  const uint32_t nload = (uint32_t)(L - h);
  job.l = job.a = job.tok = 0;
  job.replace = job.marked = 0;
  int32_t pc = w.count <= kPathMax ? w.e + 1 : kPathMax + 1;
  if (h > 0 && (pc > kPathMax || (pc == kPathMax && h < L))) {
    // no trail, or none after this insertion
    int64_t fail[4];
    int32_t at = 0;
    last = uni(mark_by_lookup(P, state, B, q, h, &at, fail));
    start = uni(at);
    s = load_st_lds(state);
    if (last < 0) {
      KVR_FAIL_CHECK(s, (int32_t)fail[0], fail[1], fail[2], fail[3]);
      return s.err;
    }
    pc = kPathMax + 1;
    read = false;
    job.marked = 1;
  }
  if (h < L) {
    int32_t len, known[3];
    int32_t fh = w.fh;
    uint32_t fh_next;
    if (KVR_WAVE == 1 || !read) {
      const NodeRec lr = load_node(P.nodes, last);
      len = lr.len;
      known[0] = lr.nchild;
      known[1] = lr.ccap;
      known[2] = (int32_t)lr.coff;
      fh_next = fh >= 0 ? uni(P.nodes[fh].off) : 0u;
    } else {
      len = __builtin_amdgcn_readlane(w.words, 2);
      known[0] = __builtin_amdgcn_readlane(w.words, 3);
      known[2] = __builtin_amdgcn_readlane(w.words, 4);
      known[1] = __builtin_amdgcn_readlane(w.words, 5);
      fh_next = (uint32_t)__builtin_amdgcn_readlane(w.words, KVR_WAVE == 1 ? 0 : 8);
    }
    int32_t a = last;
    uint32_t sel = s.arena_sel;
    if (last != 0 && h - start < len) {
      int64_t fail[4];
      uint32_t coff, err;
      store_st_lds(state, s);
      wave_mem_sync();
      a = uni(split_out_of_line(P, state, last, h - start, &coff, &err, fail));
      s = load_st_lds(state);
      if (a < 0) {
        s.err = uni(err) ? uni(err) : (uint32_t)KVR_DEV_INTERNAL;
        s.dbg_check = (int32_t)fail[0];
        s.dbg_val[0] = fail[1];
        s.dbg_val[1] = fail[2];
        s.dbg_val[2] = fail[3];
        return s.err;
      }
      split = last;
      fh = -1;
      sel = s.arena_sel;
      known[0] = 1;
      known[1] = 2;
      known[2] = (int32_t)uni(coff);
    }
    // the walked part ends here (its last entry may have ended deeper: a split
    // edge, or one trimmed since)
    if (pc > 0 && pc <= kPathMax && lane_id() == 0) {
      trail_node(t)[pc - 1] = a;
      trail_end(t)[pc - 1] = h;
    }
    job.replace = a != 0 && known[0] == 0;
    uint32_t eoff;
    if (!place_edge(P, s, nload, (uint32_t)h, eoff)) return s.err;
    // no fence: nothing reads the new edge's words before the fence that
    // ends this half (a collection fences first)
    copy_words(arena_of(P, s.arena_sel), eoff, q, h, (int32_t)nload);
    const int32_t l = take_node(P, s, fh, fh_next);
    if (l < 0) return s.err;
    if (lane_id() == 0) {
      NodeRec nl;
      nl.parent = a;
      nl.off = eoff;
      nl.len = (int32_t)nload;
      nl.nchild = 0;
      nl.coff = 0;
      nl.ccap = 0;
      nl.mphase = 0;
      nl.ma = 0;
      P.nodes[l] = nl;
    }
    job.tok = uni(q[h]);
    if (!child_add(P, s, a, job.tok, l, known, sel, false)) return s.err;
    job.l = l;
    job.a = a;
    if (pc <= kPathMax) trail_add(t, pc, l, L);
  }
  if (lane_id() == 0) t[0] = pc;
  wave_mem_sync();
  return 0;
}

// ---------------------------------------------------------------- insertion, after the load

// The marking walk over the cached part of the path, along its trail in the
// updated tree (the records of all its nodes loaded at once, one lane each).
__device__ __forceinline__ void mark_cached(const Ptrs& P, St& s, uint32_t B, const PipeJob& job, const int32_t* t) {
  const int32_t pc = uni(t[0]);
  NodeRec pre;
  pre.parent = pre.len = pre.nchild = pre.ccap = pre.ma = 0;
  pre.off = pre.coff = pre.mphase = 0;
  if (KVR_WAVE >= kPathMax && lane_id() < pc) pre = P.nodes[trail_node(t)[lane_id()]];
  int32_t d = 0;
  for (int32_t e = 0; e < pc && d < job.h; ++e) {
    const int32_t c = uni(trail_node(t)[e]);
    const NodeRec nc = KVR_WAVE >= kPathMax ? node_from_lane(pre, e) : P.nodes[c];
    const int32_t cov = nc.len < job.h - d ? nc.len : job.h - d;
    if (c <= 0 || (uint32_t)c >= s.hwm || cov <= 0) {
      KVR_FAIL_CHECK(s, 2, c, nc.len, d);
      return;
    }
    mark_edge(P, s, B, c, nc, cov, nc.nchild == 0 || (job.replace && c == job.a));
    d += cov;
  }
  if (d < job.h) KVR_FAIL_CHECK(s, 1, pc, d, job.h);
  wave_mem_sync();  // the marks above are read again below
}

// Is a match of query m on the worker of an insertion (of query job.k < m), taken
// before its evictions end, the match that they leave?  They only remove tokens, so it never grows; it is
// as long as it was while its last token stays:
//   * a token of the inserted path stays (that path's leaf is no candidate,
//     and an eviction takes leaf tokens only): h <= on_path, a lower bound of the
//     LCP of the two queries;
//   * a token of the last match taken here stays (that one was final), so a
//     match that read no node is final;
//   * a token marked in the current phase stays while no new phase starts
//     (job.calm): |T| stays at most B, as at most L tokens join, and U never
//     runs empty, since of the |S| - |T| unmarked tokens only those of one path,
//     left unmarked above the token that started a phase, can stay internal.
// The evictions may run meanwhile.  What they change on the way of a match
// that this accepts is the child arrays of its nodes, where a removed entry's
// slot takes a copy of the last entry before the count drops, so a child that
// stays is always found.
__device__ __forceinline__ bool match_stays(const NodeRec* nodes, const PipeJob& job, int32_t h, int32_t on_path,
                                            bool walked, const MatchEnd& me) {
  if (job.nev == 0 || !walked || h <= on_path || h == 0) return true;
  if (!job.calm || me.node == 0) return false;
  // the phase and length of the node's prefix marks, written together
  const uint64_t m = __hip_atomic_load(reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(nodes + me.node) + offsetof(NodeRec, mphase)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
  return uni((uint32_t)m) == job.phase && uni((int32_t)(m >> 32)) >= me.pos;
}

// ---------------------------------------------------------------- the order of matches and insertions
// A worker's matches and insertions are ordered by its state word: the number
// of queries matched on it, and below it five flags.  A wave takes the match of
// query m by exchanging (m, no reader) for (m, reader), so each match is taken
// once and in order.  The routing wave sets the owner flag and waits for a
// reader before it hands the insertion over; once the leaf is loaded (loaded
// flag), matches go on beside the evictions: the next query's at once, later ones after the
// marks (marked flag), which read the trail that the match after the next
// writes.  One that the evictions could still change is put off (deferred
// flag) until they end and the owner's flags are cleared.

constexpr uint32_t kReader = 1u, kOwner = 2u, kLoaded = 4u, kMarked = 8u, kDeferred = 16u;
constexpr uint32_t kCountShift = 5;
constexpr uint32_t kCountMask = 0x7ffffffu;  // counts are compared modulo 2^27
// Insertions between routing and the end of their evictions, at most:
// insertion k has its record in slot k % kJobs.
constexpr uint32_t kJobs = 8;

// May the match of query m be taken on a worker in this state, owned (if so)
// by the insertion of query k?  (nbuf: how many queries have a trail.)  Beside
// an insertion, not for a query past k + kJobs: the match reads the insertion's
// record when its walk is over, which may be after the evictions, and the slot
// is written again when query k + kJobs is routed.  That needs this worker's
// match of k + kJobs, which is taken after this one or is this one.
__device__ __forceinline__ bool can_match(uint32_t sv, uint32_t m, uint32_t k, uint32_t nbuf) {
  const uint32_t c = m << kCountShift;
  if (sv == c) return true;
  const uint32_t ahead = m - k;
  return (sv == (c | kOwner | kLoaded | kMarked) && ahead <= kJobs) || (sv == (c | kOwner | kLoaded) && ahead < nbuf);
}

// Take the match that state sv allows; false when another wave was first.  (An
// acquire: the word may have gone through another insertion and come back to sv
// since it was read.)
__device__ __forceinline__ bool claim_match(uint32_t* st, uint32_t sv) {
  uint32_t old = sv;
  if (lane_id() == 0)
    __hip_atomic_compare_exchange_strong(st, &old, sv | kReader, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
  return uni(old) == sv;
}

// What matches read and write besides the trees (LDS).
struct MatchArea {
  uint32_t W, nbuf;
  const int32_t* q;      // the first query buffer
  uint32_t qstride;
  const int32_t* len;    // length of q_k in slot k & 7
  const int32_t* ell;    // LCP(q_k, q_k+1) in slot k & 7
  int32_t* h;            // h of q_k on worker w at [query_slot(k) * kMaxWorkers + w]
  int32_t* trail;        // [nbuf][W][kTrailWords]
  const uint32_t* tree;  // kStWords per worker
  const uint32_t* rootf;
  uint32_t* state;       // state words
  const uint32_t* owner; // the insertion that owns a worker
  const PipeJob* jobs;
  unsigned long long* mtok;  // matched tokens per worker
};

// Take the (claimed) match of query m on worker w (P), whose state was sv.
template <int kU>
__device__ __forceinline__ void take_match(const MatchArea& a, const Ptrs& P, uint32_t m, uint32_t w, uint32_t sv) {
  const uint32_t mp = query_slot(m, a.nbuf), mq = query_slot(m + a.nbuf - 1u, a.nbuf);  // its slot, the last one's
  int32_t* hp = a.h + mp * kMaxWorkers + w;
  const int32_t h_old = uni(a.h[mq * kMaxWorkers + w]);
  const int32_t ell = m > 0u ? uni(a.ell[(m - 1u) & 7u]) : 0;
  MatchEnd me{};
  bool walked = false;
  const int32_t h = match_ahead<kU>(P.nodes, arena_of(P, uni(a.tree[w * kStWords + 12])), a.rootf + w * kRootFilterWords,
                                    P.A, a.q + mp * a.qstride, uni(a.len[m & 7u]), h_old, ell,
                                    a.trail + (mq * a.W + w) * kTrailWords, a.trail + (mp * a.W + w) * kTrailWords,
                                    walked, me);
  bool stays = true;
  if (sv & kOwner) {
    // beside the evictions of an earlier query's insertion: this match
    // and the inserted path agree at least up to the LCPs in between
    const uint32_t k = uni(a.owner[w]);
    int32_t on_path = k + 1u == m ? ell : 0;
    if (k + 2u == m) {
      const int32_t e0 = uni(a.ell[k & 7u]);
      on_path = e0 < ell ? e0 : ell;
    }
    stays = match_stays(P.nodes, load_job(&a.jobs[k % kJobs]), h, on_path, walked, me);
  }
  if (stays && lane_id() == 0) {
    *hp = h;
    atomicAdd(&a.mtok[w], (unsigned long long)(uint32_t)h);
  }
  uint32_t* st = &a.state[w];
  if (stays) {  // one more query matched, and no reader
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane_id() == 0)
      __hip_atomic_fetch_add(st, (1u << kCountShift) - kReader, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  } else if (lane_id() == 0) {
    // put off until the owner is done, or to be taken again if it just was
    uint32_t old = sv | kReader;
    if (!__hip_atomic_compare_exchange_strong(st, &old, sv | kDeferred, __ATOMIC_RELEASE, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP))
      __hip_atomic_fetch_and(st, ~kReader, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// Is the match of query m on worker w zero without a look at the tree?  (As
// match_ahead finds it: no cached path starts with its first token, or the query
// before shares a token with it and has none cached here.)
__device__ __forceinline__ bool zero_match(const MatchArea& a, uint32_t m, uint32_t w) {
  const int32_t ell = m > 0u ? a.ell[(m - 1u) & 7u] : 0;
  const int32_t count = a.trail[(query_slot(m + a.nbuf - 1u, a.nbuf) * a.W + w) * kTrailWords];
  if (ell > 0 && count <= kPathMax) return count == 0;
  return !rf_may(a.rootf + w * kRootFilterWords, a.q[query_slot(m, a.nbuf) * a.qstride]);
}

// Take the match of query m on worker w, whose state is sv and allows it, if it is
// zero.  One lane's work: the lanes of a wave do so for as many workers at once,
// where a wave takes any other match alone.
__device__ __forceinline__ bool take_zero_match(const MatchArea& a, uint32_t m, uint32_t w, uint32_t sv) {
  uint32_t* st = &a.state[w];
  uint32_t old = sv;
  if (!zero_match(a, m, w) ||
      !__hip_atomic_compare_exchange_strong(st, &old, sv | kReader, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_WORKGROUP))
    return false;
  if (!zero_match(a, m, w)) {  // (the word may have come back to sv since it was read)
    __hip_atomic_fetch_and(st, ~kReader, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    return false;
  }
  const uint32_t mp = query_slot(m, a.nbuf);
  a.h[mp * kMaxWorkers + w] = 0;
  a.trail[(mp * a.W + w) * kTrailWords] = 0;
  __hip_atomic_fetch_add(st, (1u << kCountShift) - kReader, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  return true;
}

// What the routing wave knows of the insertion of a path of L tokens with h
// cached into a worker with this state (which nothing changes until the load).
__device__ __forceinline__ void plan_insertion(PipeJob& job, const uint32_t* state, uint32_t B, uint32_t maxL, int32_t h,
                                               int32_t L) {
  const uint32_t phase = uni(state[0]), cnt = uni(state[1]), size = uni(state[2]);
  const uint32_t nload = (uint32_t)(L - h);
  job.h = h;
  job.L = L;
  job.nfree = B - size;
  job.nev = nload > job.nfree ? nload - job.nfree : 0u;
  job.phase = phase;
  job.calm = (uint64_t)cnt + (uint32_t)L <= B && (uint64_t)size >= (uint64_t)cnt + (uint32_t)h + job.nev + maxL;
}

// The match of the next query on the worker of an insertion that has been
// planned but not loaded, from the match taken on the tree as it is (h_pre, its
// trail in tn; ell = LCP of the two queries).  The load adds the inserted path's
// prefixes only, so h = max(h_pre, ell) and the tree need not be walked again;
// `stays` as match_stays says.
__device__ __forceinline__ int32_t match_before_load(const NodeRec* nodes, const PipeJob& job, int32_t h_pre,
                                                     int32_t ell, const int32_t* tn, bool& stays) {
  stays = true;
  if (h_pre <= ell) return ell;
  if (job.nev == 0) return h_pre;
  MatchEnd me{0, 0};
  const TrailView v = view_trail(tn);
  if (v.count > 0 && v.count <= kPathMax) {
    me.node = v.node(v.count - 1);
    me.pos = h_pre - v.start(v.count - 1);
  }
  stays = match_stays(nodes, job, h_pre, ell, true, me);
  return h_pre;
}

// That match's trail after the load (tk = the trail of the inserted query):
// where the next query leaves the inserted path, that path's trail up to there;
// else its own, with the head of the split edge (which both pass, as then ell is
// the depth of the split) in front of the split node.
__device__ __forceinline__ void trail_after_load(const PipeJob& job, int32_t split, int32_t h_pre, int32_t ell,
                                                 const int32_t* tk, int32_t* tn) {
  if (h_pre <= ell) {
    const TrailView k = view_trail(tk);
    int32_t pc = k.count;
    if (pc <= kPathMax) {
      pc = ell > 0 ? k.at(ell) + 1 : 0;
      k.copy_to(tn, pc);
    }
    if (lane_id() == 0) tn[0] = pc;
    return;
  }
  if (split <= 0) return;
  const TrailView v = view_trail(tn);
  if (v.count > kPathMax) return;
  int32_t at = -1;
  if (KVR_WAVE == 1) {
    for (int32_t e = 0; e < v.count; ++e)
      if (v.node(e) == split) at = e;
  } else {
    const uint64_t m = __ballot(lane_id() < v.count && v.vnode == split);
    if (m) at = first_lane(m);
  }
  if (at < 0) return;
  if (v.count < kPathMax) {
    // entries from `at` on move up by one
    if (KVR_WAVE == 1) {
      for (int32_t e = v.count - 1; e >= at; --e) {
        tn[1 + e + 1] = v.node(e);
        tn[1 + kPathMax + e + 1] = v.end(e);
      }
    } else if (lane_id() >= at && lane_id() < v.count) {
      tn[1 + lane_id() + 1] = v.vnode;
      tn[1 + kPathMax + lane_id() + 1] = v.vend;
    }
    if (lane_id() == 0) {
      trail_node(tn)[at] = job.a;
      trail_end(tn)[at] = job.h;
    }
  }
  if (lane_id() == 0) tn[0] = v.count + 1;  // (kPathMax + 1 is "unknown")
}

// Rank in the leaf list of the leaf that an insertion added (its entry still
// missing from the list): the place of its parent when that was a leaf, else
// next to its neighbours among the parent's children.  -1: an inconsistency.
__device__ __forceinline__ int32_t rank_of_leaf(const Ptrs& P, uint32_t hwm, uint32_t nleaves, const int32_t* ar,
                                                const PipeJob& job) {
  int32_t x = job.a;
  bool after = false;
  if (!job.replace) {
    const NodeRec na = load_node(P.nodes, job.a);
    x = uni(child_neighbor(ar, na, job.tok, true));
    after = x >= 0;
    if (!after) x = uni(child_neighbor(ar, na, job.tok, false));
    if (x < 0) return 0;  // the only leaf
    // down to the last (first) leaf of that child's subtree
    for (uint32_t steps = 0; steps <= hwm; ++steps) {
      if (x <= 0 || (uint32_t)x >= hwm) return -1;
      const NodeRec nx = load_node(P.nodes, x);
      if (nx.nchild == 0) break;
      x = uni(after ? child_neighbor(ar, nx, (int64_t)1 << 32, true) : child_neighbor(ar, nx, -1, false));
    }
  }
  const int32_t pos = arr_find(P.leaf, nleaves, x);
  return pos < 0 ? -1 : (after ? pos + 1 : pos);
}

// ---------------------------------------------------------------- completions and decay

// The LBGR state of the replica's workers in LDS, one lane per worker.
struct LbgrLds {
  double* P;          // load estimate
  double* theta;      // [4][W] residual model
  int64_t* Wb;        // observed-latency backlog
  int64_t* done_at;   // completion time of the oldest pending record (INT64_MAX: none)
  uint32_t* head;     // pending ring
  uint32_t* count;
  uint32_t* size;     // |S| once the insertions routed so far are done
  uint32_t W;
};
constexpr uint32_t kLbgrBytes = 8 * 7 + 4 * 3;  // per worker

constexpr int64_t kNever = 0x7fffffffffffffffll;

// Completions with t_done <= t of worker w (FIFO), then decay to t and drain
// the observed-latency backlog.  tick, tick_prev = t / dt and tprev / dt.
__device__ __forceinline__ void decay_lds(const Consts& C, const LbgrLds& b, uint32_t w, WorkerHdr* hdr,
                                          const PendRec* pend, uint32_t PC, int64_t t, int64_t tprev, int64_t tick,
                                          int64_t tick_prev) {
  double Pl = b.P[w];
  int64_t at = b.done_at[w], tl = tick_prev;
  if (at <= t) {
    uint32_t head = b.head[w], cnt = b.count[w];
    double theta[4];
    for (int a = 0; a < 4; ++a) theta[a] = b.theta[a * b.W + w];
    uint64_t done = 0;
    do {
      const uint32_t next = head + 1 == PC ? 0u : head + 1;
      const PendRec pr = pend[head];
      const int64_t at2 = pend[next].t_done;
      const int64_t td = pr.t_done / C.dt_us;
      Pl = Pl * pow_int(C.rho, (uint64_t)(td - tl));
      tl = td;
      const double rem = pr.chat * pow_int(C.rho, (uint64_t)(td - pr.t_route / C.dt_us));
      const double np = Pl - rem;
      Pl = np > 0.0 ? np : 0.0;
      double phi[4];
      phi[0] = (double)pr.h * 0.001;
      phi[1] = (double)(pr.L - pr.h) * 0.001;
      phi[2] = pr.x3;
      phi[3] = 1.0;
      double res = theta[0] * phi[0];
      res = res + theta[1] * phi[1];
      res = res + theta[2] * phi[2];
      res = res + theta[3] * phi[3];
      const double ehat_now = pr.base + res;
      const double e_obs = (double)(pr.t_done - pr.t_route) * 1e-6;
      online_update(C, theta, hdr->Pm, phi, e_obs - ehat_now);
      head = next;
      cnt -= 1;
      done += 1;
      at = cnt > 0 ? at2 : kNever;
    } while (at <= t);
    for (int a = 0; a < 4; ++a) b.theta[a * b.W + w] = theta[a];
    b.head[w] = head;
    b.count[w] = cnt;
    b.done_at[w] = at;
    __hip_atomic_fetch_add(&hdr->completions, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  b.P[w] = Pl * pow_int(C.rho, (uint64_t)(tick - tl));
  const int64_t nb = b.Wb[w] - (t - tprev);
  b.Wb[w] = nb > 0 ? nb : 0;
}

// commit_route on that state: the routed worker's lane adds the estimated
// service time to the load estimate, advances the observed-latency queue and
// queues the completion record.  The counters go to the header as atomics
// whose results nothing waits for.  KVR_DEV_* bits.
__device__ __forceinline__ uint32_t commit_lds(const Consts& C, const Ptrs& P, const LbgrLds& b, uint32_t w,
                                               const RouteView& v, double chat, int32_t h, int32_t L, int64_t t,
                                               int32_t olen) {
  WorkerHdr* hdr = P.hdr;
  b.P[w] = v.P + chat;
  const int64_t cost = C.true_cached_us * h + C.true_miss_us * (int64_t)(L - h) + C.true_out_us * (int64_t)olen;
  const int64_t e_us = v.Wb + cost;
  b.Wb[w] = e_us;
  uint32_t err = 0;
  if (v.pend_count >= P.PC) {
    err |= KVR_DEV_PENDING_FULL;
  } else {
    uint32_t slot = v.pend_head + v.pend_count;
    if (slot >= P.PC) slot -= P.PC;
    PendRec pr;
    pr.t_route = t;
    pr.t_done = t + e_us;
    pr.chat = chat;
    pr.base = chat + v.P;
    pr.x3 = v.P;
    pr.h = h;
    pr.L = L;
    P.pend[slot] = pr;
    b.count[w] = v.pend_count + 1u;
    if (v.pend_count == 0u) b.done_at[w] = pr.t_done;
    __hip_atomic_fetch_max(&hdr->pending_max, (uint64_t)(v.pend_count + 1u), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __hip_atomic_fetch_add(&hdr->routed, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __hip_atomic_fetch_add(&hdr->prompt_tokens, (uint64_t)L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __hip_atomic_fetch_add(&hdr->hit_tokens, (uint64_t)h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __hip_atomic_fetch_add(&hdr->lat_sum_us, (uint64_t)e_us, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __hip_atomic_fetch_max(&hdr->lat_max_us, (uint64_t)e_us, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return err;
}

}  // namespace kvr

#endif  // KVR_TRAIL_H
