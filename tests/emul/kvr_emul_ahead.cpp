// kvr_emul_ahead.cpp - sequential CPU replay of the pipelined step kernel's
// per-wave logic (kvr_trail.h, unchanged, one lane), in the orders that the
// kernel's waves can take it (tests only): the next query matched on every
// worker before this one is routed, the routed worker's match taken again
// after the load and, where that is not final, after the evictions, and the
// second halves of several insertions outstanding at once.  Which order is
// taken at each step comes from a seeded generator.
#include "emul_wave.h"

#include "../../paper_2601_18999_amd/csrc/kvr_trail.h"

#include <cstring>
#include <vector>

using namespace kvr;

namespace {

struct Hook {
  bool todo;
  PipeJob job;
  uint32_t* state;
  void before_list(const Ptrs& P, St& s) {
    if (!todo) return;
    todo = false;
    const int32_t pos = rank_of_leaf(P, s.hwm, s.nleaves, arena_of(P, s.arena_sel), job);
    if (pos < 0 || (uint32_t)pos > s.nleaves) {
      KVR_FAIL_CHECK(s, 4, pos, s.nleaves, job.a);
      return;
    }
    if (job.replace) {
      P.leaf[pos] = job.l;
    } else {
      arr_insert(P.leaf, s.nleaves, (uint32_t)pos, job.l, false);
      s.nleaves += 1;
    }
  }
  void keep(const Ptrs&, const St& s) { store_st_lds(state, s); }
  static constexpr bool kWordsMustCome = true;
  void words_late(St& s) { KVR_FAIL_CHECK(s, 7, job.k, job.worker, job.rn); }
};

}  // namespace

// counts: of the matches taken between an insertion's load and its evictions,
// [0] those of the next query that were final where the two queries part, [1]
// those final on marked tokens or a final match before, [2] those taken again
// after the evictions; [3] those of later queries than the next; of the matches
// taken before the load, [4] those that stood after it and [5] those put off
extern "C" int emul_ahead(const kvr_config* cfg, uint64_t n, const int32_t* tokens, const uint64_t* offsets,
                          const int64_t* arrival, const uint16_t* out_len, int32_t* route, int32_t* hits,
                          int32_t* all_hits, kvr_worker_stats* out, uint32_t ucap, uint64_t order_seed,
                          uint64_t* counts) {
  const Layout L = make_layout(*cfg);
  std::vector<uint64_t> mem((L.total + 255) / 8 + 32);
  char* ws = reinterpret_cast<char*>(((uintptr_t)mem.data() + 255) & ~(uintptr_t)255);
  Consts C{};
  C.seed = cfg->seed;
  C.alpha_cached = cfg->alpha_cached;
  C.alpha_miss = cfg->alpha_miss;
  C.rho = cfg->rho;
  C.lr = cfg->lr;
  C.nlms_eps = cfg->nlms_eps;
  C.rls_p0 = cfg->rls_p0;
  C.dt_us = cfg->decay_interval_us;
  C.true_cached_us = cfg->true_cached_us;
  C.true_miss_us = cfg->true_miss_us;
  C.true_out_us = cfg->true_out_us;
  C.update = cfg->update;
  C.router = KVR_ROUTE_LBGR;
  const uint32_t W = L.W, B = L.B;
  uint64_t rs = order_seed * 2 + 1;
  auto coin = [&](uint32_t m) {
    rs = rs * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)(rs >> 33) % m;
  };
  std::vector<int32_t> ubuf(4 * (size_t)(ucap ? ucap : 1));
  UStage us;
  us.node = ubuf.data();
  us.len = us.node + ucap;
  us.top = us.len + ucap;
  us.par = us.top + ucap;
  us.cap = ucap;
  // query buffers as the kernel has them: 16-byte aligned, padded
  const uint32_t qw = ((L.maxL + 3u) & ~3u) + 8u;
  std::vector<int4> qmem(3 * qw / 4 + 8);
  auto qbuf = [&](uint64_t k) { return reinterpret_cast<int32_t*>(qmem.data()) + (k % 3) * qw + 4; };
  for (uint32_t r = 0; r < L.R; ++r) {
    std::vector<uint32_t> tree((size_t)kStWords * W), rootf((size_t)kRootFilterWords * W);
    std::vector<int32_t> trail((size_t)3 * W * kTrailWords);
    std::vector<double> lbd(5 * W);
    std::vector<int64_t> lbi(2 * W);
    std::vector<uint32_t> lbu(3 * W);
    LbgrLds lb{lbd.data(), lbd.data() + W, lbi.data(), lbi.data() + W, lbu.data(), lbu.data() + W, lbu.data() + 2 * W, W};
    for (uint32_t i = 0; i < W; ++i) {
      const Ptrs P = worker_ptrs(ws, L, r, i);
      init_worker(P, cfg->rls_p0);
      std::memcpy(&tree[(size_t)i * kStWords], P.hdr, 4 * (kStWords - 1));
      lb.done_at[i] = kNever;
    }
    auto trail_of = [&](uint64_t k, uint32_t w) { return trail.data() + ((k % 3) * W + w) * kTrailWords; };
    auto len = [&](uint64_t k) { return (int32_t)(offsets[k + 1] - offsets[k]); };
    auto lcp = [&](uint64_t k) {  // of q_k and q_k+1
      const int32_t m = len(k) < len(k + 1) ? len(k) : len(k + 1);
      int32_t x = 0;
      while (x < m && tokens[offsets[k] + x] == tokens[offsets[k + 1] + x]) ++x;
      return x;
    };
    int32_t h[2][kMaxWorkers] = {}, h2[kMaxWorkers];
    bool ahead2[kMaxWorkers] = {};  // q_k+2 matched
    uint64_t matched[kMaxWorkers] = {};
    auto match = [&](uint64_t m, uint32_t w, int32_t h_old, bool& ended, MatchEnd& me) {
      const Ptrs P = worker_ptrs(ws, L, r, w);
      return match_ahead<2>(P.nodes, arena_of(P, tree[w * kStWords + 12]), &rootf[w * kRootFilterWords], P.A, qbuf(m),
                            len(m), h_old, m ? lcp(m - 1) : 0, trail_of(m + 2, w), trail_of(m, w), ended, me);
    };
    // outstanding second halves, at most one per worker
    std::vector<PipeJob> open;
    std::vector<uint32_t> rw;
    std::vector<St> after_marks(W);
    auto marks = [&](PipeJob& job) {
      if (job.pre) return;  // (a flag of this replay)
      job.pre = 1;
      after_marks[job.worker] = load_st_lds(&tree[job.worker * kStWords]);
      if (!job.marked)
        mark_cached(worker_ptrs(ws, L, r, job.worker), after_marks[job.worker], B, job, trail_of(job.k, job.worker));
    };
    auto second_half = [&](PipeJob job) -> uint32_t {
      const Ptrs P = worker_ptrs(ws, L, r, job.worker);
      marks(job);
      EvictJob ej;
      ej.s = after_marks[job.worker];
      if (ej.s.err) return ej.s.err;
      const uint32_t rn = job.nev - (job.nev ? coin(job.nev + 1) / 2 : 0);  // some words left to the evicting wave
      rw.resize(rn + 1);
      for (uint32_t d = 0; d < rn; ++d) rw[d] = (uint32_t)(philox_word0(job.k, job.worker, d, 0ull, C.seed, r) >> 32);
      ej.ia = InsertArgs{C.seed, job.k, job.worker, r, B, rn, rw.data(), nullptr, 0, 1, nullptr, nullptr};
      ej.h = job.h;
      ej.L = job.L;
      ej.l = job.l;
      ej.nfree = job.nfree;
      ej.nev = job.nev;
      ej.c0 = ej.s.cnt;
      ej.reset_at = job.h < job.L && ej.c0 + (uint32_t)(job.L - job.h) >= B + 1u ? job.h + (int32_t)(B - ej.c0) : -1;
      ej.worker = job.worker;
      ej.final_size = 0;
      Hook hook{job.h < job.L, job, &tree[job.worker * kStWords]};
      int64_t dbg[4];
      return rlt_evict<false>(P, ej, us, dbg, nullptr, 0, 0, hook);
    };
    for (uint64_t k = 0; k < n; ++k) {
      const int cur = (int)(k & 1);
      // stage up to q_k+2
      for (uint64_t s = k ? k + 2 : 0; s <= k + 2 && s < n; ++s)
        std::memcpy(qbuf(s), tokens + offsets[s], 4 * (size_t)len(s));
      bool ended;
      MatchEnd me;
      if (k == 0)
        for (uint32_t w = 0; w < W; ++w) matched[w] += h[0][w] = match(0, w, 0, ended, me);
      // q_k+1 on any worker without an insertion outstanding, before q_k is routed
      bool ahead[kMaxWorkers] = {};
      auto free_of = [&](uint32_t w) {
        for (const PipeJob& j : open)
          if (j.worker == w) return false;
        return true;
      };
      if (k + 1 < n)
        for (uint32_t w = 0; w < W; ++w)
          if (ahead2[w] || (free_of(w) && coin(4))) {
            h[cur ^ 1][w] = ahead2[w] ? h2[w] : match(k + 1, w, h[cur][w], ended, me);
            ahead[w] = true;
            ahead2[w] = false;
            if (k + 2 < n && free_of(w) && coin(3)) {
              h2[w] = match(k + 2, w, h[cur ^ 1][w], ended, me);
              ahead2[w] = true;
            }
          }
      // completions and decay, route, commit
      const int64_t tp = k ? arrival[k - 1] : 0;
      double eh[kMaxWorkers], ch[kMaxWorkers];
      RouteView v[kMaxWorkers];
      uint32_t best = 0;
      for (uint32_t w = 0; w < W; ++w) {
        const Ptrs P = worker_ptrs(ws, L, r, w);
        decay_lds(C, lb, w, P.hdr, P.pend, P.PC, arrival[k], tp, arrival[k] / C.dt_us, tp / C.dt_us);
        v[w] = RouteView{};
        v[w].P = lb.P[w];
        for (int x = 0; x < 4; ++x) v[w].theta[x] = lb.theta[x * W + w];
        v[w].Wb = lb.Wb[w];
        v[w].pend_head = lb.head[w];
        v[w].pend_count = lb.count[w];
        eh[w] = lbgr_score(C, v[w], h[cur][w], len(k), &ch[w]);
        if (eh[w] < eh[best]) best = w;
        if (all_hits) all_hits[(r * n + k) * W + w] = h[cur][w];
      }
      const Ptrs P = worker_ptrs(ws, L, r, best);
      uint32_t err = commit_lds(C, P, lb, best, v[best], ch[best], h[cur][best], len(k), arrival[k],
                                query_out_len(out_len, k));
      if (err) return (int)err;
      route[r * n + k] = (int32_t)best;
      hits[r * n + k] = h[cur][best];
      // the worker's earlier insertion finishes first; others as they like
      for (size_t x = 0; x < open.size();) {
        if (open[x].worker == best || coin(4) == 0 || open.size() >= 3) {
          if ((err = second_half(open[x]))) return (int)err;
          open.erase(open.begin() + (long)x);
        } else {
          ++x;
        }
      }
      // the insertion as planned before its load, and what it makes of a match of
      // q_k+1 taken on the tree as it is
      PipeJob job{};
      uint32_t* state = &tree[best * kStWords];
      plan_insertion(job, state, B, L.maxL, h[cur][best], len(k));
      job.k = (uint32_t)k;
      job.worker = best;
      bool stays = false;
      int32_t h_pre = 0, ha = 0;
      const bool pre = k + 1 < n && ahead[best];
      if (pre) {
        h_pre = h[cur ^ 1][best];
        ha = match_before_load(P.nodes, job, h_pre, lcp(k), trail_of(k + 1, best), stays);
      }
      // the load
      St s = load_st_lds(state);
      int32_t split;
      err = load_leaf(P, s, state, B, qbuf(k), trail_of(k, best), job, split);
      store_st_lds(state, s);
      if (err) return (int)err;
      if (h[cur][best] == 0) rf_add(&rootf[best * kRootFilterWords], job.tok);
      h[cur][best] = len(k);
      open.push_back(job);
      ahead2[best] = false;
      if (pre) {
        trail_after_load(job, split, h_pre, lcp(k), trail_of(k, best), trail_of(k + 1, best));
        const std::vector<int32_t> ta(trail_of(k + 1, best), trail_of(k + 1, best) + kTrailWords);
        const int32_t hw = match(k + 1, best, len(k), ended, me);
        if (ha != hw) return -9;
        const int32_t* tw = trail_of(k + 1, best);
        if (ta[0] <= kPathMax) {  // a trail that is kept is the one a walk finds
          if (ta[0] != tw[0]) return -10;
          for (int32_t x = 0; x < ta[0]; ++x)
            if (ta[1 + x] != tw[1 + x] || ta[1 + kPathMax + x] != tw[1 + kPathMax + x]) return -11;
        }
        std::memcpy(trail_of(k + 1, best), ta.data(), 4 * kTrailWords);
        h[cur ^ 1][best] = ha;
        if (!stays) ahead[best] = false;
        counts[4 + (stays ? 0 : 1)] += 1;
        if (stays && coin(2)) {  // and stays
          if ((err = second_half(open.back()))) return (int)err;
          open.pop_back();
          if (match(k + 1, best, len(k), ended, me) != ha) return -12;
          std::memcpy(trail_of(k + 1, best), ta.data(), 4 * kTrailWords);
        }
      }
      if (k + 1 == n) continue;
      // q_k+1 on the workers not done yet: beside an insertion that is outstanding,
      // or after its evictions where those could change it
      for (uint32_t w = 0; w < W; ++w) {
        if (!ahead[w]) {
          // (the match three queries on writes the trail that the marks read)
          for (PipeJob& j : open)
            if (j.worker == w && (j.k + 1 < k || coin(2))) marks(j);
          int32_t hn = match(k + 1, w, h[cur][w], ended, me);
          for (size_t x = 0; x < open.size(); ++x)
            if (open[x].worker == w) {
              const PipeJob j = open[x];
              int32_t on_path = j.k == k ? lcp(k) : 0;
              if (j.k + 1 == k) on_path = lcp(k) < lcp(j.k) ? lcp(k) : lcp(j.k);
              const bool stays = match_stays(worker_ptrs(ws, L, r, w).nodes, j, hn, on_path, ended, me);
              if (!stays || coin(3) == 0) {
                if ((err = second_half(j))) return (int)err;
                open.erase(open.begin() + (long)x);
                const int32_t hp = match(k + 1, w, h[cur][w], ended, me);
                if (stays && hp != hn) return -8;  // the early match was not final
                hn = hp;
              }
              counts[j.k < k ? 3 : !stays ? 2 : hn == lcp(k) ? 0 : 1] += 1;
              break;
            }
          h[cur ^ 1][w] = hn;
        }
        matched[w] += (uint64_t)h[cur ^ 1][w];
      }
    }
    for (const PipeJob& j : open)
      if (uint32_t err = second_half(j)) return (int)err;
    for (uint32_t w = 0; w < W; ++w) {
      const Ptrs P = worker_ptrs(ws, L, r, w);
      WorkerHdr* hd = P.hdr;
      std::memcpy(static_cast<void*>(hd), &tree[(size_t)w * kStWords], 4 * (kStWords - 1));
      hd->P = lb.P[w];
      for (int x = 0; x < 4; ++x) hd->theta[x] = lb.theta[x * W + w];
      hd->Wb = lb.Wb[w];
      hd->tl = n ? arrival[n - 1] : 0;
      hd->pend_head = lb.head[w];
      hd->pend_count = lb.count[w];
      hd->matched_tokens = matched[w];
      if (!worker_stats(P, out + (uint64_t)r * W + w)) return -7;
    }
  }
  return 0;
}
