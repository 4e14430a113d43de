// kvr_emul_waves.cpp - the waves of the pipelined step kernel on the CPU (tests
// only): a routing wave, two evicting waves and helpers as coroutines of one
// lane each, which run kvr_trail.h unchanged and hand over to one another at
// any atomic, fence or wave-uniform read, as a seeded generator says.  So a
// match is cut between its walk and its verdict, an insertion between any two
// of its steps, and any wave can be held back while the others go on for
// several queries (an insertion that outlasts the next seven).  Records,
// flags and draw words live in the kernel's rings, with its slots.
#include <cstdint>
static void emul_step();
#define KVR_EMUL_STEP() emul_step()
#include "emul_wave.h"

#include "../../paper_2601_18999_amd/csrc/kvr_trail.h"

#include <ucontext.h>

#include <cstring>
#include <functional>
#include <memory>
#include <vector>

using namespace kvr;

namespace {

// ---------------------------------------------------------------- coroutines
struct Actor {
  ucontext_t ctx;
  std::vector<char> stack;
  std::function<void()> body;
  uint32_t weight;
  uint32_t after;                 // steps of its own before it is held (0: none planned)
  std::function<bool()> release;  // held until this, or for kHold hand-overs
  uint64_t held_until;
  bool done;
};

struct Sched {
  static constexpr uint64_t kHold = 4000;
  std::vector<std::unique_ptr<Actor>> actors;
  ucontext_t main;
  Actor* now = nullptr;
  uint64_t rs = 1, switches = 0, until = 0;
  uint32_t rate = 8;
  bool hung = false;

  uint32_t coin(uint32_t m) {
    rs = rs * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)(rs >> 33) % m;
  }
  // Hold the running wave, after some steps, until release().
  void hold(uint32_t after, std::function<bool()> release) {
    now->after = after;
    now->release = std::move(release);
  }
  // the next wave to run; now and then other waves get slow or stand still
  void hand_over() {
    if (++switches > 40000000ull) hung = true;
    if (switches >= until) {
      // all alike but for some that stand still, or speeds at random
      static const uint32_t speeds[] = {0, 1, 8, 64};
      const uint32_t still = coin(4);
      until = switches + 20 + coin(still ? 20000 : 4000);
      for (auto& a : actors) a->weight = still ? 8 : speeds[coin(4)];
      for (uint32_t x = 0; x < still; ++x) actors[coin((uint32_t)actors.size())]->weight = 0;
    }
    uint32_t sum = 0, left = 0;
    std::vector<uint32_t> w;
    for (auto& a : actors) {
      if (a->held_until && (switches >= a->held_until || a->release())) a->held_until = 0;
      w.push_back(a->done || a->held_until ? 0 : a->weight);
      sum += w.back();
      left += !a->done;
    }
    if (left == 0) return;
    if (sum == 0) {  // all that could run stand still
      for (size_t x = 0; x < w.size(); ++x) w[x] = !actors[x]->done;
      sum = left;
    }
    uint32_t pick = coin(sum);
    size_t x = 0;
    while (pick >= w[x]) pick -= w[x++];
    Actor* next = actors[x].get();
    if (next == now) return;
    Actor* from = now;
    now = next;
    swapcontext(&from->ctx, &next->ctx);
  }
};

Sched* g_s = nullptr;

void entry() {
  Sched* s = g_s;
  Actor* me = s->now;
  me->body();
  me->done = true;
  bool left = false;
  for (auto& a : s->actors) left |= !a->done;
  if (!left) {
    s->now = nullptr;
    swapcontext(&me->ctx, &s->main);
  }
  for (;;) s->hand_over();
}

void run_all(Sched& s) {
  g_s = &s;
  for (auto& a : s.actors) {
    a->stack.resize(512 << 10);
    getcontext(&a->ctx);
    a->ctx.uc_stack.ss_sp = a->stack.data();
    a->ctx.uc_stack.ss_size = a->stack.size();
    a->ctx.uc_link = nullptr;
    makecontext(&a->ctx, entry, 0);
    a->done = false;
    a->weight = 1;
    a->after = 0;
    a->held_until = 0;
  }
  s.now = s.actors[0].get();
  swapcontext(&s.main, &s.now->ctx);
  g_s = nullptr;
}

void wait_step() {  // in a wait: another wave's turn
  if (g_s && g_s->now) g_s->hand_over();
}

}  // namespace

static void emul_step() {
  if (!g_s || !g_s->now) return;
  Actor* a = g_s->now;
  const bool held = a->after && --a->after == 0;
  if (held) a->held_until = g_s->switches + Sched::kHold;
  if (held || g_s->coin(g_s->rate) == 0) g_s->hand_over();
}

namespace {

constexpr uint32_t kEvictors = 2, kHelpers = 3;

struct Flags {
  uint32_t routed, fronts, staged, decayed, handed, ticket, end, stop;
};

struct WaveHook {
  bool todo;
  PipeJob job;
  const uint32_t* ready;
  const int32_t* rank;
  uint32_t* state;
  Flags* f;
  void before_list(const Ptrs& P, St& s) {
    if (!todo) return;
    todo = false;
    const uint32_t want = ((job.k + 1u) << 2) | 3u;
    while (*ready != want) {
      if (f->stop || g_s->hung) {
        KVR_FAIL_CHECK(s, 5, job.k, job.worker, 0);
        return;
      }
      wait_step();
    }
    const int32_t pos = *rank;
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

// hold_draws: one insertion in so many has its draws held back (0: none).
// counts: matches whose insertion (of query k) ended between the claim and the
// verdict, [0] in all, [1] of query k + 5 and later; [2] matches put off; [3]
// insertions that were open when the seventh after them was loaded; [4] matches
// beside an insertion that were accepted past the inserted path; [5] matches
// taken as zero
extern "C" int emul_waves(const kvr_config* cfg, uint64_t n64, const int32_t* tokens, const uint64_t* offsets,
                          const int64_t* arrival, const uint16_t* out_len, int32_t* route, int32_t* hits,
                          int32_t* all_hits, kvr_worker_stats* out, uint32_t ucap, uint32_t nbuf, int32_t router,
                          uint64_t order_seed, uint32_t hold_draws, uint64_t* counts) {
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
  const uint32_t W = L.W, B = L.B, n = (uint32_t)n64;
  const uint32_t qw = ((L.maxL + 3u) & ~3u) + 8u;
  for (uint32_t r = 0; r < L.R; ++r) {
    // ---- what the kernel keeps in LDS
    std::vector<int4> qmem(nbuf * qw / 4 + 8);
    int32_t* q0 = reinterpret_cast<int32_t*>(qmem.data()) + 4;
    std::vector<uint32_t> tree((size_t)kStWords * W), rootf((size_t)kRootFilterWords * W), state(W), owner(W);
    std::vector<int32_t> trail((size_t)nbuf * W * kTrailWords), h(4 * kMaxWorkers);
    std::vector<unsigned long long> mtok(W);
    std::vector<double> lbd(5 * W);
    std::vector<int64_t> lbi(2 * W);
    std::vector<uint32_t> lbu(3 * W);
    LbgrLds lb{lbd.data(), lbd.data() + W, lbi.data(), lbi.data() + W, lbu.data(), lbu.data() + W, lbu.data() + 2 * W, W};
    int32_t ell[8], len[8] = {}, olen[8] = {}, hit[kJobs] = {}, rank[kJobs] = {};
    int64_t arr[8] = {};
    PipeJob jobs[kJobs] = {};
    uint32_t jdone[kJobs] = {}, best_of[kJobs] = {}, rank_ready[kJobs] = {}, prog[kJobs][16] = {};
    uint64_t rn_of[kJobs] = {};
    uint32_t reader_held[kJobs] = {};  // k + 1: a match beside insertion k is held back
    std::vector<uint32_t> words((size_t)kJobs * L.maxL);
    Flags f{};
    uint32_t err = 0;
    for (int32_t& e : ell) e = 0x7fffffff;
    for (uint32_t i = 0; i < W; ++i) {
      const Ptrs P = worker_ptrs(ws, L, r, i);
      init_worker(P, cfg->rls_p0);
      std::memcpy(&tree[(size_t)i * kStWords], P.hdr, 4 * (kStWords - 1));
      lb.done_at[i] = kNever;
    }
    const auto fail = [&](uint32_t e) {
      if (!err) err = e ? e : 1u << 30;
      f.stop = 1;
    };
    const auto stopped = [&] { return f.stop || g_s->hung; };
    MatchArea ma;
    ma.W = W;
    ma.nbuf = nbuf;
    ma.q = q0;
    ma.qstride = qw;
    ma.len = len;
    ma.ell = ell;
    ma.h = h.data();
    ma.trail = trail.data();
    ma.tree = tree.data();
    ma.rootf = rootf.data();
    ma.state = state.data();
    ma.owner = owner.data();
    ma.jobs = jobs;
    ma.mtok = mtok.data();
    Sched s;
    s.rs = order_seed * 2 + 1;
    s.rate = 4 + (uint32_t)(order_seed % 5) * 12;
    const bool zeros = order_seed % 2 == 0;  // (as in the form for many workers)
    const auto match = [&](uint32_t m, uint32_t w, uint32_t sv) {
      const uint32_t k = owner[w];
      const uint64_t before = mtok[w];
      // now and then held back in its walk while the insertion ends and others follow
      if ((sv & kOwner) && s.coin(kJobs) < m - k) {
        const uint32_t upto = k + 2 + s.coin(kJobs + 1);
        reader_held[k % kJobs] = k + 1;
        s.hold(8 + s.coin(24), [&, upto] { return f.handed >= upto; });
      }
      take_match<2>(ma, worker_ptrs(ws, L, r, w), m, w, sv);
      s.now->after = 0;
      if (sv & kOwner) {
        const bool ended = !(state[w] & kLoaded) || owner[w] != k;
        counts[0] += ended;
        counts[1] += ended && m - k >= 5;
        if (state[w] & kDeferred)
          counts[2] += 1;
        else
          counts[4] += mtok[w] - before > (uint64_t)ell[(m - 1) & 7];
      }
    };
    const auto add = [&](std::function<void()> body) {
      s.actors.push_back(std::make_unique<Actor>());
      s.actors.back()->body = std::move(body);
    };
    // ---- routing wave
    add([&] {
      for (uint32_t kq = 0; kq < n && !stopped();) {
        bool open = false, can = false;
        uint32_t mw = 0, msv = 0;
        for (uint32_t w = 0; w < W; ++w) {
          const uint32_t sv = state[w];
          if ((sv >> kCountShift) != (kq & kCountMask)) continue;
          open = true;
          if (!can && can_match(sv, kq, owner[w], nbuf)) {
            can = true;
            mw = w;
            msv = sv;
          }
        }
        if (open) {
          if (can && f.staged >= (kq + 1) * kHelpers) {
            if (claim_match(&state[mw], msv)) match(kq, mw, msv);
          } else {
            wait_step();
          }
          continue;
        }
        const uint32_t k = kq, cur = query_slot(k, nbuf), nxt = query_slot(k + 1, nbuf), slot = k % kJobs;
        while (f.decayed < k + 1 && !stopped()) wait_step();
        while (k >= kJobs && jdone[slot] != k - kJobs + 1 && !stopped()) wait_step();
        if (stopped()) break;
        const int32_t Lp = len[k & 7];
        double eh[kMaxWorkers], ch[kMaxWorkers];
        RouteView v[kMaxWorkers];
        uint32_t best = 0;
        for (uint32_t w = 0; w < W; ++w) {
          v[w] = RouteView{};
          v[w].P = lb.P[w];
          for (int x = 0; x < 4; ++x) v[w].theta[x] = lb.theta[x * W + w];
          v[w].Wb = lb.Wb[w];
          v[w].pend_head = lb.head[w];
          v[w].pend_count = lb.count[w];
          eh[w] = lbgr_score(C, v[w], h[cur * kMaxWorkers + w], Lp, &ch[w]);
          if (eh[w] < eh[best]) best = w;
        }
        if (router == KVR_ROUTE_ROUND_ROBIN) best = k % W;
        const Ptrs P = worker_ptrs(ws, L, r, best);
        const int32_t hb = h[cur * kMaxWorkers + best];
        const uint32_t size = lb.size[best], nload = (uint32_t)(Lp - hb), nfree = B - size;
        const uint32_t nev = nload > nfree ? nload - nfree : 0u;
        if (const uint32_t e = commit_lds(C, P, lb, best, v[best], ch[best], hb, Lp, arr[k & 7], olen[k & 7])) {
          fail(e);
          break;
        }
        lb.size[best] = size + nload - nev;
        const uint32_t rn = nev - (nev ? s.coin(nev + 1) / 2 : 0);  // some words left to the evicting wave
        for (uint32_t& p : prog[slot]) p = 0;
        best_of[slot] = best;
        hit[slot] = hb;
        rn_of[slot] = ((uint64_t)(k + 1) << 32) | rn;
        rank_ready[slot] = 0;
        f.routed = k + 1;
        emul_step();
        uint32_t sb;
        while ((sb = __hip_atomic_fetch_or(&state[best], kOwner, 0, 0)) & kOwner) {
          if (stopped()) return;
          wait_step();
        }
        while (sb & kReader) {
          if (stopped()) return;
          wait_step();
          sb = state[best];
        }
        const uint32_t pre = ((sb >> kCountShift) - (k + 1)) & kCountMask;
        PipeJob job{};
        plan_insertion(job, &tree[best * kStWords], B, L.maxL, hb, Lp);
        job.pre = -1;
        uint32_t change = 0;
        if (pre) {
          const int32_t h_pre = h[nxt * kMaxWorkers + best];
          bool stays;
          const int32_t hn = match_before_load(P.nodes, job, h_pre, ell[k & 7],
                                               trail.data() + (nxt * W + best) * kTrailWords, stays);
          int32_t diff = (stays ? hn : 0) - h_pre;
          for (uint32_t x = 2; x <= pre; ++x) {
            diff -= h[query_slot(k + x, nbuf) * kMaxWorkers + best];
            change -= 1u << kCountShift;
          }
          h[nxt * kMaxWorkers + best] = hn;
          mtok[best] += (unsigned long long)(int64_t)diff;
          if (stays)
            job.pre = h_pre;
          else
            change += kDeferred - (1u << kCountShift);
        }
        emul_step();
        // (field by field, as the kernel writes it)
        PipeJob& j = jobs[slot];
        j.k = k;
        j.worker = best;
        j.h = job.h;
        j.L = job.L;
        j.nfree = job.nfree;
        j.nev = job.nev;
        emul_step();
        j.rn = rn;
        j.r0 = slot * L.maxL;
        j.calm = job.calm;
        j.phase = job.phase;
        j.pre = job.pre;
        owner[best] = k;
        h[cur * kMaxWorkers + best] = Lp;
        emul_step();
        __hip_atomic_fetch_add(&state[best], change, 0, 0);
        f.handed = k + 1;
        kq = k + 1;
      }
      f.end = 1;
    });
    // ---- evicting waves
    std::vector<std::vector<int32_t>> ubuf(kEvictors, std::vector<int32_t>(4 * (size_t)(ucap ? ucap : 1)));
    for (uint32_t e = 0; e < kEvictors; ++e)
      add([&, e] {
        UStage us;
        us.node = ubuf[e].data();
        us.len = us.node + ucap;
        us.top = us.len + ucap;
        us.par = us.top + ucap;
        us.cap = ucap;
        for (;;) {
          const uint32_t k = f.ticket++;
          for (;;) {
            const uint32_t ended = f.end;
            emul_step();
            if (f.handed > k) break;
            if (ended || stopped()) return;
            wait_step();
          }
          const uint32_t slot = k % kJobs, buf = query_slot(k, nbuf);
          PipeJob job = load_job(&jobs[slot]);
          const Ptrs P = worker_ptrs(ws, L, r, job.worker);
          uint32_t* t = &tree[job.worker * kStWords];
          int32_t* tr = trail.data() + (buf * W + job.worker) * kTrailWords;
          EvictJob ej;
          ej.s = load_st_lds(t);
          int32_t split;
          const uint32_t lerr = load_leaf(P, ej.s, t, B, q0 + buf * qw, tr, job, split);
          store_st_lds(t, ej.s);
          if (lerr) return fail(lerr);
          if (job.pre >= 0)
            trail_after_load(job, split, job.pre, ell[k & 7], tr,
                             trail.data() + (query_slot(k + 1, nbuf) * W + job.worker) * kTrailWords);
          while (f.fronts != k) {
            if (stopped()) return;
            wait_step();
          }
          if (k >= 7 && jdone[(k - 7) % kJobs] != k - 6) counts[3] += 1;
          if (job.h == 0) rf_add(&rootf[job.worker * kRootFilterWords], job.tok);
          PipeJob& j = jobs[slot];
          j.l = job.l;
          j.a = job.a;
          j.tok = job.tok;
          j.replace = job.replace;
          j.marked = job.marked;
          ell[(k + nbuf - 1) & 7] = 0x7fffffff;
          __hip_atomic_fetch_or(&state[job.worker], kLoaded, 0, 0);
          if (job.h < job.L) rank_ready[slot] = ((k + 1) << 2) | 1u;
          f.fronts = k + 1;
          emul_step();
          if (!job.marked) mark_cached(P, ej.s, B, job, tr);
          atomicOr(&state[job.worker], kMarked);
          // now and then held back until other insertions are loaded, or a match is
          // held back beside it
          if (job.nev > 0 && s.coin(2)) {
            const uint32_t upto = k + 2 + s.coin(kJobs);
            s.hold(1 + s.coin(40), [&, upto, slot, k] { return f.fronts >= upto || reader_held[slot] == k + 1; });
          }
          WaveHook hook{job.h < job.L, job, &rank_ready[slot], &rank[slot], t, &f};
          ej.ia = InsertArgs{C.seed, k, job.worker, r, B, job.rn, words.data() + job.r0, job.rn ? prog[slot] : nullptr,
                             1, 2, nullptr, nullptr};
          ej.h = job.h;
          ej.L = job.L;
          ej.l = job.l;
          ej.nfree = job.nfree;
          ej.nev = job.nev;
          ej.c0 = ej.s.cnt;
          ej.reset_at = job.h < job.L && ej.c0 + (uint32_t)(job.L - job.h) >= B + 1u ? job.h + (int32_t)(B - ej.c0) : -1;
          ej.worker = job.worker;
          ej.final_size = 0;
          int64_t dbg[4];
          const uint32_t ee = ej.s.err ? ej.s.err : rlt_evict<false>(P, ej, us, dbg, nullptr, 0, 0, hook);
          if (ee) return fail(ee);
          s.now->after = 0;
          __hip_atomic_fetch_and(&state[job.worker], ~(kOwner | kLoaded | kMarked | kDeferred), 0, 0);
          jdone[slot] = k + 1;
        }
      });
    // ---- helpers
    for (uint32_t hw = 0; hw < kHelpers; ++hw)
      add([&, hw] {
        uint32_t sN = 0, dN = 0;
        int64_t tick_prev = 0;
        if (hw == 0) {
          for (uint32_t w = 0; w < W; ++w) {
            const Ptrs P = worker_ptrs(ws, L, r, w);
            decay_lds(C, lb, w, P.hdr, P.pend, P.PC, arrival[0], 0, arrival[0] / C.dt_us, 0);
          }
          tick_prev = arrival[0] / C.dt_us;
          f.decayed = 1;
        }
        for (;;) {
          emul_step();
          const Flags v = f;
          if (v.stop || g_s->hung) return;
          if (dN < v.routed && (hw > 0 || sN > dN + 1 || dN + 1 == n)) {
            const uint32_t k = dN++, slot = k % kJobs;
            if (hw == 0) {
              const uint32_t best = best_of[slot];
              route[(uint64_t)r * n + k] = (int32_t)best;
              hits[(uint64_t)r * n + k] = hit[slot];
              for (uint32_t w = 0; w < W && all_hits; ++w)
                all_hits[((uint64_t)r * n + k) * W + w] =
                    w == best ? hit[slot] : h[query_slot(k, nbuf) * kMaxWorkers + w];
              if (k + 1 < n) {
                const int64_t t = arr[(k + 1) & 7], tp = arr[k & 7], tick = t / C.dt_us;
                for (uint32_t w = 0; w < W; ++w) {
                  const Ptrs P = worker_ptrs(ws, L, r, w);
                  decay_lds(C, lb, w, P.hdr, P.pend, P.PC, t, tp, tick, tick_prev);
                }
                tick_prev = tick;
                f.decayed = k + 2;
              }
            } else if (hw == 1) {
              const uint64_t info = rn_of[slot];
              const uint32_t rn = (uint32_t)info;
              if ((uint32_t)(info >> 32) == k + 1 && rn) {
                const uint32_t best = best_of[slot];
                uint32_t* rw = words.data() + slot * L.maxL;
                uint32_t rounds = 0;
                // held back in its draws until later insertions have the slot
                if (hold_draws && s.coin(hold_draws) == 0)
                  s.hold(1 + s.coin(2 * rn), [&, k] { return f.handed > k + kJobs; });
                for (uint32_t d = 0; d < rn; d += 2) {
                  for (uint32_t x = d; x < d + 2 && x < rn; ++x)
                    rw[x] = (uint32_t)(philox_word0(k, best, x, 0ull, C.seed, r) >> 32);
                  prog[slot][0] = ++rounds;
                  emul_step();
                }
                s.now->after = 0;
              }
            }
            continue;
          }
          bool ranked = false;
          for (uint32_t slot = 0; slot < kJobs && !ranked; ++slot) {
            const uint32_t want = rank_ready[slot];
            if ((want & 3u) != 1u || atomicCAS(&rank_ready[slot], want, want + 1) != want) continue;
            const PipeJob job = load_job(&jobs[slot]);
            const St st = load_st_lds(&tree[job.worker * kStWords]);
            const Ptrs P = worker_ptrs(ws, L, r, job.worker);
            rank[slot] = rank_of_leaf(P, st.hwm, st.nleaves, arena_of(P, st.arena_sel), job);
            rank_ready[slot] = want + 2;
            ranked = true;
          }
          if (ranked) continue;
          if (sN < n && sN < v.fronts + nbuf && v.staged >= sN * kHelpers) {
            const int32_t Ln = (int32_t)(offsets[sN + 1] - offsets[sN]), Lc = sN ? len[(sN - 1) & 7] : 0;
            if (hw == 0) {
              len[sN & 7] = Ln;
              olen[sN & 7] = query_out_len(out_len, sN);
              arr[sN & 7] = arrival[sN];
            }
            int32_t* qn = q0 + query_slot(sN, nbuf) * qw;
            const int32_t* qc = q0 + query_slot(sN + nbuf - 1, nbuf) * qw;
            int32_t m = Lc < Ln ? Lc : Ln;
            for (int32_t x = (int32_t)hw; x < Ln; x += (int32_t)kHelpers) {
              qn[x] = tokens[offsets[sN] + x];
              if (x < m && qc[x] != qn[x]) m = x;
            }
            emul_step();
            atomicMin(&ell[(sN - 1) & 7], m);
            f.staged += 1;
            sN += 1;
            continue;
          }
          if (v.routed < n) {
            const uint32_t whole = v.staged / kHelpers;
            uint32_t lim = v.fronts + nbuf;
            if (lim > whole) lim = whole;
            uint32_t mw = W, mm = 0, msv = 0;
            for (uint32_t x = 0; x < W; ++x) {
              const uint32_t w = (x + hw * W / kHelpers) % W, sv = state[w];
              const uint32_t m = v.routed + (((sv >> kCountShift) - v.routed) & kCountMask);
              if (m >= lim || !can_match(sv, m, owner[w], nbuf)) continue;
              if (zeros && take_zero_match(ma, m, w, sv)) {
                counts[5] += 1;
                continue;
              }
              if (mw < W && m >= mm) continue;
              mw = w;
              mm = m;
              msv = sv;
            }
            if (mw < W) {
              if (claim_match(&state[mw], msv)) match(mm, mw, msv);
              continue;
            }
          }
          if (v.end && dN >= v.routed && v.fronts == n) return;
          wait_step();
        }
      });
    run_all(s);
    if (s.hung) return -20;
    if (err) return (int)err;
    for (uint32_t w = 0; w < W; ++w) {
      const Ptrs P = worker_ptrs(ws, L, r, w);
      WorkerHdr* hd = P.hdr;
      std::memcpy(static_cast<void*>(hd), &tree[(size_t)w * kStWords], 4 * (kStWords - 1));
      hd->P = lb.P[w];
      for (int x = 0; x < 4; ++x) hd->theta[x] = lb.theta[x * W + w];
      hd->Wb = lb.Wb[w];
      hd->tl = arrival[n - 1];
      hd->pend_head = lb.head[w];
      hd->pend_count = lb.count[w];
      hd->matched_tokens = mtok[w];
      if (!worker_stats(P, out + (uint64_t)r * W + w)) return -7;
    }
  }
  return 0;
}
