// rkc_tiny.h -- replay of one pool of at most E events (E = 2 or 4) by one lane.
//
// Batches of very short traces (the capacity sweep: two events a pool) are bound by what a pool costs
// before and after its events, which a wavefront per pool pays once per pool: LDS set-up, a chain
// of dependent loads, the final passes.  Here a lane replays a pool, so a wavefront's 64 pools share
// each of these.  Same contract and outputs as the other kernels; the state is held by event step
// in E-entry arrays that full unrolling keeps in registers, and everything the other kernels
// maintain incrementally is recomputed from them:
//   requests  the request of PREFILL step u: live bit, chain, R (shared extent it holds), length
//   claims    the claim of CLAIM step u: live bit, meta word, its steps; L, chain, T from the event
//   chains    named at the step that first registers positions of the chain: id, registered length n
//   touches   of step u: chain and extent; position p was last touched at the newest u with extent > p
//   runs      of FINISH step u: the finished request's private blocks [lo, top)
// Live sets in id order are bit masks over steps, and so is the deferral queue (requests enter it in
// step order and leave it from the front).
//
// Plain C++ on one pool's data (no lanes, no memory but the pool's own arrays), so that it also
// compiles for the host, where it is checked against the oracle.
#ifndef RKC_TINY_H
#define RKC_TINY_H

#include <stdint.h>

#include "rkc.h"

#ifdef __HIPCC__
#define RKC_TINY_FN __host__ __device__ __forceinline__
#define RKC_UNROLL _Pragma("unroll")
#else
#define RKC_TINY_FN inline
#define RKC_UNROLL
#endif

// One lane per pool or one wavefront per pool (compact kernel), for a batch within the compact kernel's limits.
// A lane's unrolled code runs every event type that its wave's pools hold in turn, so its time depends on the
// mix and hardly on the number of pools; a wavefront's pays for every pool.  By lane against by wavefront:
//   two events: batches of one claim and one prefill a pool 7.3 us at any size up to 8,192 pools against 6.8 us
//   (64 pools), 7.3 (1,024), 8.5 (4,096) and 11.9 (8,192); pools of 80 blocks with mixed events 9.1 to 12.2 us
//   against 6.4, 7.3, 9.3 and 13.2; 131,072 pools 19.6 against 144 us.  So from the first batch on that
//   is not resident as wavefronts all at once.
//   three and four events: 65,536 pools 22 to 51 us against 75 to 95, 49,152 pools 22 to 51 against 58 to 73
//   (both of these with a pass of about 2 us over the batch before them); 32,768 pools 48 us by lane at the
//   longest, 39 to 48 by wavefront.
//   eight events: 331 us against 121 us at 65,536 pools, never worth it.
// A lane writes its pool's unused claim slots by itself, so it takes pools with few slots only.
inline bool rkc_tiny_serves(int32_t n_pools, int32_t max_events, int32_t max_slots) {
  return max_slots <= 8 && ((max_events <= 2 && n_pools > 4096) || (max_events <= 4 && n_pools >= 49152));
}

// the batch limits a pool's descriptor is checked against
struct rkc_tiny_limits {
  int64_t n_events_total, n_slots_total;
  int32_t max_usable, max_events, max_chains, max_reqs, max_claims, max_slots;
};

template <int E>
struct rkc_tiny {
  typedef uint32_t u32;
  typedef int32_t i32;
  static_assert(E <= 8, "per-code counters are 4 bits wide");
  static constexpr u32 NONE = 0xFFFFFFFFu;
  // claim meta: state[0:3) eff[3:5) hard[5] prio[6:8) pending[8] decision[9:12) demotable[12]
  // best_effort[13] relaxed_by_runtime[14] offloadable[15]
  static constexpr u32 M_PEND = 1u << 8, M_DEMQ = 1u << 12, M_BE = 1u << 13, M_RELAXED = 1u << 14, M_OFFQ = 1u << 15;

  struct Event { u32 w[4]; };
  struct Claim {
    u32 m;                      // meta
    u32 dem, exp, rel, pf, harm;  // steps, NONE when it never happened
    u32 blk;                    // active refusals attributed to it
  };
  struct Out { u32 code, flags, n16; i32 id, a, b; };
  struct Alloc { u32 ok, E_, resident, post, unclaimed; };

  // descriptor
  u32 U, mode, maxq, maxr, nslots, nch, dlim, relax_on, t2cap;
  Event ev[E];
  u32 rq_live, rq_c[E], rq_R[E], rq_len[E];
  u32 cl_live, slots;  // live claims; CLAIM steps that took a telemetry slot
  Claim cl[E];
  u32 ch_id[E], ch_n[E];
  u32 to_c[E], to_x[E];
  u32 run_lo[E], run_top[E];
  u32 dq, dq_cnt, retried;  // deferred requests; DEFERRED outcomes of the front one
  u32 F, A, peak, status, t2, t2pk, nslot, evicted;
  // pool telemetry: outcomes per code and claim decisions, 4 bits each, and the rest as words
  uint64_t hist;
  u32 decs, vic, res, post, dropped, hits, nharm, npf, nexp, ndem, nrel, rsv, rrf, rdem, offc, offb, rest;

  RKC_TINY_FN static u32 umin(u32 a, u32 b) { return a < b ? a : b; }
  RKC_TINY_FN static u32 umax(u32 a, u32 b) { return a > b ? a : b; }
  RKC_TINY_FN static u32 sub0(u32 a, u32 b) { return a > b ? a - b : 0u; }
  RKC_TINY_FN static u32 pop(u32 m) { return (u32)__builtin_popcount(m); }
  // element i of a register array
  RKC_TINY_FN static u32 at(const u32 (&v)[E], u32 i) {
    u32 r = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) r = (u32)u == i ? v[u] : r;
    return r;
  }
  RKC_TINY_FN u32 evw(int k, u32 i) const {
    u32 r = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) r = (u32)u == i ? ev[u].w[k] : r;
    return r;
  }
  // the k-th set bit of m (k < popcount)
  RKC_TINY_FN static u32 kth(u32 m, u32 k) {
    RKC_UNROLL for (int u = 0; u < E - 1; u++)
      if (k > 0) { m &= m - 1; k--; }
    return (u32)__builtin_ctz(m);
  }

  RKC_TINY_FN bool hard() const { return mode == RKC_MODE_HARD; }
  RKC_TINY_FN bool softl() const { return mode & 1u; }  // soft levels and acceptance
  RKC_TINY_FN bool noadm() const { return mode == RKC_MODE_NOADMIT; }
  RKC_TINY_FN static u32 st(u32 m) { return m & 7u; }
  RKC_TINY_FN static u32 eff(u32 m) { return (m >> 3) & 3u; }
  RKC_TINY_FN static u32 prio(u32 m) { return (m >> 6) & 3u; }
  RKC_TINY_FN bool live(int u) const { return (cl_live >> u) & 1u; }
  RKC_TINY_FN bool hmat(int u) const {
    return live(u) && st(cl[u].m) == RKC_ST_MATERIALIZED && eff(cl[u].m) == RKC_PROT_HARD;
  }
  // soft level that claim u ranks victims at, 0 for none
  RKC_TINY_FN u32 level(int u) const {
    const u32 m = cl[u].m;
    const bool l = softl() && live(u) &&
                   ((st(m) == RKC_ST_MATERIALIZED && eff(m) == RKC_PROT_SOFT) || st(m) == RKC_ST_DEMOTED);
    return l ? prio(m) + 1u : 0u;
  }
  RKC_TINY_FN static u32 packed_of(u32 m) {
    return ((m >> 9) & 7u) | (st(m) << 4) | (((m >> 5) & 1u) << 8) | (prio(m) << 9) | (eff(m) << 11) |
           (((m >> 12) & 15u) << 13);
  }

  // chain c: registered length, leading positions held by live requests, hard protection extent
  RKC_TINY_FN u32 n_of(u32 c) const {
    u32 r = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) r = ch_id[u] == c ? ch_n[u] : r;
    return r;
  }
  RKC_TINY_FN u32 hold_of(u32 c) const {
    u32 r = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) r = umax(r, ((rq_live >> u) & 1u) && rq_c[u] == c ? rq_R[u] : 0u);
    return r;
  }
  RKC_TINY_FN u32 prot_of(u32 c, u32 but = 0) const {  // but: claims left out
    u32 r = 0;
    RKC_UNROLL for (int u = 0; u < E; u++)
      r = umax(r, hard() && hmat(u) && !((but >> u) & 1u) && ev[u].w[2] == c ? ev[u].w[1] : 0u);
    return r;
  }
  RKC_TINY_FN void name(u32 t, u32 c, u32 n) {  // chain c holds n registered positions
    u32 found = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const bool on = ch_id[u] == c;
      ch_n[u] = on ? n : ch_n[u];
      found |= (u32)on;
    }
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const bool nw = !found && (u32)u == t;
      ch_id[u] = nw ? c : ch_id[u];
      ch_n[u] = nw ? n : ch_n[u];
    }
  }
  RKC_TINY_FN void touch(u32 t, u32 c, u32 x) {
    RKC_UNROLL for (int u = 0; u < E; u++) {
      to_c[u] = (u32)u == t ? c : to_c[u];
      to_x[u] = (u32)u == t ? x : to_x[u];
    }
  }
  // evictable blocks (above the hits h of chain hc), and protected resident blocks
  RKC_TINY_FN u32 evictable(i32 hc, u32 h) const {
    u32 e = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const u32 c = ch_id[u];
      u32 lo = umax(hold_of(c), prot_of(c));
      if ((i32)c == hc) lo = umax(lo, h);
      e += c != NONE ? sub0(ch_n[u], lo) : 0u;
      e += run_top[u] - run_lo[u];
    }
    return e;
  }
  RKC_TINY_FN u32 protected_resident() const {
    u32 p = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) p += ch_id[u] != NONE ? sub0(prot_of(ch_id[u]), hold_of(ch_id[u])) : 0u;
    return p;
  }

  // FREE blocks first, then the smallest (level, last use) runs from the chain tops and the private
  // runs (which win a tie with a chain touched at the step they finished).
  RKC_TINY_FN Alloc alloc(u32 need, i32 hc, u32 h) {
    Alloc r = {1, 0, 0, 0, 0};
    if (need <= F) {
      F -= need;
      return r;
    }
    r.E_ = evictable(hc, h);
    if (need > F + r.E_) {
      r.ok = 0;
      return r;
    }
    u32 K = need - F;
    F = 0;
    vic += K;
    const u32 K0 = K;
    // every pass takes a whole run; a chain has at most one per touch and soft level
    for (u32 guard = 0; K > 0 && guard < 8u * E * E; guard++) {
      u32 best = NONE, bu = 0, blo = 0;
      RKC_UNROLL for (int u = 0; u < E; u++) {
        const u32 c = ch_id[u], n = ch_n[u];
        u32 lo = umax(hold_of(c), prot_of(c));
        if ((i32)c == hc) lo = umax(lo, h);
        if (c != NONE && n > lo) {
          u32 lu = 0, lvl = 0, rl = lo;
          RKC_UNROLL for (int v = 0; v < E; v++) {
            lu = to_c[v] == c && to_x[v] >= n ? (u32)v : lu;
            lvl = umax(lvl, ev[v].w[2] == c && live(v) && ev[v].w[1] >= n ? level(v) : 0u);
          }
          RKC_UNROLL for (int v = 0; v < E; v++) {
            rl = umax(rl, to_c[v] == c && (u32)v > lu ? to_x[v] : 0u);
            rl = umax(rl, live(v) && ev[v].w[2] == c && level(v) > lvl ? ev[v].w[1] : 0u);
          }
          const u32 key = (lvl << 8) | (lu << 1) | 1u;
          if (key < best) { best = key; bu = (u32)u; blo = rl; }
        }
        const u32 kr = run_top[u] > run_lo[u] ? (u32)u << 1 : NONE;
        if (kr < best) { best = kr; bu = (u32)u; }
      }
      if (best == NONE) { status |= (u32)RKC_PS_INTERNAL; break; }  // cannot happen: feasibility was checked
      if (!(best & 1u)) {
        const u32 m = umin(K, at(run_top, bu) - at(run_lo, bu));
        RKC_UNROLL for (int u = 0; u < E; u++) run_top[u] -= (u32)u == bu ? m : 0u;
        K -= m;
      } else {
        const u32 c = at(ch_id, bu), n = at(ch_n, bu);
        const u32 m = umin(K, n - blo), nw = n - m;
        u32 covA = 0, covS = 0;
        RKC_UNROLL for (int v = 0; v < E; v++) {
          const u32 cm = cl[v].m, s = st(cm);
          const bool on = live(v) && ev[v].w[2] == c && eff(cm) != RKC_PROT_OFFLOADED;
          covA = umax(covA, on ? ev[v].w[1] : 0u);
          covS = umax(covS, on && (s == RKC_ST_OBSERVED || s == RKC_ST_MATERIALIZED || s == RKC_ST_HARMED) ? ev[v].w[1] : 0u);
        }
        const u32 rs = sub0(umin(n, covA), nw), sc = sub0(umin(n, covS), nw);
        r.resident += rs;
        r.post += rs - sc;
        RKC_UNROLL for (int u = 0; u < E; u++) ch_n[u] = (u32)u == bu ? nw : ch_n[u];
        K -= m;
        evicted = 1;
      }
    }
    if (K) status |= (u32)RKC_PS_INTERNAL;  // cannot happen
    r.unclaimed = K0 - r.resident;
    return r;
  }

  RKC_TINY_FN void refusal(u32 need, i32 hc, u32 h, u32 Hc, Out& o) {
    u32 Pr = protected_resident();
    if (hard() && hc >= 0) Pr -= sub0(umin(prot_of((u32)hc), h), hold_of((u32)hc));
    const u32 req = A + Hc + need;
    o.id = -1;
    o.n16 = 0;
    if (Pr > 0 && req <= U) {
      o.code = RKC_OC_REFUSED_CLAIM;
      RKC_UNROLL for (int u = E - 1; u >= 0; u--) {
        const u32 c = ev[u].w[2];
        u32 cov = hold_of(c);
        if ((i32)c == hc) cov = umax(cov, h);
        const bool b = hmat(u) && ev[u].w[1] > cov;
        cl[u].blk += (u32)b;
        o.n16 += (u32)b;
        o.id = b ? u : o.id;  // (the claim's id is its step: the smallest comes last)
      }
    } else {
      o.code = RKC_OC_REFUSED_CAPACITY;
    }
    o.a = (i32)Pr;
    o.b = (i32)req;
  }

  // Runtime relaxation of a hard-protection pool (lowest priority, then lowest id, as few claims as
  // make the request fit, none when all would not do): returns the claims relaxed.
  RKC_TINY_FN u32 relax(u32 t, u32 need, i32 hc, u32 h) {
    if (!hard() || !relax_on || need <= F) return 0;
    u32 avail = F + evictable(hc, h);
    if (need <= avail) return 0;
    u32 cand = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const u32 c = ev[u].w[2];
      u32 cov = hold_of(c);
      if ((i32)c == hc) cov = umax(cov, h);
      cand |= hmat(u) && (cl[u].m & (M_DEMQ | M_OFFQ)) && ev[u].w[1] > cov ? 1u << u : 0u;
    }
    u32 picked = 0, offs = 0, room = sub0(t2cap, t2), moved = 0;
    RKC_UNROLL for (int k = 0; k < E; k++) {
      if (cand && need > avail) {
        u32 best = NONE, m = 0, L = 0, c = 0;
        RKC_UNROLL for (int u = E - 1; u >= 0; u--) {
          const u32 p = (prio(cl[u].m) << 8) | (u32)u;
          if (((cand >> u) & 1u) && p < best) { best = p; m = cl[u].m; L = ev[u].w[1]; c = ev[u].w[2]; }
        }
        const u32 i = best & 255u;
        cand &= ~(1u << i);
        const bool off = (m & M_OFFQ) && L <= room;
        if (off || (m & M_DEMQ)) {
          if (off) { room -= L; moved += L; offs |= 1u << i; }
          u32 base = hold_of(c);
          if ((i32)c == hc) base = umax(base, h);
          const u32 n = n_of(c), before = prot_of(c, picked);
          picked |= 1u << i;
          avail += sub0(n, umax(base, prot_of(c, picked))) - sub0(n, umax(base, before));
        }
      }
    }
    if (need > avail) return 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const bool p = (picked >> u) & 1u, o = (offs >> u) & 1u;
      const u32 m = cl[u].m;
      if (p && o) cl[u].m = (m & ~(3u << 3)) | (RKC_PROT_OFFLOADED << 3) | M_RELAXED;
      if (p && !o) { cl[u].m = (m & ~7u) | RKC_ST_DEMOTED | M_RELAXED; cl[u].dem = t; }
    }
    const u32 no = pop(offs);
    rdem += pop(picked) - no;
    if (no) {
      t2 += moved;
      t2pk = umax(t2pk, t2);
      offc += no;
      offb += moved;
    }
    return pop(picked);
  }

  RKC_TINY_FN void served(const Alloc& r, u32 relaxed, Out& o) {
    o.code = r.resident ? RKC_OC_EVICT_RESIDENT : RKC_OC_ADMIT;
    o.a = (i32)r.resident;
    o.flags |= (r.post ? (u32)RKC_FL_POST_RELEASE_LOSS : 0u) | (r.unclaimed ? (u32)RKC_FL_EVICT_UNCLAIMED : 0u);
    post += r.post;
    res += r.resident;
    if (relaxed) { o.code = RKC_OC_RELAXED; o.n16 = relaxed; }
  }

  // Request rid (its S, chain and P from its PREFILL event) at step t.
  RKC_TINY_FN void admit(u32 t, u32 rid, bool late, Out& o) {
    const u32 S = evw(1, rid), cc = evw(2, rid), P = evw(3, rid);
    i32 hc = -1;
    u32 h = 0, Hc = 0;
    if (P > 0) {
      hc = (i32)cc;
      h = umin(P, n_of(cc));
      Hc = sub0(h, hold_of(cc));
    }
    const u32 need = S - h;
    const u32 relaxed = relax(t, need, hc, h);
    const Alloc r = alloc(need, hc, h);
    if (!r.ok) {
      refusal(need, hc, h, Hc, o);
      const bool by_claim = o.code == RKC_OC_REFUSED_CLAIM;
      if (late) {
        if (by_claim && dq_cnt < dlim) {
          dq_cnt++;
          o.code = RKC_OC_DEFERRED;
        } else {
          dq &= dq - 1;
          dq_cnt = 1;
          rrf++;
        }
      } else if (by_claim && dlim > 0 && pop(dq) < maxr) {
        dq |= 1u << t;
        o.code = RKC_OC_DEFERRED;
      }
    } else {
      A += Hc + need;
      u32 R = 0;
      if (hc >= 0) {
        const u32 n = n_of(cc);  // victims may have shortened this chain above the hits
        R = noadm() ? h : P;
        name(t, cc, !noadm() && P > n ? P : n);
        if (R) touch(t, cc, R);
      }
      RKC_UNROLL for (int u = 0; u < E; u++) {
        if ((u32)u == rid) { rq_c[u] = hc >= 0 ? cc : NONE; rq_R[u] = R; rq_len[u] = S; }
      }
      rq_live |= 1u << rid;
      if (late) {
        dq &= dq - 1;
        dq_cnt = 1;
        rsv++;
      }
      o.id = (i32)rid;
      o.b = (i32)h;
      hits += h;
      served(r, relaxed, o);
      if (hard() && P > h && t2cap > 0) {
        // positions past the hits that a claim holding a second-tier copy covers are restored
        u32 e = 0;
        RKC_UNROLL for (int u = 0; u < E; u++)
          e = umax(e, live(u) && ev[u].w[2] == cc && eff(cl[u].m) == RKC_PROT_OFFLOADED ? ev[u].w[1] : 0u);
        rest += sub0(umin(P, e), h);
      }
    }
  }

  // one event; returns its outcome
  RKC_TINY_FN Out step(u32 t) {
    const u32 w0 = evw(0, t), w1 = evw(1, t), w2 = evw(2, t), w3 = evw(3, t), type = w0 & 15u;
    Out o = {RKC_OC_NOOP, 0, 0, -1, 0, 0};
    evicted = 0;
    // expiry at the start of the step
    u32 expired = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const u32 m = cl[u].m, dur = ev[u].w[0] >> 16;
      if (live(u) && (st(m) == RKC_ST_MATERIALIZED || st(m) == RKC_ST_DEMOTED) && dur && (u32)u + dur <= t) {
        u32 m2 = (m & ~7u) | RKC_ST_EXPIRED;
        if (eff(m) == RKC_PROT_OFFLOADED) {
          // the second-tier copy is dropped; a predicate that held only through it fails now
          t2 -= ev[u].w[1];
          m2 &= ~(3u << 3);
          if ((m & M_PEND) && n_of(ev[u].w[2]) < ev[u].w[3]) {
            m2 &= ~M_PEND;
            cl[u].pf = t;
            o.flags |= RKC_FL_PRED_FAIL;
            npf++;
          }
        }
        cl[u].m = m2;
        cl[u].exp = t;
        expired++;
      }
    }
    if (expired) {
      o.flags |= RKC_FL_EXPIRED;
      o.n16 = expired;
      nexp += expired;
    }
    const bool fb = (i32)w1 < 1 || (i32)w1 > RKC_MAX_FIELD_BLOCKS, cb = w2 >= nch;
    const bool tb = (i32)w3 < 0 || (i32)w3 > (i32)w1;
    const u32 nreq = pop(rq_live), ncl = pop(cl_live);
    bool bad = false;
    u32 rid = t;
    bool adm = false;
    if (type == RKC_EV_PREFILL) {
      bad = fb || tb || ((i32)w3 > 0 && cb);
      adm = !bad;
    } else if (type == RKC_EV_RETRY && hard() && dq) {
      rid = (u32)__builtin_ctz(dq);
      adm = true;
    }
    if (adm && nreq >= maxr) {
      status |= RKC_PS_REQUEST_TABLE;  // (a retried request stays queued)
      bad = true;
      adm = false;
    }
    if (adm) {
      admit(t, rid, type == RKC_EV_RETRY, o);
    } else if (type == RKC_EV_EXTEND) {
      bad = fb;
      if (!bad && nreq > 0) {
        const u32 i = kth(rq_live, w2 % nreq);
        const u32 relaxed = relax(t, w1, -1, 0);
        const Alloc r = alloc(w1, -1, 0);
        if (!r.ok) {
          refusal(w1, -1, 0, 0, o);
        } else {
          A += w1;
          RKC_UNROLL for (int u = 0; u < E; u++) rq_len[u] += (u32)u == i ? w1 : 0u;
          o.id = (i32)i;
          o.b = (i32)A;
          served(r, relaxed, o);
        }
      }
    } else if (type == RKC_EV_CLAIM) {
      if (nslot >= nslots) {
        status |= RKC_PS_SLOT_TABLE;
        bad = true;
      } else {
        nslot++;
        slots |= 1u << t;
        bad = fb || cb || tb;
        if (!bad && ncl >= maxq) {
          status |= RKC_PS_CLAIM_TABLE;
          bad = true;
        }
        if (!bad) claim(t, w0, w1, w2, o);
      }
    } else if (type == RKC_EV_FINISH) {
      if (nreq > 0) finish(t, kth(rq_live, w1 % nreq), o);
    } else if (type == RKC_EV_RELEASE || type == RKC_EV_DEMOTE) {
      lifecycle(t, type, w1, o);
    } else if (type > RKC_EV_RETRY) {
      bad = true;
    }
    if (bad) { o.code = RKC_OC_INVALID; o.id = -1; o.a = o.b = 0; }
    if (evicted) {
      // predicate sweep: claims whose chain fell below their threshold fail for the first time
      u32 pfs = 0, hms = 0;
      RKC_UNROLL for (int u = 0; u < E; u++) {
        const u32 m = cl[u].m;
        if (live(u) && (m & M_PEND) && eff(m) != RKC_PROT_OFFLOADED && n_of(ev[u].w[2]) < ev[u].w[3]) {
          const bool hm = st(m) == RKC_ST_MATERIALIZED;
          cl[u].m = hm ? (m & ~(M_PEND | 7u)) | RKC_ST_HARMED : m & ~M_PEND;
          cl[u].pf = t;
          cl[u].harm = hm ? t : cl[u].harm;
          pfs++;
          hms += (u32)hm;
        }
      }
      npf += pfs;
      nharm += hms;
      o.flags |= (pfs ? (u32)RKC_FL_PRED_FAIL : 0u) | (hms ? (u32)RKC_FL_HARM : 0u);
    }
    peak = umax(peak, A);
    hist += (uint64_t)1 << (4u * o.code);
    return o;
  }

  RKC_TINY_FN void claim(u32 t, u32 w0, u32 L, u32 c, Out& o) {
    const u32 hardq = (w0 >> 4) & 1u, pr = (w0 >> 5) & 3u, beq = (w0 >> 8) & 1u;
    const u32 req = (w0 & (1u << 7) ? M_DEMQ : 0u) | (beq ? M_BE : 0u) | (w0 & (1u << 9) ? M_OFFQ : 0u);
    const bool obs = !softl() || beq;
    const u32 n0 = n_of(c), h = umin(L, n0), need = L - h;
    const Alloc r = alloc(need, (i32)c, h);
    const u32 ef = beq ? RKC_PROT_NONE : hard() ? (hardq ? RKC_PROT_HARD : RKC_PROT_SOFT)
                 : mode == RKC_MODE_SOFT ? RKC_PROT_SOFT : RKC_PROT_NONE;
    const u32 lowered = mode == RKC_MODE_SOFT && hardq;
    const u32 dec = !r.ok ? (obs ? RKC_DEC_SHADOW : RKC_DEC_REJECTED)
                  : obs ? RKC_DEC_SHADOW : lowered ? RKC_DEC_ACCEPTED_APPROX : RKC_DEC_ACCEPTED;
    const u32 state = !r.ok ? RKC_ST_REJECTED : obs ? RKC_ST_OBSERVED : RKC_ST_MATERIALIZED;
    const u32 m = state | (ef << 3) | (hardq << 5) | (pr << 6) | (r.ok ? M_PEND : 0u) | (dec << 9) | req;
    RKC_UNROLL for (int u = 0; u < E; u++) cl[u].m = (u32)u == t ? m : cl[u].m;
    decs += 1u << (8u * (dec - 1u));
    if (!r.ok) {
      o.code = RKC_OC_MATFAIL;
      o.id = (i32)t;
      o.a = (i32)need;
      o.b = (i32)(F + r.E_);
    } else {
      o.flags |= obs ? (u32)RKC_FL_SHADOW : lowered ? (u32)RKC_FL_LOWERED : 0u;
      cl_live |= 1u << t;
      name(t, c, umax(n_of(c), L));
      touch(t, c, L);
      o.id = (i32)t;
      o.b = (i32)need;
      served(r, 0, o);
    }
  }

  RKC_TINY_FN void finish(u32 t, u32 i, Out& o) {
    const u32 c = at(rq_c, i), R = at(rq_R, i), len = at(rq_len, i);
    rq_live &= ~(1u << i);
    u32 turned = 0;
    if (c != NONE) {
      turned = sub0(R, hold_of(c));
      if (R) touch(t, c, R);
    }
    // write no-admit drops the request's own blocks; otherwise they become a private run
    const u32 own = len - R, drop = noadm() ? own : 0u, kept = own - drop;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      const bool me = (u32)u == t && kept > 0;
      run_lo[u] = me ? R : run_lo[u];
      run_top[u] = me ? len : run_top[u];
    }
    turned += kept;
    F += drop;
    A -= turned + drop;
    dropped += drop;
    o.code = RKC_OC_FINISHED;
    o.id = (i32)i;
    o.a = (i32)turned;
    o.b = (i32)drop;
    if (drop) o.flags |= RKC_FL_NOADMIT_DROP;
  }

  RKC_TINY_FN void lifecycle(u32 t, u32 type, u32 sel, Out& o) {
    u32 set = cl_live;
    if (type == RKC_EV_DEMOTE) {
      set = 0;
      RKC_UNROLL for (int u = 0; u < E; u++) {
        const u32 m = cl[u].m;
        set |= softl() && live(u) && st(m) == RKC_ST_MATERIALIZED && ((m >> 5) & 1u) && eff(m) != RKC_PROT_OFFLOADED ? 1u << u : 0u;
      }
    }
    if (set) {
      const u32 i = kth(set, sel % pop(set));
      const bool rel = type == RKC_EV_RELEASE;
      RKC_UNROLL for (int u = 0; u < E; u++) {
        if ((u32)u == i) {
          if (rel && eff(cl[u].m) == RKC_PROT_OFFLOADED) t2 -= ev[u].w[1];  // the copy is dropped
          cl[u].m = (cl[u].m & ~7u) | (rel ? RKC_ST_RELEASED : RKC_ST_DEMOTED);
          cl[u].rel = rel ? t : cl[u].rel;
          cl[u].dem = rel ? cl[u].dem : t;
        }
      }
      if (rel) { cl_live &= ~(1u << i); nrel++; } else { ndem++; }
      o.code = rel ? RKC_OC_RELEASED : RKC_OC_DEMOTED;
      const u32 L = evw(1, i);
      o.id = (i32)i;
      o.a = (i32)umin(n_of(evw(2, i)), L);
      o.b = (i32)evw(3, i);
    }
  }

  // Telemetry word w of the finished pool (w a constant where this is called from unrolled code).
  RKC_TINY_FN u32 tel(int w) const {
    if (w < 10) return (u32)(hist >> (4 * w)) & 15u;
    if (w >= 15 && w <= 18) return (decs >> (8 * (w - 15))) & 255u;
    switch (w) {
      case 10: return vic;
      case 11: return res;
      case 12: return post;
      case 13: return dropped;
      case 14: return hits;
      case 19: return nharm;
      case 20: return npf;
      case 21: return nexp;
      case 22: return ndem;
      case 23: return nrel;
      case 24: return peak;
      case 25: return A;
      case 26: return U - F - A;
      case 27: return F;
      case 28: return protected_resident();
      case 29: return pop(rq_live);
      case 30: return pop(cl_live);
      case 31: return status;
      case 32: return (u32)(hist >> (4 * RKC_OC_DEFERRED)) & 15u;
      case 33: return rsv;
      case 34: return rrf;
      case 35: return pop(dq);
      case 36: return (u32)(hist >> (4 * RKC_OC_RELAXED)) & 15u;
      case 37: return rdem;
      case 38: return offc;
      case 39: return offb;
      case 40: return rest;
      case 41: return t2pk;
      default: return 0;
    }
  }

  // The pool's replay: outcomes at out, telemetry at ptel, claim records at rec.
  RKC_TINY_FN void run(const rkc_pool_desc& d, const rkc_event* e, rkc_outcome* out, rkc_pool_telemetry* ptel,
                       rkc_claim_telemetry* rec) {
    const u32 ne = (u32)d.n_events;
    U = (u32)d.usable_blocks; mode = (u32)(d.mode & ~RKC_MODE_RELAX); nch = (u32)d.n_chains;
    maxq = (u32)d.max_live_claims; maxr = (u32)d.max_live_requests; nslots = (u32)d.n_claim_slots;
    dlim = (u32)d.defer_limit; relax_on = (d.mode & RKC_MODE_RELAX) != 0; t2cap = (u32)d.offload_blocks;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      rkc_event x = {{RKC_EV_NOP, 0, 0, 0}};
      if ((u32)u < ne) x = e[u];
      RKC_UNROLL for (int k = 0; k < 4; k++) ev[u].w[k] = (u32)x.w[k];
      rq_c[u] = NONE; rq_R[u] = rq_len[u] = 0;
      cl[u] = Claim{0, NONE, NONE, NONE, NONE, NONE, 0};
      ch_id[u] = to_c[u] = NONE; ch_n[u] = to_x[u] = run_lo[u] = run_top[u] = 0;
    }
    rq_live = cl_live = slots = dq = 0; dq_cnt = 1;
    F = U; A = peak = status = t2 = t2pk = nslot = evicted = 0;
    hist = 0;
    decs = vic = res = post = dropped = hits = nharm = npf = nexp = ndem = nrel = rsv = rrf = rdem = offc = offb = rest = 0;
    for (u32 t = 0; t < ne && t < (u32)E; t++) {
      const Out o = step(t);
      out[t] = rkc_outcome{{(i32)(o.code | (o.flags << 8) | (o.n16 << 16)), o.id, o.a, o.b}};
    }
    // claim records, slot by slot in step order, then the unused slots
    u32 s = 0;
    RKC_UNROLL for (int u = 0; u < E; u++) {
      if ((slots >> u) & 1u) {
        const Claim& q = cl[u];
        // (a malformed or table-rejected claim has no meta word and reports nothing)
        const bool acc = q.m != 0 && st(q.m) != RKC_ST_REJECTED;
        rec[s] = rkc_claim_telemetry{{u, (i32)packed_of(q.m), acc ? u : -1, (i32)q.dem, (i32)q.exp, (i32)q.rel, (i32)q.pf,
                                      (i32)q.harm, (i32)q.blk, q.m ? (i32)umin(n_of(ev[u].w[2]), ev[u].w[1]) : 0}};
        s++;
      }
    }
    for (; s < nslots; s++) rec[s] = rkc_claim_telemetry{{-1, 0, -1, -1, -1, -1, -1, -1, 0, 0}};
    RKC_UNROLL for (int w = 0; w < 64; w++) ptel->w[w] = (i32)tel(w);
  }
};

// Pool `pool` of a batch of pools of at most E events (descriptor checks included).
template <int E>
RKC_TINY_FN void rkc_tiny_pool(const rkc_tiny_limits& g, const rkc_pool_desc& d, const rkc_event* events,
                               rkc_outcome* outcomes, rkc_pool_telemetry* ptel, rkc_claim_telemetry* claims) {
  const int32_t mode = d.mode & ~RKC_MODE_RELAX;
  const bool ev_ok = d.n_events >= 0 && d.event_offset >= 0 && d.event_offset + d.n_events <= g.n_events_total;
  const bool sl_ok = d.n_claim_slots >= 0 && d.claim_slot_offset >= 0 && d.claim_slot_offset + d.n_claim_slots <= g.n_slots_total;
  const bool ok = ev_ok && sl_ok && d.usable_blocks >= 1 && d.usable_blocks <= g.max_usable && mode >= 0 && mode <= 3 &&
                  d.n_events <= g.max_events && d.n_chains >= 0 && d.n_chains <= g.max_chains && d.max_live_claims >= 0 &&
                  d.max_live_claims <= g.max_claims && d.max_live_requests >= 0 && d.max_live_requests <= g.max_reqs &&
                  d.n_claim_slots <= g.max_slots && d.defer_limit >= 0 && d.offload_blocks >= 0 && d.reserved[0] == 0 &&
                  d.reserved[1] == 0 && d.reserved[2] == 0;
  if (ok) {
    rkc_tiny<E> p;
    p.run(d, events + d.event_offset, outcomes + d.event_offset, ptel, claims + d.claim_slot_offset);
  } else {
    if (ev_ok)
      for (int32_t i = 0; i < d.n_events; i++) outcomes[d.event_offset + i] = rkc_outcome{{RKC_OC_INVALID, -1, 0, 0}};
    if (sl_ok)
      for (int32_t i = 0; i < d.n_claim_slots; i++)
        claims[d.claim_slot_offset + i] = rkc_claim_telemetry{{-1, 0, -1, -1, -1, -1, -1, -1, 0, 0}};
    for (int w = 0; w < 64; w++) ptel->w[w] = w == 31 ? RKC_PS_DESCRIPTOR : w == RKC_OC_INVALID && ev_ok ? d.n_events : 0;
  }
}

#endif
