// rkc_big.hip -- the replay kernel for large pools: one wavefront per pool, 32-bit pool state in LDS.
//
// Same contract, same outputs, as the general kernel in rkc_replay.hip; serves the batches beyond the
// compact kernel's 16-bit encoding that keep to
//   usable blocks < 2^20, events per pool <= 65,536, shared chains <= 256, live requests <= 16,384,
//   claim slots <= 65,536 (any number of live claims),
// where it is the faster one: big_pays in rkc_replay.hip weighs the pools that a CU holds at a time, the
// claim table and the length of the traces.
// Such batches have few pools per CU (a pool of 262,144 blocks keeps up to 16,384 requests live), so a
// pool's step is a chain of latencies, and what the general kernel spends it on is memory: its
// live-request list in global scratch (an extend 1,700 cycles, a finish 6,200), state words re-read
// between phases, one code path for all policies.  Here:
//   - the live requests are 8 bytes each (id:16, chain:8, R:20, length:20 bits) in a ring in LDS, all
//     16,384 of them in 128 KB; a finish closes its gap from the shorter side of the ring;
//   - each chain's record (32 bytes: n, hold, prot, bottom step, extent above the bottom, covA, stack
//     top, stack bottom) is read once per event into scalar registers; every branch is wave-uniform;
//   - the pool policy selects an event loop specialized at compile time;
//   - claims are 16 bytes (id | chain, L, T, meta | duration) plus slot and blocked count, the first
//     64 in registers, one per lane, the next 192 in LDS; their steps go straight into their
//     telemetry records;
//   - touch-stack nodes take the LDS the rest leaves, then global scratch.
// Representation, eviction order and why they are exact: rkc_lean.hip.
// A step is a chain of LDS round trips (~130 cycles each), so the first 64 claims and the FIFO's
// front sit in registers, loads are issued before they are needed (free-list head, FIFO's next run,
// hold count), and touching the prefix that was touched last only rewrites a step (4.17 -> 3.52 ms
// and 60.9 -> 54.5 ms on the batches below).
// Measured against the general kernel: 64 pools of 262,144 blocks x 65,536 events 133 -> 50.5 ms (the launch
// ends with its slowest pool: of four batches the slowest takes 141 -> 62 ms, with a mean of 42 ms a pool), 512
// pools of 65,536 blocks x 4,096 events 7.72 -> 3.35 ms; 0.6 to 1 us an event.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rkc.h"
#include "rkc_big.h"
#include "rkc_guard.h"

namespace {

typedef uint32_t u32;
typedef int32_t i32;
typedef uint64_t u64;
typedef int64_t i64;

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32 lds_u32;
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(1))) u32 glb_u32;
typedef __attribute__((address_space(1))) u32x2 glb_u32x2;
typedef __attribute__((address_space(1))) u32x4 glb_u32x4;

constexpr u32 NIL = 0xFFFFFFFFu;
constexpr u32 KINF = 0xFFFFFFFFu;  // key of a chain with no candidate
constexpr u32 NEVER = 0xFFFFFFFFu;
constexpr u32 kLoopMax = 0x20000u;  // no walk of a touch stack is longer (counted down in its loop word)

enum : u32 { ST_OBSERVED = 1, ST_MATERIALIZED = 2, ST_DEMOTED = 3, ST_EXPIRED = 4, ST_RELEASED = 5, ST_HARMED = 6,
             ST_REJECTED = 7 };
enum : u32 { DEC_ACCEPTED = 1, DEC_APPROX = 2, DEC_SHADOW = 3, DEC_REJECTED = 4 };
// pool telemetry words accumulated lane-distributed
enum : u32 { TW_VICTIMS = 10, TW_RESIDENT = 11, TW_POST = 12, TW_DROPPED = 13, TW_HITS = 14,
             TW_ACCEPTED = 15, TW_HARM = 19, TW_PREDFAIL = 20, TW_EXPIRED = 21, TW_DEMOTED = 22,
             TW_RELEASED = 23, TW_RETRY_SERVED = 33, TW_RETRY_REFUSED = 34, TW_RUNTIME_DEMOTED = 37,
             TW_OFF_CLAIMS = 38, TW_OFF_BLOCKS = 39, TW_RESTORED = 40 };
// words of a claim record written when the step happens
enum : u32 { RW_DEM = 3, RW_EXST = 4, RW_PF = 6, RW_HARM = 7 };

// live-claim meta (low half of w): state[0:3) eff[3:5) hard[5] prio[6:8) pending[8] decision[9:12)
// demotable[12] best_effort[13] relaxed_by_runtime[14] offloadable[15]; the high half is the duration
constexpr u32 M_PEND = 1u << 8, M_DEMQ = 1u << 12, M_BE = 1u << 13, M_RELAXED = 1u << 14, M_OFFQ = 1u << 15;
__device__ __forceinline__ u32 m_state(u32 m) { return m & 7u; }
__device__ __forceinline__ u32 m_eff(u32 m) { return (m >> 3) & 3u; }
__device__ __forceinline__ u32 m_hard(u32 m) { return (m >> 5) & 1u; }
__device__ __forceinline__ u32 m_prio(u32 m) { return (m >> 6) & 3u; }
__device__ __forceinline__ u32 m_dec(u32 m) { return (m >> 9) & 7u; }
__device__ __forceinline__ u32 packed_of(u32 m) {
  return m_dec(m) | (m_state(m) << 4) | (m_hard(m) << 8) | (m_prio(m) << 9) | (m_eff(m) << 11) |
         (((m >> 12) & 15u) << 13);
}

// ---- wave primitives (all 64 lanes active) ----------------------------------------------------
// A value every lane holds identically, moved to a scalar register (the checking build verifies that
// the active lanes agree and counts the calls where they do not).
#ifdef RKC_CHECK_UNIFORM
__device__ unsigned int g_big_uniform_violations;
__device__ __forceinline__ u32 ufl(u32 v) {
  const u32 f = (u32)__builtin_amdgcn_readfirstlane((int)v);
  if (__ballot(v != f) != 0 && __lane_id() == (u32)__builtin_ctzll(__ballot(true)))
    atomicAdd(&g_big_uniform_violations, 1u);
  return f;
}
#else
__device__ __forceinline__ u32 ufl(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }
#endif
__device__ __forceinline__ u32x4 ufl4(u32x4 v) { return u32x4{ufl(v.x), ufl(v.y), ufl(v.z), ufl(v.w)}; }
__device__ __forceinline__ u32 rdl(u32 v, u32 l) { return (u32)__builtin_amdgcn_readlane((int)v, (int)l); }
// x mod n for wave-uniform x and 1 <= n <= 65,536, on the vector unit:
// x / n from a double-precision reciprocal (v_rcp_f64: relative error about 2^-24) refined by one
// Newton step (2^-46, so x / n is off by less than 2^-14 / n, while it is at least 1 / n below the
// next integer unless x is n - 1 short of it).  Truncated, it is the quotient or, when x is a multiple
// of n, one less; the smaller of the remainder and the remainder less n, unsigned, corrects that.
__device__ __forceinline__ u32 umod(u32 x, u32 n) {
  const double dn = (double)n;
  double r = __builtin_amdgcn_rcp(dn);
  r = __builtin_fma(r, __builtin_fma(-dn, r, 1.0), r);
  const u32 q = (u32)((double)x * r);
  const u32 m = x - q * n;
  return ufl(min(m, m - n));
}
__device__ __forceinline__ u32 sub0(u32 a, u32 b) { return a > b ? a - b : 0u; }
// The byte offset of entry i (wave-uniform) of an array of 2^SH-byte entries, in one vector instruction.
template <int SH>
__device__ __forceinline__ u32 vofs(u32 i) {
  u32 r;
  asm("v_lshlrev_b32_e64 %0, %1, %2" : "=v"(r) : "n"(SH), "s"(ufl(i)));
  return r;
}
// Entry i (wave-uniform) of the array of 2^SH-byte entries at byte `at` of the workgroup's LDS (the kernel
// has no static LDS, which the build sees to, so its dynamic LDS starts at address 0).
template <class T, int SH>
__device__ __forceinline__ __attribute__((address_space(3))) T* lat(u32 at, u32 i) {
  return (__attribute__((address_space(3))) T*)(vofs<SH>(i) + at);
}
__device__ __forceinline__ u32 wrl(u32 old, u32 v, u32 l) { return __lane_id() == l ? v : old; }
__device__ __forceinline__ u64 ballot(bool p) { return __ballot(p); }

template <int CTRL>
__device__ __forceinline__ u32 dpp(u32 v) {
  return (u32)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
struct OpMax { __device__ static u32 f(u32 a, u32 b) { return a > b ? a : b; } };
struct OpMin { __device__ static u32 f(u32 a, u32 b) { return a < b ? a : b; } };
struct OpAdd { __device__ static u32 f(u32 a, u32 b) { return a + b; } };
// Row-level butterflies (quad perms, half-row and row mirrors), then two row broadcasts that leave the
// result in lane 63 (the rows they have no source for are not used).
template <class Op>
__device__ __forceinline__ u32 wreduce(u32 v) {
  v = Op::f(v, dpp<0xB1>(v));   // quad_perm [1,0,3,2]
  v = Op::f(v, dpp<0x4E>(v));   // quad_perm [2,3,0,1]
  v = Op::f(v, dpp<0x141>(v));  // row_half_mirror
  v = Op::f(v, dpp<0x140>(v));  // row_mirror
  v = Op::f(v, dpp<0x142>(v));  // row_bcast:15
  v = Op::f(v, dpp<0x143>(v));  // row_bcast:31
  return rdl(v, 63);
}
__device__ __forceinline__ u32 wmax(u32 v) { return wreduce<OpMax>(v); }
__device__ __forceinline__ u32 wmin(u32 v) { return wreduce<OpMin>(v); }
__device__ __forceinline__ u32 wsum(u32 v) { return wreduce<OpAdd>(v); }
// lane l receives lane l + 1's value (lane 63 keeps its own)
__device__ __forceinline__ u32 shift_down(u32 v) {
  return (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
}

// chain record (two 16-byte groups)
struct G0 { u32 n, hold, prot, bt, nx, covA, stop, sbot; };

struct AllocRes { u32 ok, E, resident, post, unclaimed, hit; };

// LDS of one pool: fixed regions first, then the request ring (rkc_big_args::ring entries) and the
// touch-stack nodes.
constexpr u32 kChains = 256, kClaimsLds = 256;
constexpr u32 L_COLD = 0, L_HIST = 64, L_KEYS = 128, L_HCNT = L_KEYS + 4 * kChains, L_MARK = L_HCNT + 4 * kChains,
              L_CH = L_MARK + 64, L_CL = L_CH + 32 * kChains, L_CX = L_CL + 16 * kClaimsLds, L_RQ = L_CX + 8 * kClaimsLds;

// ---- one pool ---------------------------------------------------------------------------------
// MODE: the pool policy; EXT: a hard-protection pool that defers or relaxes.
template <int MODE, bool EXT>
struct Big {
  static constexpr u32 mode = MODE;
  u32 lane;
  u32 cst;  // lane 0 U, 1 chains, 2 live-claim cap, 3 live-request cap, 4 claim slots, 5 node cap,
            // 6 defer limit, 7 relaxation on, 8 second-tier capacity
  __device__ __forceinline__ u32 U() const { return rdl(cst, 0); }
  __device__ __forceinline__ u32 nch() const { return rdl(cst, 1); }
  __device__ __forceinline__ u32 maxq() const { return rdl(cst, 2); }
  __device__ __forceinline__ u32 maxr() const { return rdl(cst, 3); }
  __device__ __forceinline__ u32 nslots() const { return rdl(cst, 4); }
  __device__ __forceinline__ u32 ncap() const { return rdl(cst, 5); }
  __device__ __forceinline__ u32 dlim() const { return rdl(cst, 6); }
  __device__ __forceinline__ u32 relax_on() const { return rdl(cst, 7); }
  __device__ __forceinline__ u32 t2cap() const { return rdl(cst, 8); }
  __device__ __forceinline__ static constexpr bool softl() { return MODE & 1; }
  __device__ __forceinline__ static constexpr bool shadm() { return !(MODE & 1); }
  __device__ __forceinline__ static constexpr bool hardm() { return MODE == RKC_MODE_HARD; }
  __device__ __forceinline__ static constexpr bool noadm() { return MODE == RKC_MODE_NOADMIT; }
  __device__ __forceinline__ static constexpr bool ext() { return MODE == RKC_MODE_HARD && EXT; }
  __device__ __forceinline__ static bool offl(u32 m) { return ext() && m_eff(m) == RKC_PROT_OFFLOADED; }

  // memory
  lds_u32* cold;
  lds_u32* hist;
  lds_u32* kk;       // eviction key per chain: level << 25 | last use << 9 | chain + 1
  lds_u32* hcnt;     // live requests holding exactly the chain's hold
  lds_u32* mark;     // 256 chain bits: chains to recompute
  lds_u32x4* ch;
  lds_u32x4* cll;    // claims [64, 256)
  lds_u32x2* cxl;
  glb_u32x4* clg;    // claims past them
  glb_u32x2* cxg;
  lds_u32x2* rq;     // ring
  u32 rmask, rhead;
  lds_u32x4* ndl;    // nodes: extent, step, up (newer), down (older)
  glb_u32x4* ndg;
  u32 nl;
  glb_u32x2* fifo;   // finished requests' private runs: low end:20 step_lo:12 | top:20 step_hi:4
  glb_u32x2* slot2;  // per slot: L | chain << 20, and NEVER or a rejected claim's id | packed word
  glb_u32x4* dq;     // deferred requests: PREFILL step, S, chain, P
  rkc_claim_telemetry* rec;
  __device__ __forceinline__ static u32 pack_rejected(u32 id, u32 packed) {
    return id | ((packed & 0x7FFFu) | ((packed >> 16) << 15)) << 16;
  }

  u32 tv;  // pool telemetry word `lane`
  u32 F, A, PR, peak, E;
  u32 nreq, ncl, nexp, sweep_due, vic, post, nslot;
  // FIFO of private runs: head, tail, the front run's eviction key (KINF when there is none) and
  // bounds, and the run behind it (loaded ahead, so that taking a whole run does not wait for memory)
  u32 qh, qt, fkey, flo, ftop;
  u32x2 fnext;
  __device__ __forceinline__ static u32x2 run_pack(u32 t, u32 lo, u32 top) { return u32x2{lo | (t << 20), top | ((t >> 12) << 20)}; }
  __device__ __forceinline__ void fifo_pop() {
    qh++;
    fkey = KINF;
    if (qh != qt) {
      const u32 a = ufl(fnext.x), b = ufl(fnext.y);
      fkey = ((a >> 20) | ((b >> 20) << 12)) << 9;
      flo = a & 0xFFFFFu;
      ftop = b & 0xFFFFFu;
      if (qh + 1 != qt) fnext = fifo[qh + 1];
    }
  }
  __device__ __forceinline__ void fifo_push(u32 t, u32 lo, u32 top) {
    const u32x2 e = run_pack(t, lo, top);
    if (qh == qt) {
      fkey = t << 9;
      flo = lo;
      ftop = top;
    } else if (qh + 1 == qt) {
      fnext = e;
    }
    fifo[qt] = e;  // every lane, one value
    qt++;
  }
  // scalars that only a few paths touch
  enum : u32 { C_STATUS = 0, C_T2, C_DQH, C_DQL, C_DQC, C_T2PK, C_WORDS };
  __device__ __forceinline__ u32 cget(u32 w) const { return ufl(cold[w]); }
  __device__ __forceinline__ void set_status(u32 bits) { cold[C_STATUS] = cget(C_STATUS) | bits; }

  __device__ __forceinline__ void tadd(u32 w, u32 v) {
    asm volatile("" : "+s"(w));  // (the lane comparison stays where it is used)
    tv += lane == w ? v : 0u;
  }

  // -- chain records --
  __device__ __forceinline__ G0 rd0(u32 c) {
    const lds_u32x4* r = lat<u32x4, 5>(L_CH, c);
    const u32x4 a = r[0], b = r[1];
    return G0{ufl(a.x), ufl(a.y), hardm() ? ufl(a.z) : 0u, ufl(a.w), ufl(b.x), ufl(b.y), ufl(b.z), ufl(b.w)};
  }
  __device__ __forceinline__ void wr0(u32 c, const G0& g) {
    lds_u32x4* r = lat<u32x4, 5>(L_CH, c);
    r[0] = u32x4{g.n, g.hold, g.prot, g.bt};
    r[1] = u32x4{g.nx, g.covA, g.stop, g.sbot};
  }
  __device__ __forceinline__ u32 chain_n(u32 c) { return ((lds_u32*)(ch + 2 * c))[0]; }
  __device__ __forceinline__ u32 chain_hold(u32 c) { return ((lds_u32*)(ch + 2 * c))[1]; }

  // -- live requests: R:20 chain:8 id_hi:4 | length:20 id_lo:12 (a request without a chain has R = 0) --
  __device__ __forceinline__ static u32x2 rq_pack(u32 id, u32 c, u32 R, u32 len) {
    return u32x2{R | (c << 20) | ((id >> 12) << 28), len | (id << 20)};
  }
  __device__ __forceinline__ static u32 rq_id(u32x2 e) { return ((e.x >> 28) << 12) | (e.y >> 20); }
  __device__ __forceinline__ static u32 rq_c(u32x2 e) { return (e.x >> 20) & 255u; }
  __device__ __forceinline__ static u32 rq_R(u32x2 e) { return e.x & 0xFFFFFu; }
  __device__ __forceinline__ static u32 rq_len(u32x2 e) { return e.y & 0xFFFFFu; }
  __device__ __forceinline__ u32 ring(u32 j) const { return (rhead + j) & rmask; }
  // Entries [lo, hi), at most 64 KU of them, move by one place (D = -1 or 1).  All are loaded before any is
  // stored.  Where neither side wraps around the ring, one address with constant offsets serves every
  // access; entries past hi are loaded with the rest and not stored.
  template <int KU, int D>
  __device__ __forceinline__ void rq_move(u32 lo, u32 hi) {
    const u32 p = ring(lo);
    u32x2 v[KU];
    if (__builtin_expect(p >= 1u && p + 64u * KU <= rmask, 1)) {
      lds_u32x2* q = rq + p + lane;
#pragma unroll
      for (int u = 0; u < KU; u++) v[u] = q[64 * u];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < KU; u++)
        if (lo + 64u * u + lane < hi) q[64 * u + D] = v[u];
    } else {
#pragma unroll
      for (int u = 0; u < KU; u++) v[u] = rq[ring(lo + 64u * u + lane)];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < KU; u++)
        if (lo + 64u * u + lane < hi) rq[ring(lo + 64u * u + lane + D)] = v[u];
    }
    __builtin_amdgcn_wave_barrier();
  }
  // Entries [i, n) move down one place (closing a gap below them) or up one place (opening one at i), in
  // rounds that run away from the destination, so that no store lands on an entry a later round loads:
  // rounds of 512 entries, the last 128 in rounds of their own (a round costs its chunks, full or not).
  __device__ __forceinline__ void rq_down(u32 i, u32 n) {
    while (n > i + 128) {
      const u32 hi = min(n, i + 512);
      rq_move<8, -1>(i, hi);
      i = hi;
    }
    if (n > i) rq_move<2, -1>(i, n);
  }
  __device__ __forceinline__ void rq_up(u32 i, u32 n) {
    while (n > i + 128) {
      const u32 lo = n > i + 512 ? n - 512 : i;
      rq_move<8, 1>(lo, n);
      n = lo;
    }
    if (n > i) rq_move<2, 1>(i, n);
  }
  // Remove entry i of nreq, closing the gap from its shorter side.
  __device__ __forceinline__ void rq_remove(u32 i) {
    if (2 * i + 1 < nreq) {
      rq_up(0, i);
      rhead = (rhead + 1) & rmask;
    } else {
      rq_down(i + 1, nreq);
    }
    nreq--;
  }
  // Insert e at its id-ordered place.
  __device__ __forceinline__ void rq_insert(u32x2 e) {
    const u32 id = ufl(rq_id(e));
    u32 below = 0;
    for (u32 base = 0; base < nreq; base += 64) {
      const u32 j = base + lane;
      below += (u32)(j < nreq && rq_id(rq[ring(j)]) < id);
    }
    const u32 k = wsum(below);
    rq_up(k, nreq);
    rq[ring(k)] = e;
  }
  // largest R of the live requests on chain c, and how many hold it
  __device__ __forceinline__ u32 rq_hold(u32 c, u32& cnt) {
    u32 m = 0, k = 0;
#pragma unroll 4
    for (u32 base = 0; base < nreq; base += 64) {
      const u32 j = base + lane;
      const u32x2 e = rq[ring(j)];
      const u32 R = j < nreq && rq_c(e) == c ? rq_R(e) : 0u;
      k = R > m ? 1u : k + (u32)(R == m);
      m = max(m, R);
    }
    const u32 hm = wmax(m);
    cnt = wsum(m == hm ? k : 0u);
    return hm;
  }

  // -- touch-stack nodes --
  __device__ __forceinline__ u32x4 nget(u32 i) {
    u32x4 v;
    if (__builtin_expect(i < nl, 1)) v = ndl[i]; else v = ndg[i - nl];
    return ufl4(v);
  }
  __device__ __forceinline__ void nset(u32 i, u32x4 v) {
    if (__builtin_expect(i < nl, 1)) ndl[i] = v; else ndg[i - nl] = v;
  }
  __device__ __forceinline__ void nset_links(u32 i, u32 up, u32 down) {
    if (__builtin_expect(i < nl, 1)) ((lds_u32x2*)(ndl + i))[1] = u32x2{up, down};
    else ((glb_u32x2*)(ndg + (i - nl)))[1] = u32x2{up, down};
  }
  __device__ __forceinline__ void nset_t(u32 i, u32 t) {
    if (__builtin_expect(i < nl, 1)) ((lds_u32*)(ndl + i))[1] = t; else ((glb_u32*)(ndg + (i - nl)))[1] = t;
  }
  // free list (its head stays in a vector register: the next head's load is not waited for here)
  u32 fnode, bump;
  __device__ __forceinline__ u32 nalloc() {
    u32 i = ufl(fnode);
    if (i != NIL) {
      if (__builtin_expect(i < nl, 1)) fnode = ndl[i].w; else fnode = ndg[i - nl].w;
    } else if (bump < ncap()) {
      i = bump++;
    } else {
      set_status(0x80000000u);  // cannot happen: one node per touch, at most node cap - 2 touches
      i = 0;
    }
    return i;
  }
  __device__ __forceinline__ void nfree(u32 i) {
    nset_links(i, NIL, fnode);
    fnode = i;
  }

  __device__ __forceinline__ static u32 evictable(u32 n, u32 hold, u32 prot) { return sub0(n, max(hold, prot)); }

  // -- claims: chunk 0 (claims 0..63) in registers, one per lane; chunks 1 to 3 in LDS, the rest in
  //    global scratch --
  u32x4 q0;  // id | chain << 16, L, T, meta | duration << 16
  u32x2 x0;  // slot, blocked count
  __device__ __forceinline__ u32x4 cl_ld(u32 base) const {  // this lane's claim of the chunk at base
    u32x4 v;
    if (base == 0) v = q0; else if (base < kClaimsLds) v = cll[base + lane]; else v = clg[base - kClaimsLds + lane];
    return v;
  }
  __device__ __forceinline__ u32x2 cx_ld(u32 base) const {
    u32x2 v;
    if (base == 0) v = x0; else if (base < kClaimsLds) v = cxl[base + lane]; else v = cxg[base - kClaimsLds + lane];
    return v;
  }
  // f(base, claim of this lane, whether it is live) over the chunks
  template <class Fn>
  __device__ __forceinline__ void claims(Fn f) const {
    f(0u, q0, lane < ncl);
    for (u32 base = 64; __builtin_expect(base < ncl, 0); base += 64) f(base, cl_ld(base), base + lane < ncl);
  }
  // the meta word, or the blocked count, of this lane's claim of a chunk where p holds
  __device__ __forceinline__ void cl_set_w(u32 base, bool p, u32 w) {
    if (base == 0) q0.w = p ? w : q0.w;
    else if (p) {
      if (base < kClaimsLds) ((lds_u32*)(cll + base + lane))[3] = w;
      else ((glb_u32*)(clg + (base - kClaimsLds + lane)))[3] = w;
    }
  }
  __device__ __forceinline__ void cx_set_blk(u32 base, bool p, u32 b) {
    if (base == 0) x0.y = p ? b : x0.y;
    else if (p) {
      if (base < kClaimsLds) ((lds_u32*)(cxl + base + lane))[1] = b;
      else ((glb_u32*)(cxg + (base - kClaimsLds + lane)))[1] = b;
    }
  }
  // claim j (wave-uniform)
  __device__ __forceinline__ void cl_put(u32 j, u32x4 v, u32x2 x) {
    if (j < 64) {
      const bool me = lane == j;
      q0.x = me ? v.x : q0.x; q0.y = me ? v.y : q0.y; q0.z = me ? v.z : q0.z; q0.w = me ? v.w : q0.w;
      x0.x = me ? x.x : x0.x; x0.y = me ? x.y : x0.y;
    } else if (j < kClaimsLds) { cll[j] = v; cxl[j] = x; } else { clg[j - kClaimsLds] = v; cxg[j - kClaimsLds] = x; }
  }
  __device__ __forceinline__ u32x4 cl_get(u32 j) const {
    u32x4 v;
    if (j < 64) {
      v = u32x4{rdl(q0.x, j), rdl(q0.y, j), rdl(q0.z, j), rdl(q0.w, j)};
    } else {
      if (j < kClaimsLds) v = cll[j]; else v = clg[j - kClaimsLds];
      v = ufl4(v);
    }
    return v;
  }
  __device__ __forceinline__ u32x2 cx_get(u32 j) const {
    u32x2 v;
    if (j < 64) {
      v = u32x2{rdl(x0.x, j), rdl(x0.y, j)};
    } else {
      if (j < kClaimsLds) v = cxl[j]; else v = cxg[j - kClaimsLds];
      v = u32x2{ufl(v.x), ufl(v.y)};
    }
    return v;
  }
  // lane-parallel writes to claims in global scratch reach later reads by other lanes
  __device__ __forceinline__ void cl_fence() {
    if (__builtin_expect(ncl > kClaimsLds, 0)) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ static u32 c_id(u32x4 v) { return v.x & 0xFFFFu; }
  __device__ __forceinline__ static u32 c_ch(u32x4 v) { return v.x >> 16; }
  __device__ __forceinline__ static u32 lo16(u32 v) { return v & 0xFFFFu; }
  __device__ __forceinline__ static bool leveled(u32 m) {
    return (m_state(m) == ST_MATERIALIZED && m_eff(m) == RKC_PROT_SOFT) || m_state(m) == ST_DEMOTED;
  }
  __device__ __forceinline__ static bool hmat(u32 m) { return m_state(m) == ST_MATERIALIZED && m_eff(m) == RKC_PROT_HARD; }
  // soft level of position p of chain c
  __device__ __forceinline__ u32 level_of(u32 c, u32 p) const {
    u32 v = 0;
    claims([&](u32, u32x4 q, bool lv) {
      const bool on = lv && c_ch(q) == c && leveled(lo16(q.w)) && q.y > p;
      v = max(v, on ? m_prio(q.w) + 1u : 0u);
    });
    return wmax(v);
  }
  // positions at or above the result have a level <= lvl
  __device__ __forceinline__ u32 level_floor(u32 c, u32 lvl) const {
    u32 v = 0;
    claims([&](u32, u32x4 q, bool lv) {
      const bool on = lv && c_ch(q) == c && leveled(lo16(q.w)) && m_prio(q.w) + 1u > lvl;
      v = max(v, on ? q.y : 0u);
    });
    return wmax(v);
  }

  // Key of chain c's top run; advances a stale stack bottom (the node above it reaches n).
  __device__ __forceinline__ u32 top_key(u32 c, G0& g, bool& moved) {
    u32 key = KINF;
    if (g.n > max(g.hold, g.prot)) {
      if (g.nx >= g.n) {
        moved = true;
        u32 b = g.sbot;
        u32x4 nb = nget(b);
        u32 up = nb.z, nxv = 0;
        u32 left = up != NIL ? kLoopMax : 0u;
        while (left) {
          const u32x4 nu = nget(up);
          nxv = nu.x;
          if (nxv >= g.n) {
            nfree(b);  // node b leaves the stack; up becomes the bottom
            b = up;
            nb = nu;
            up = nb.z;
            nxv = 0;
            left = up != NIL ? left - 1u : 0u;
          } else {
            left = 0;
          }
        }
        nset_links(b, up, NIL);
        g.sbot = b;
        g.bt = nb.y;
        g.nx = nxv;
      }
      const u32 lvl = (softl() && g.covA >= g.n) ? level_of(c, g.n - 1) : 0u;
      key = (lvl << 25) | (g.bt << 9) | (c + 1);
    }
    return key;
  }

  // Record a touch of positions [0, x) of chain c at step t (x > 0).
  __device__ __forceinline__ void touch(G0& g, u32 x, u32 t) {
    u32 tp = g.stop, tpd = NIL, reuse = NIL, same = 0;
    u32 left = tp != NIL ? kLoopMax : 0u;
    while (left) {
      const u32x4 nt = nget(tp);
      tpd = nt.w;
      if (nt.x < x) {
        // the node leaves the stack; the last one to leave becomes the new node
        if (reuse != NIL) nfree(reuse);
        reuse = tp;
        tp = tpd;
        left = tp != NIL ? left - 1u : 0u;
      } else {
        same = nt.x == x;
        left = 0;
      }
    }
    u32 st = tp, sb = g.sbot, bt = g.bt, nx = g.nx;
    if (same) {
      // the extent is on the stack already (the same prefix touched again): only its step changes
      nset_t(tp, t);
      const bool bottom = tp == sb;
      if (reuse != NIL) {
        nfree(reuse);
        nset_links(tp, NIL, tpd);
        nx = bottom ? 0u : nx;
      }
      bt = bottom ? t : bt;
    } else {
      st = reuse != NIL ? reuse : nalloc();
      nset(st, u32x4{x, t, NIL, tp});
      if (tp != NIL) {
        nset_links(tp, st, tpd);
        nx = tp == sb ? x : nx;
      } else {
        sb = st;
        bt = t;
        nx = 0;
      }
    }
    g.stop = st; g.sbot = sb; g.bt = bt; g.nx = nx;
  }

  // Apply new (n, hold, prot) to chain c, optionally touch [0, x) at t, refresh the key and store.
  __device__ __forceinline__ void commit(u32 c, G0 g, u32 nn, u32 hh, u32 pp, u32 x, u32 t) {
    E += evictable(nn, hh, pp) - evictable(g.n, g.hold, g.prot);
    if (hardm()) PR += sub0(pp, hh) - sub0(g.prot, g.hold);
    g.n = nn; g.hold = hh; g.prot = pp;
    if (x) touch(g, x, t);
    bool moved = false;
    const u32 key = top_key(c, g, moved);
    *lat<u32, 2>(L_KEYS, c) = key;
    wr0(c, g);
  }

  // After a lifecycle change of claims on chain c: the extent of its live claims, its hard
  // protection extent, and its key.
  __device__ __forceinline__ void recompute(u32 c) {
    u32 pv = 0, cv = 0;
    claims([&](u32, u32x4 q, bool lv) {
      const bool on = lv && c_ch(q) == c;
      pv = max(pv, on && hardm() && hmat(lo16(q.w)) ? q.y : 0u);
      cv = max(cv, on && !offl(q.w) ? q.y : 0u);
    });
    const u32 pp = hardm() ? wmax(pv) : 0u;
    G0 g = rd0(c);
    g.covA = wmax(cv);
    commit(c, g, g.n, g.hold, pp, 0, 0);
  }
  __device__ __forceinline__ void mark_lane(bool p, u32 c) {
    if (p) __hip_atomic_fetch_or(mark + (c >> 5), 1u << (c & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ void recompute_marked() {
    __builtin_amdgcn_wave_barrier();
    for (u32 w = 0; w < kChains / 32; w++) {
      u32 b = ufl(mark[w]);
      if (b) {
        mark[w] = 0;
        for (; b; b &= b - 1) recompute(32u * w + (u32)__builtin_ctz(b));
      }
    }
  }

  // Expiry at the start of step t (claims materialized or demoted with a duration).
  __device__ __forceinline__ void expire(u32 t, u32& flags, u32& expired) {
    u32 nx = NEVER, cnt = 0, nf = 0, drop = 0;
    claims([&](u32 base, u32x4 q, bool lv) {
      const u32 m = lo16(q.w), dur = q.w >> 16, st = m_state(m);
      const bool cand = lv && (st == ST_MATERIALIZED || st == ST_DEMOTED) && dur != 0;
      const u32 ex = c_id(q) + dur;
      const bool hit = cand && ex <= t;
      nx = min(nx, cand && !hit ? ex : NEVER);
      const u64 hb = ballot(hit);
      if (hb) {
        u32 m2 = (m & ~7u) | ST_EXPIRED;
        bool fail = false;
        if (ext()) {
          // responsibility ends: an offloaded claim's second-tier copy is dropped, and a predicate
          // that held only through it fails now (no harm: the claim is expired)
          const bool off = hit && m_eff(m) == RKC_PROT_OFFLOADED;
          drop += off ? q.y : 0u;
          fail = off && (m & M_PEND) && chain_n(hit ? c_ch(q) : 0u) < q.z;
          m2 = off ? m2 & ~(3u << 3) : m2;
          m2 = fail ? m2 & ~M_PEND : m2;
          nf += (u32)__builtin_popcountll(ballot(fail));
        }
        const u32 slot = cx_ld(base).x;
        cl_set_w(base, hit, m2 | (dur << 16));
        if (hit) {
          rec[slot].w[RW_EXST] = (i32)t;
          if (fail) rec[slot].w[RW_PF] = (i32)t;
        }
        mark_lane(hit, c_ch(q));
        cnt += (u32)__builtin_popcountll(hb);
      }
    });
    nexp = wmin(nx);
    expired = cnt;
    if (cnt) {
      if (ext()) cold[C_T2] = cget(C_T2) - wsum(drop);
      cl_fence();
      recompute_marked();
      flags |= RKC_FL_EXPIRED | (nf ? (u32)RKC_FL_PRED_FAIL : 0u);
      tadd(TW_EXPIRED, cnt);
      tadd(TW_PREDFAIL, nf);
    }
  }

  // Predicate sweep after evictions: a claim whose chain now holds fewer than T leading blocks
  // fails for the first time; a materialized (accepted) claim is harmed (§3.2).
  __device__ __forceinline__ u32 sweep(u32 t) {
    u32 pf = 0, hc = 0;
    claims([&](u32 base, u32x4 q, bool lv) {
      const u32 m = lo16(q.w);
      const u32 c = lv ? c_ch(q) : 0u;
      const bool fail = lv && (m & M_PEND) && chain_n(c) < q.z && !offl(m);
      const u64 fb = ballot(fail);
      if (fb) {
        const bool harm = fail && m_state(m) == ST_MATERIALIZED;
        const u32 m2 = (m & ~M_PEND & ~(harm ? 7u : 0u)) | (harm ? ST_HARMED : 0u);
        const u32 slot = cx_ld(base).x;
        cl_set_w(base, fail, m2 | (q.w & 0xFFFF0000u));
        if (fail) {
          rec[slot].w[RW_PF] = (i32)t;
          if (harm) rec[slot].w[RW_HARM] = (i32)t;
        }
        mark_lane(fail, c);
        pf += (u32)__builtin_popcountll(fb);
        hc += (u32)__builtin_popcountll(ballot(harm));
      }
    });
    u32 fl = 0;
    if (pf) {
      tadd(TW_PREDFAIL, pf);
      tadd(TW_HARM, hc);
      cl_fence();
      recompute_marked();
      fl = RKC_FL_PRED_FAIL | (hc ? (u32)RKC_FL_HARM : 0u);
    }
    return fl;
  }

  // ALLOC: FREE blocks first, then the (need - F) smallest-key candidates.  hc >= 0 names the chain
  // whose leading h blocks are the event's own hits (not candidates).
  __device__ __forceinline__ AllocRes alloc(u32 need, i32 hc, u32 h, const G0& ghc) {
    AllocRes r = {1, 0, 0, 0, 0, 0};
    if (need <= F) {
      F -= need;
    } else {
      u32 Ec = E;
      // candidates of chain hc start at hlo (without one the record is all zeros and nothing is taken off)
      const u32 lo = max(ghc.hold, ghc.prot), hlo = max(lo, h);
      Ec -= sub0(min(ghc.n, hlo), lo);
      r.E = Ec;
      if (need > F + Ec) {
        r.ok = 0;
      } else {
        u32 K = need - F;
        F = 0;
        const u32 K0 = K;
        vic += K;
        if (hc >= 0 && ghc.n <= hlo) *lat<u32, 2>(L_KEYS, (u32)hc) = KINF;
        // (every pass lowers K, so the loop ends whatever it meets; rkc_guard.h)
        while (K > 0) {
          const u32x4 k4 = ((lds_u32x4*)kk)[lane];
          const u32 m1 = wmin(min(min(k4.x, k4.y), min(k4.z, k4.w)));
          if (!noadm() && fkey < m1) {
            // the oldest finished request's private run (level 0)
            const u32 m = min(K, ftop - flo);
            E -= m;
            K = rkc_left(K, m);
            ftop -= m;
            if (ftop == flo) fifo_pop();
          } else if (m1 != KINF) {
            const u32 c = (m1 & 511u) - 1u;
            G0 g = rd0(c);
            const u32 nn = g.n;
            u32 lo = max(g.hold, g.prot);
            if ((i32)c == hc) { lo = max(lo, h); r.hit = 1; }
            // the top run shares (level, last use): positions below nx were touched later, positions
            // below a higher-level claim's footprint rank higher
            u32 run_lo = max(lo, g.nx);
            if (softl() && g.covA > run_lo) run_lo = max(run_lo, level_floor(c, m1 >> 25));
            const u32 m = min(K, nn - run_lo);
            const u32 nw = nn - m;
            if (g.covA > nw) {
              // victims inside live claims: resident; inside only demoted / expired ones: post-release
              u32 cv = 0, due = 0;
              claims([&](u32, u32x4 q, bool lv) {
                const u32 st = m_state(q.w);
                const u32 on = (u32)lv & (u32)(c_ch(q) == c) & (u32)!offl(q.w);
                // observed (1), materialized (2) or harmed (6)
                cv = max(cv, (on & (0x46u >> st) & 1u) ? q.y : 0u);
                due |= on & (u32)((q.w & M_PEND) != 0) & (u32)(q.z > nw);
              });
              const u32 covS = wmax(cv);
              const u32 rs = min(nn, g.covA) - nw;
              r.resident += rs;
              r.post += rs - sub0(min(nn, covS), nw);
              if (ballot(due)) sweep_due = 1;
            }
            E -= m;
            g.n = nw;
            K = rkc_left(K, m);
            bool moved = false;
            u32 key = top_key(c, g, moved);
            if (nw <= lo) key = KINF;
            *lat<u32, 2>(L_KEYS, c) = key;
            if (moved) wr0(c, g);
            else *lat<u32, 5>(L_CH, c) = g.n;
          } else {
            set_status(0x80000000u);  // cannot happen: feasibility was checked
            K = 0;
          }
        }
        r.unclaimed = K0 - r.resident;
      }
    }
    return r;
  }

  struct Out {
    u32 code, flags, n16;
    i32 id, a, b;
  };

  // Refusal record of an active event that cannot be served (§3.4; §5.4 refusal record).
  __device__ __forceinline__ void refusal(u32 need, i32 hc, u32 h, u32 Hc, const G0& ghc, Out& o) {
    u32 Pr = PR;
    if (hardm()) Pr -= sub0(min(ghc.prot, h), ghc.hold);
    const u32 req = A + Hc + need;
    o.id = -1;
    o.n16 = 0;
    if (hardm() && Pr > 0 && req <= U()) {
      o.code = RKC_OC_REFUSED_CLAIM;
      u32 mn = NEVER, nb = 0;
      claims([&](u32 base, u32x4 q, bool lv) {
        const u32 c = lv ? c_ch(q) : 0u;
        u32 cov = chain_hold(c);
        if ((i32)c == hc) cov = max(cov, h);
        const bool blk = lv && hmat(lo16(q.w)) && q.y > cov;
        const u64 bb = ballot(blk);
        if (bb) {
          cx_set_blk(base, blk, cx_ld(base).y + 1u);
          nb += (u32)__builtin_popcountll(bb);
          mn = min(mn, blk ? c_id(q) : NEVER);
        }
      });
      o.id = (i32)wmin(mn);
      o.n16 = min(nb, 65535u);
      cl_fence();
    } else {
      o.code = RKC_OC_REFUSED_CAPACITY;
    }
    o.a = (i32)Pr;
    o.b = (i32)req;
  }

  __device__ __forceinline__ void served(const AllocRes& r, Out& o) {
    o.code = r.resident ? RKC_OC_EVICT_RESIDENT : RKC_OC_ADMIT;
    o.a = (i32)r.resident;
    o.flags |= (r.post ? (u32)RKC_FL_POST_RELEASE_LOSS : 0u) | (r.unclaimed ? (u32)RKC_FL_EVICT_UNCLAIMED : 0u);
    post += r.post;
  }

  __device__ __forceinline__ void dq_pop(u32 dh, u32 dl) {
    cold[C_DQH] = dh + 1 == maxr() ? 0u : dh + 1;
    cold[C_DQL] = dl - 1;
    cold[C_DQC] = 1;
  }

  // Largest footprint of the materialized hard claims on chain c.
  __device__ __forceinline__ u32 hard_extent(u32 c) const {
    u32 v = 0;
    claims([&](u32, u32x4 q, bool lv) { v = max(v, lv && c_ch(q) == c && hmat(lo16(q.w)) ? q.y : 0u); });
    return wmax(v);
  }

  // Runtime relaxation (§3.1 demotable, offloadable; §3.5 "relax resident claim", "offload resident"):
  // the blocking claims that allow demotion or offload are taken lowest priority first, then lowest id,
  // each offloaded when it allows it and its footprint fits the second tier's free room, else demoted
  // when it allows it, else left alone, until the allocation fits; none changes when it never does.
  // A pick changes its claim's meta word at once and is marked in the top bit of its blocked count
  // (which stays below 2^17); the marked claims are kept or changed back in one pass at the end.
  // Returns the claims relaxed.
  __device__ __forceinline__ u32 relax(u32 t, u32 need, i32 hc, u32 h, G0& ghc) {
    u32 k = 0;
    if (relax_on() && need > F) {
      u32 Ec = E;
      if (hc >= 0) {
        const u32 lo = max(ghc.hold, ghc.prot);
        Ec -= sub0(min(ghc.n, max(lo, h)), lo);
      }
      u32 avail = F + Ec;
      if (need > avail) {
        u32 room = sub0(t2cap(), cget(C_T2)), moved = 0, no = 0, from = 0;
        bool go = true;
        for (u32 guard = 0; go && need > avail && guard <= ncl; guard++) {
          u32 best = NEVER, bj = 0;
          claims([&](u32 base, u32x4 q, bool lv) {
            const u32 c = lv ? c_ch(q) : 0u;
            u32 cov = chain_hold(c);
            if ((i32)c == hc) cov = max(cov, h);
            const u32 key = (m_prio(q.w) << 16) | c_id(q);
            const bool cand = lv && hmat(lo16(q.w)) && (q.w & (M_DEMQ | M_OFFQ)) && q.y > cov && key >= from && key < best;
            best = cand ? key : best;
            bj = cand ? base + lane : bj;
          });
          const u32 wb = wmin(best);
          if (wb == NEVER) {
            go = false;
          } else {
            from = wb + 1;
            const u32 j = rdl(bj, (u32)__builtin_ctzll(ballot(best == wb)));
            const u32x4 q = cl_get(j);
            const u32 m = lo16(q.w), L = q.y, c = c_ch(q);
            const bool off = (m & M_OFFQ) && L <= room;
            if (off || (m & M_DEMQ)) {
              if (off) { room -= L; moved += L; no++; }
              const u32 before = hard_extent(c);
              const u32 m2 = (off ? (m & ~(3u << 3)) | (RKC_PROT_OFFLOADED << 3) : (m & ~7u) | ST_DEMOTED) | M_RELAXED;
              cl_put_w(j, m2 | (q.w & 0xFFFF0000u));
              cx_put_blk(j, cx_get(j).y | kPicked);
              cl_fence();
              const u32 after = hard_extent(c);
              const G0 g = rd0(c);
              const u32 base = (i32)c == hc ? max(g.hold, h) : g.hold;
              avail += evictable(g.n, base, after) - evictable(g.n, base, before);
              k++;
            }
          }
        }
        const bool fits = need <= avail;
        if (k > 0) {
          claims([&](u32 base, u32x4 q, bool lv) {
            const u32x2 x = cx_ld(base);
            const bool p = lv && (x.y & kPicked);
            const u32 m = lo16(q.w);
            const bool off = m_eff(m) == RKC_PROT_OFFLOADED;
            cx_set_blk(base, p, x.y & ~kPicked);
            if (fits) {
              if (p && !off) rec[x.x].w[RW_DEM] = (i32)t;
            } else {
              const u32 m2 = (off ? (m & ~(3u << 3)) | (RKC_PROT_HARD << 3) : (m & ~7u) | ST_MATERIALIZED) & ~M_RELAXED;
              cl_set_w(base, p, m2 | (q.w & 0xFFFF0000u));
            }
            mark_lane(p && fits, c_ch(q));
          });
        }
        if (k) cl_fence();
        if (fits) {
          recompute_marked();
          tadd(TW_RUNTIME_DEMOTED, k - no);
          if (no) {
            const u32 used = cget(C_T2) + moved;
            cold[C_T2] = used;
            cold[C_T2PK] = max(cget(C_T2PK), used);
            tadd(TW_OFF_CLAIMS, no);
            tadd(TW_OFF_BLOCKS, moved);
          }
          if (hc >= 0) ghc = rd0((u32)hc);
        } else {
          k = 0;
        }
      }
    }
    return k;
  }
  static constexpr u32 kPicked = 1u << 31;
  __device__ __forceinline__ void cx_put_blk(u32 j, u32 b) {
    if (j < 64) x0.y = lane == j ? b : x0.y;
    else if (j < kClaimsLds) ((lds_u32*)(cxl + j))[1] = b;
    else ((glb_u32*)(cxg + (j - kClaimsLds)))[1] = b;
  }
  __device__ __forceinline__ void cl_put_w(u32 j, u32 w) {
    if (j < 64) q0.w = lane == j ? w : q0.w;
    else if (j < kClaimsLds) ((lds_u32*)(cll + j))[3] = w;
    else ((glb_u32*)(clg + (j - kClaimsLds)))[3] = w;
  }

  // Serve request rid (S blocks, shared chain cc when P > 0, shared prefix P) at step t; late: a
  // retried request, inserted into the live list by id and taken off the deferral ring (dh, dl).
  __device__ __forceinline__ void admit(u32 t, u32 rid, u32 S, u32 cc, u32 P, bool late, u32 dh, u32 dl, Out& o) {
    i32 hc = -1;
    u32 h = 0, Hc = 0, hk = 0;
    G0 g = {0, 0, 0, 0, 0, 0, 0, 0};
    if (P > 0) {
      hc = (i32)cc;
      hk = *lat<u32, 2>(L_HCNT, cc);
      g = rd0(cc);
      h = min(P, g.n);
      Hc = sub0(h, g.hold);
    }
    const u32 need = S - h;
    u32 relaxed = 0;
    if (ext()) relaxed = relax(t, need, hc, h, g);
    const AllocRes r = alloc(need, hc, h, g);
    if (!r.ok) {
      refusal(need, hc, h, Hc, g, o);
      if (ext()) {
        const bool by_claim = o.code == RKC_OC_REFUSED_CLAIM;
        if (late) {
          const u32 cnt = cget(C_DQC);
          if (by_claim && cnt < dlim()) {
            cold[C_DQC] = cnt + 1;
            o.code = RKC_OC_DEFERRED;
          } else {
            dq_pop(dh, dl);
            tadd(TW_RETRY_REFUSED, 1);
          }
        } else if (by_claim && dlim() > 0) {
          const u32 h0 = cget(C_DQH), l0 = cget(C_DQL);
          if (l0 < maxr()) {
            const u32 slot = h0 + l0 >= maxr() ? h0 + l0 - maxr() : h0 + l0;
            dq[slot] = u32x4{t, S, cc, P};  // every lane, one value
            cold[C_DQL] = l0 + 1;
            o.code = RKC_OC_DEFERRED;
          }
        }
      }
    } else {
      A += Hc + need;
      u32 R = 0;
      if (hc >= 0) {
        const G0 g2 = r.hit ? rd0(cc) : g;  // victims may have shortened this chain above the hits
        R = noadm() ? h : P;
        const u32 nn = (!noadm() && P > g2.n) ? P : g2.n;
        // (the chain's hold is the largest R of its live requests; hcnt counts those holding it)
        if (R > 0 && R >= g2.hold) *lat<u32, 2>(L_HCNT, cc) = R > g2.hold ? 1u : hk + 1u;
        commit(cc, g2, nn, max(g2.hold, R), g2.prot, R, t);
      }
      const u32x2 e = rq_pack(rid, hc >= 0 ? cc : 0u, R, S);
      if (late) {
        rq_insert(e);
        dq_pop(dh, dl);
        tadd(TW_RETRY_SERVED, 1);
      } else {
        *lat<u32x2, 3>(L_RQ, ring(nreq)) = e;
      }
      nreq++;
      o.id = (i32)rid;
      o.b = (i32)h;
      served(r, o);
      if (relaxed) { o.code = RKC_OC_RELAXED; o.n16 = min(relaxed, 65535u); }
      if (ext() && P > h && t2cap() > 0) {
        // positions past the hits that a claim holding a second-tier copy covers are restored
        u32 ev = 0;
        claims([&](u32, u32x4 q, bool lv) {
          ev = max(ev, lv && c_ch(q) == cc && m_eff(q.w) == RKC_PROT_OFFLOADED ? q.y : 0u);
        });
        tadd(TW_RESTORED, sub0(min(P, wmax(ev)), h));
      }
    }
  }

  __device__ __forceinline__ void ev_prefill(u32 t, u32 w1, u32 w2, u32 w3, u32 bad, Out& o) {
    if (__builtin_expect(bad, 0)) {
      o.code = RKC_OC_INVALID;
    } else if (__builtin_expect(nreq >= maxr(), 0)) {
      o.code = RKC_OC_INVALID;
      set_status(RKC_PS_REQUEST_TABLE);
    } else {
      admit(t, t, w1, w2, w3, false, 0, 0, o);
    }
  }

  __device__ __forceinline__ void ev_retry(u32 t, Out& o) {
    const u32 dh = cget(C_DQH), dl = cget(C_DQL);
    if (dl > 0) {
      if (nreq >= maxr()) {
        o.code = RKC_OC_INVALID;  // the request stays queued
        set_status(RKC_PS_REQUEST_TABLE);
      } else {
        const u32x4 q = ufl4(dq[dh]);
        admit(t, q.x, q.y, q.z, q.w, true, dh, dl, o);
      }
    }
  }

  __device__ __forceinline__ void ev_extend(u32 t, u32 w1, u32 w2, u32 bad, Out& o) {
    if (__builtin_expect(bad, 0)) {
      o.code = RKC_OC_INVALID;
    } else if (__builtin_expect(nreq > 0, 1)) {
      const u32 need = w1, at = ring(umod(w2, nreq));
      lds_u32x2* ep = lat<u32x2, 3>(L_RQ, at);
      const u32x2 e = *ep;  // (in flight over the allocation)
      G0 g = {0, 0, 0, 0, 0, 0, 0, 0};
      u32 relaxed = 0;
      if (ext()) relaxed = relax(t, need, -1, 0, g);
      const AllocRes r = alloc(need, -1, 0, g);
      if (!r.ok) {
        refusal(need, -1, 0, 0, g, o);
      } else {
        A += need;
        ((lds_u32*)ep)[1] = e.y + need;  // (a length stays below 2^20: it never exceeds U)
        o.id = (i32)ufl(rq_id(e));
        o.b = (i32)A;
        served(r, o);
        if (relaxed) { o.code = RKC_OC_RELAXED; o.n16 = min(relaxed, 65535u); }
      }
    }
  }

  __device__ __forceinline__ void ev_claim(u32 t, u32 w0, u32 w1, u32 w2, u32 w3, u32 bad, Out& o) {
    if (__builtin_expect(nslot >= nslots(), 0)) {
      o.code = RKC_OC_INVALID;
      set_status(RKC_PS_SLOT_TABLE);
    } else {
      const u32 s = nslot++;
      bool ok = !bad;
      if (ok && ncl >= maxq()) { set_status(RKC_PS_CLAIM_TABLE); ok = false; }
      if (__builtin_expect(!ok, 0)) {
        slot2[s] = u32x2{0u, pack_rejected(t, 0)};  // every lane, one value
        o.code = RKC_OC_INVALID;
      } else {
        const u32 L = w1, c = w2, T = w3;
        const u32 hardq = (w0 >> 4) & 1u, prio = (w0 >> 5) & 3u, dur = w0 >> 16;
        const u32 beq = (w0 >> 8) & 1u;  // best effort: observed in every policy
        const u32 req_bits = (w0 & (1u << 7) ? M_DEMQ : 0u) | (beq ? M_BE : 0u) | (w0 & (1u << 9) ? M_OFFQ : 0u);
        const bool obs = shadm() || beq;
        const G0 g = rd0(c);
        const u32 h = min(L, g.n), need = L - h;
        const AllocRes r = alloc(need, (i32)c, h, g);
        const u32 eff = beq ? RKC_PROT_NONE : hardm() ? (hardq ? RKC_PROT_HARD : RKC_PROT_SOFT)
                      : (mode == RKC_MODE_SOFT ? RKC_PROT_SOFT : RKC_PROT_NONE);
        if (!r.ok) {
          const u32 dec = obs ? DEC_SHADOW : DEC_REJECTED;
          const u32 m = ST_REJECTED | (eff << 3) | (hardq << 5) | (prio << 6) | (dec << 9) | req_bits;
          // (a footprint that did not fit may exceed the pool, whose chains never do: cap it there)
          slot2[s] = u32x2{min(L, U()) | (c << 20), pack_rejected(t, packed_of(m))};
          o.code = RKC_OC_MATFAIL;
          o.id = (i32)t;
          o.a = (i32)need;
          o.b = (i32)(F + r.E);
          tadd(TW_ACCEPTED + dec - DEC_ACCEPTED, 1);
        } else {
          slot2[s] = u32x2{L | (c << 20), NEVER};
          const u32 lowered = (mode == RKC_MODE_SOFT) && hardq;
          const u32 dec = obs ? DEC_SHADOW : lowered ? DEC_APPROX : DEC_ACCEPTED;
          const u32 st = obs ? ST_OBSERVED : ST_MATERIALIZED;
          o.flags |= obs ? (u32)RKC_FL_SHADOW : lowered ? (u32)RKC_FL_LOWERED : 0u;
          const u32 m = st | (eff << 3) | (hardq << 5) | (prio << 6) | M_PEND | (dec << 9) | req_bits;
          const u32 dur_eff = obs ? 0u : dur;  // shadow claims never expire
          cl_put(ncl, u32x4{t | (c << 16), L, T, m | (dur_eff << 16)}, u32x2{s, 0u});
          if (lane == RW_DEM || lane == RW_EXST || lane == RW_PF || lane == RW_HARM) rec[s].w[lane] = -1;
          ncl++;
          cl_fence();
          if (dur_eff > 0) nexp = min(nexp, t + dur_eff);
          G0 g2 = r.hit ? rd0(c) : g;
          g2.covA = max(g2.covA, L);
          // a materialized hard claim in a hard-protection pool protects [0, L)
          const u32 pp = eff == RKC_PROT_HARD ? max(g2.prot, L) : g2.prot;
          commit(c, g2, max(g2.n, L), g2.hold, pp, L, t);
          o.id = (i32)t;
          o.b = (i32)need;
          served(r, o);
          tadd(TW_ACCEPTED + dec - DEC_ACCEPTED, 1);
        }
      }
    }
  }

  __device__ __forceinline__ void ev_finish(u32 t, u32 w1, Out& o) {
    if (nreq > 0) {
      const u32 i = umod(w1, nreq);
      const u32x2 e0 = *lat<u32x2, 3>(L_RQ, ring(i));
      const u32x2 e = u32x2{ufl(e0.x), ufl(e0.y)};
      const u32 rid = rq_id(e), c = rq_c(e), R = rq_R(e), len = rq_len(e);
      G0 g;
      u32 hk = 0;
      if (R > 0) {
        hk = *lat<u32, 2>(L_HCNT, c);
        g = rd0(c);
      }
      rq_remove(i);
      u32 turned = 0;
      if (R > 0) {
        // the hold falls only when the last request that held it finishes
        u32 hn = g.hold;
        if (R == hn) {
          hk = ufl(hk);
          if (hk > 1) {
            *lat<u32, 2>(L_HCNT, c) = hk - 1;
          } else {
            u32 cnt;
            hn = rq_hold(c, cnt);
            *lat<u32, 2>(L_HCNT, c) = cnt;
          }
        }
        turned = sub0(R, hn);
        commit(c, g, g.n, hn, g.prot, R, t);
      }
      // write no-admit drops the request's own blocks; otherwise they become a private run
      const u32 own = len - R;
      const u32 dropped = noadm() ? own : 0u, kept = own - dropped;
      turned += kept;
      F += dropped;
      E += kept;
      if (kept > 0) fifo_push(t, R, len);
      peak = max(peak, A);  // (A only falls here)
      A -= turned + dropped;
      o.code = RKC_OC_FINISHED;
      o.id = (i32)rid;
      o.a = (i32)turned;
      o.b = (i32)dropped;
      if (dropped) o.flags |= RKC_FL_NOADMIT_DROP;
      if (noadm()) tadd(TW_DROPPED, dropped);
    }
  }

  // A live claim's record words that are not written as their step happens.
  __device__ __forceinline__ void write_record(u32 j, u32 id, u32 m, u32 state, i32 rel) {
    const u32x2 x = cx_get(j);
    if (lane == 0 || lane == 1 || lane == 2 || lane == 5 || lane == 8) {
      const u32 packed = packed_of((m & ~7u) | state);
      rec[x.x].w[lane] = lane == 0 || lane == 2 ? (i32)id : lane == 1 ? (i32)packed : lane == 5 ? rel : (i32)x.y;
    }
  }

  // Claims [i + 1, ncl) move down one place.
  __device__ __forceinline__ void cl_remove(u32 i) {
    if (i < 64) {
      const bool up = lane >= i;
      q0.x = up ? shift_down(q0.x) : q0.x; q0.y = up ? shift_down(q0.y) : q0.y;
      q0.z = up ? shift_down(q0.z) : q0.z; q0.w = up ? shift_down(q0.w) : q0.w;
      x0.x = up ? shift_down(x0.x) : x0.x; x0.y = up ? shift_down(x0.y) : x0.y;
      if (__builtin_expect(ncl > 64, 0)) {
        const u32x4 v = cl_get(64);
        const u32x2 x = cx_get(64);
        cl_put(63, v, x);
      }
    }
    const u32 from = max(i, 64u);
    for (u32 base = from & ~63u; __builtin_expect(base < ncl, 0); base += 64) {
      // this chunk's entries from `from` on take their successor's value; the last lane's successor is
      // the first entry of the next chunk
      const u32 j = base + lane, src = min(j + 1, ncl - 1);
      u32x4 v;
      u32x2 x;
      if (src < kClaimsLds) { v = cll[src]; x = cxl[src]; } else { v = clg[src - kClaimsLds]; x = cxg[src - kClaimsLds]; }
      __builtin_amdgcn_wave_barrier();
      if (j >= from && j + 1 < ncl) {
        if (base < kClaimsLds) { cll[j] = v; cxl[j] = x; } else { clg[j - kClaimsLds] = v; cxg[j - kClaimsLds] = x; }
      }
      __builtin_amdgcn_wave_barrier();
    }
    cl_fence();
    ncl--;
  }

  __device__ __forceinline__ void ev_lifecycle(u32 t, u32 type, u32 w1, Out& o) {
    u32 i = NEVER;
    if (type == RKC_EV_RELEASE) {
      if (ncl > 0) i = umod(w1, ncl);
    } else if (softl()) {
      // the (w1 mod count)-th demotable claim in id order
      u32 cnt = 0;
      for (u32 base = 0; base < ncl; base += 64) {
        const u32 m = lo16(cl_ld(base).w);
        cnt += (u32)__builtin_popcountll(ballot(base + lane < ncl && m_state(m) == ST_MATERIALIZED && m_hard(m) && !offl(m)));
      }
      if (cnt > 0) {
        u32 k = umod(w1, cnt);
        for (u32 base = 0; base < ncl && i == NEVER; base += 64) {
          const u32 m = lo16(cl_ld(base).w);
          const u64 b = ballot(base + lane < ncl && m_state(m) == ST_MATERIALIZED && m_hard(m) && !offl(m));
          const u32 pc = (u32)__builtin_popcountll(b);
          if (k < pc) {
            const u32 rank = __builtin_amdgcn_mbcnt_hi((u32)(b >> 32), __builtin_amdgcn_mbcnt_lo((u32)b, 0u));
            i = base + (u32)__builtin_ctzll(ballot(((b >> lane) & 1ull) && rank == k));
          } else {
            k -= pc;
          }
        }
      }
    }
    if (i != NEVER) {
      const u32x4 q = cl_get(i);
      const u32 id = c_id(q), c = c_ch(q), m = lo16(q.w);
      if (type == RKC_EV_RELEASE) {
        write_record(i, id, m, ST_RELEASED, (i32)t);
        if (ext() && m_eff(m) == RKC_PROT_OFFLOADED) cold[C_T2] = cget(C_T2) - q.y;
        cl_remove(i);
        o.code = RKC_OC_RELEASED;
        tadd(TW_RELEASED, 1);
      } else {
        cl_put_w(i, ((m & ~7u) | ST_DEMOTED) | (q.w & 0xFFFF0000u));
        rec[cx_get(i).x].w[RW_DEM] = (i32)t;
        cl_fence();
        o.code = RKC_OC_DEMOTED;
        tadd(TW_DEMOTED, 1);
      }
      recompute(c);
      o.id = (i32)id;
      o.a = (i32)min(ufl(chain_n(c)), q.y);
      o.b = (i32)q.z;
    }
  }

  // Malformed events of a tile (lane k holds event k).
  __device__ __forceinline__ u32 malformed(u32 e0, u32 e1, u32 e2, u32 e3) const {
    const u32 ty = e0 & 15u;
    const i32 s1 = (i32)e1, s2 = (i32)e2, s3 = (i32)e3;
    const bool fb = s1 < 1 || s1 > RKC_MAX_FIELD_BLOCKS;
    const bool cb = s2 < 0 || e2 >= nch();
    const bool bad = (ty == RKC_EV_PREFILL && (fb || s3 < 0 || s3 > s1 || (s3 > 0 && cb))) ||
                     (ty == RKC_EV_EXTEND && fb) ||
                     (ty == RKC_EV_CLAIM && (fb || cb || s3 < 0 || s3 > s1));
    return (u32)bad;
  }

  __device__ __forceinline__ void step(u32 t, u32 w0, u32 w1, u32 w2, u32 w3, u32 bad, Out& o) {
    const u32 type = w0 & 15u;
    o = Out{RKC_OC_NOOP, 0, 0, -1, 0, 0};
    if (!shadm() && __builtin_expect(t >= nexp, 0)) {
      u32 expired;
      expire(t, o.flags, expired);
      o.n16 = min(expired, 65535u);
    }
    if (type == RKC_EV_PREFILL) ev_prefill(t, w1, w2, w3, bad, o);
    else if (type == RKC_EV_EXTEND) ev_extend(t, w1, w2, bad, o);
    else if (type == RKC_EV_CLAIM) ev_claim(t, w0, w1, w2, w3, bad, o);
    else if (type == RKC_EV_FINISH) ev_finish(t, w1, o);
    else if (type == RKC_EV_RELEASE || type == RKC_EV_DEMOTE) ev_lifecycle(t, type, w1, o);
    else if (ext() && type == RKC_EV_RETRY) ev_retry(t, o);
    else if ((type & ~1u) != RKC_EV_NOP) o.code = RKC_OC_INVALID;  // NOP, or RETRY with no ring
    if (__builtin_expect(sweep_due, 0)) {
      sweep_due = 0;
      o.flags |= sweep(t);
    }
  }
};

template <int MODE, bool EXT>
__device__ __forceinline__ void replay_pool(const rkc_big_args& g, const rkc_pool_desc& d, u32 pool, unsigned char* lds_raw) {
  typedef Big<MODE, EXT> BP;
  BP P;
  P.lane = __lane_id();
  const u32 l = P.lane;
  P.cst = l == 0 ? (u32)d.usable_blocks : l == 1 ? (u32)d.n_chains : l == 2 ? (u32)d.max_live_claims
        : l == 3 ? (u32)d.max_live_requests : l == 4 ? (u32)d.n_claim_slots : l == 5 ? g.node_cap
        : l == 6 ? (u32)d.defer_limit : l == 7 ? (u32)((d.mode & RKC_MODE_RELAX) != 0) : (u32)d.offload_blocks;
  const u32 U = (u32)d.usable_blocks, nslots = (u32)d.n_claim_slots;
  lds_u32* lds = (lds_u32*)lds_raw;
  P.cold = lds + L_COLD / 4;
  P.hist = lds + L_HIST / 4;
  P.kk = lds + L_KEYS / 4;
  P.hcnt = lds + L_HCNT / 4;
  P.mark = lds + L_MARK / 4;
  P.ch = (lds_u32x4*)(lds + L_CH / 4);
  P.cll = (lds_u32x4*)(lds + L_CL / 4);
  P.cxl = (lds_u32x2*)(lds + L_CX / 4);
  P.rq = (lds_u32x2*)(lds + L_RQ / 4);
  P.rmask = g.ring - 1;
  P.rhead = 0;
  P.ndl = (lds_u32x4*)(lds + (L_RQ + 8u * g.ring) / 4);
  P.nl = g.nodes_lds;
  unsigned char* scr = (unsigned char*)g.scratch + (u64)pool * g.scr_pool_bytes;
  P.ndg = (glb_u32x4*)(scr + g.scr_off_nodes);
  P.fifo = (glb_u32x2*)(scr + g.scr_off_fifo);
  P.slot2 = (glb_u32x2*)(scr + g.scr_off_slots);
  P.dq = (glb_u32x4*)(scr + g.scr_off_defer);
  P.clg = (glb_u32x4*)(scr + g.scr_off_claims);
  P.cxg = (glb_u32x2*)(scr + g.scr_off_cx);
  P.rec = g.claim_tel + d.claim_slot_offset;
  for (u32 c = l; c < kChains; c += 64) {
    P.kk[c] = KINF;
    P.hcnt[c] = 0;
    P.ch[2 * c] = u32x4{0, 0, 0, 0};
    P.ch[2 * c + 1] = u32x4{0, 0, NIL, NIL};
  }
  if (l < 16) { P.hist[l] = 0; P.mark[l] = 0; }
  if (l < BP::C_WORDS) P.cold[l] = l == BP::C_DQC ? 1u : 0u;
  P.q0 = u32x4{0, 0, 0, 0};
  P.x0 = u32x2{0, 0};
  P.tv = 0;
  P.F = U; P.A = 0; P.PR = 0; P.peak = 0; P.E = 0;
  P.nreq = 0; P.ncl = 0; P.nexp = NEVER; P.sweep_due = 0; P.vic = 0; P.post = 0; P.nslot = 0;
  P.qh = P.qt = P.flo = P.ftop = 0; P.fkey = KINF; P.fnext = u32x2{0, 0};
  P.fnode = NIL; P.bump = 0;
  __syncthreads();

  const rkc_event* __restrict__ ev = g.events + d.event_offset;
  rkc_outcome* out = g.outcomes + d.event_offset;
  const u32 ne = (u32)d.n_events;
  // the next tile's events are loaded while this one is replayed
  int4 nx = make_int4(0, 0, 0, 0);
  if (l < ne) nx = *(const int4*)(ev + l);
  for (u32 base = 0; base < ne; base += 64) {
    const u32 cnt = min(64u, ne - base);
    const int4 x = nx;
    if (base + 64 + l < ne) nx = *(const int4*)(ev + base + 64 + l);
    const u32 e0 = l < cnt ? (u32)x.x : 0u, e1 = l < cnt ? (u32)x.y : 0u, e2 = l < cnt ? (u32)x.z : 0u,
              e3 = l < cnt ? (u32)x.w : 0u;
    const u32 badv = P.malformed(e0, e1, e2, e3);
    u32 o0 = 0, o1 = 0, o2 = 0, o3 = 0;
    for (u32 k = 0; k < cnt; k++) {
      typename BP::Out o;
      P.step(base + k, rdl(e0, k), rdl(e1, k), rdl(e2, k), rdl(e3, k), rdl(badv, k), o);
      o0 = wrl(o0, o.code | (o.flags << 8) | (o.n16 << 16), k);
      o1 = wrl(o1, (u32)o.id, k); o2 = wrl(o2, (u32)o.a, k); o3 = wrl(o3, (u32)o.b, k);
    }
    const u32 oc = o0 & 255u;
    const bool quiet = oc == RKC_OC_NOOP || oc == RKC_OC_INVALID;  // id -1, a = b = 0
    o1 = quiet ? 0xFFFFFFFFu : o1; o2 = quiet ? 0u : o2; o3 = quiet ? 0u : o3;
    if (l < cnt) *(int4*)(out + base + l) = make_int4((i32)o0, (i32)o1, (i32)o2, (i32)o3);
    // outcomes per code; resident victims (a) and leading hits (b of a served prefill)
    __hip_atomic_fetch_add(P.hist + (l < cnt ? oc : 15u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const bool srv = l < cnt && (oc <= RKC_OC_EVICT_RESIDENT || (BP::ext() && oc == RKC_OC_RELAXED));
    P.tadd(TW_RESIDENT, wsum(srv ? o2 : 0u));
    const u32 ty = e0 & 15u;
    P.tadd(TW_HITS, wsum(srv && (ty == RKC_EV_PREFILL || (BP::ext() && ty == RKC_EV_RETRY)) ? o3 : 0u));
  }

  // Final records of the claims still live, then lead_end = min(final leading registered length, L)
  // of every used slot, the records of rejected claims, and blank records for unused slots.
  for (u32 j = 0; j < P.ncl; j++) {
    const u32x4 q = P.cl_get(j);
    P.write_record(j, BP::c_id(q), BP::lo16(q.w), m_state(q.w), -1);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  for (u32 s = l; s < nslots; s += 64) {
    if (s < P.nslot) {
      const u32x2 v = P.slot2[s];
      const i32 le = (i32)min(P.chain_n((v.x >> 20) & 255u), v.x & 0xFFFFFu);
      if (v.y == NEVER) {
        P.rec[s].w[9] = le;
      } else {
        const u32 pw = v.y >> 16;
        const i32 packed = (i32)((pw & 0x7FFFu) | ((pw >> 15) << 16));
        P.rec[s] = rkc_claim_telemetry{{(i32)(v.y & 0xFFFFu), packed, -1, -1, -1, -1, -1, -1, 0, le}};
      }
    } else {
      P.rec[s] = rkc_claim_telemetry{{-1, 0, -1, -1, -1, -1, -1, -1, 0, 0}};
    }
  }
  __syncthreads();
  const u32 status = P.cget(BP::C_STATUS) | (rkc_adds_up(U, P.F, P.A, P.E + P.PR) ? 0u : 0x80000000u);
  const u32 queued = P.cget(BP::C_DQL), t2peak = P.cget(BP::C_T2PK);
  i32 v = (i32)P.tv;
  if (l < 10) v += (i32)P.hist[l];
  if (l == 32) v += (i32)P.hist[RKC_OC_DEFERRED];
  if (l == 36) v += (i32)P.hist[RKC_OC_RELAXED];
  if (l == TW_VICTIMS) v = (i32)P.vic;
  else if (l == TW_POST) v = (i32)P.post;
  else if (l == 24) v = (i32)max(P.peak, P.A);
  else if (l == 25) v = (i32)P.A;
  else if (l == 26) v = (i32)(U - P.F - P.A);
  else if (l == 27) v = (i32)P.F;
  else if (l == 28) v = (i32)P.PR;
  else if (l == 29) v = (i32)P.nreq;
  else if (l == 30) v = (i32)P.ncl;
  else if (l == 31) v = (i32)status;
  else if (l == 35) v = (i32)queued;
  else if (l == 41) v = (i32)t2peak;
  g.pool_tel[pool].w[l] = v;
}

__global__ __launch_bounds__(64) void rkc_big(rkc_big_args g) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const u32 pool = blockIdx.x, lane = __lane_id();
  if ((i32)pool >= g.n_pools) return;
  const rkc_pool_desc d = g.pools[pool];
  const i64 ev_off = d.event_offset, slot_off = d.claim_slot_offset;
  const bool ev_ok = d.n_events >= 0 && ev_off >= 0 && ev_off + d.n_events <= g.n_events_total;
  const bool sl_ok = d.n_claim_slots >= 0 && slot_off >= 0 && slot_off + d.n_claim_slots <= g.n_slots_total;
  const bool ok = ev_ok && sl_ok && d.usable_blocks >= 1 && d.usable_blocks <= g.max_usable &&
                  (d.mode & ~RKC_MODE_RELAX) >= 0 && (d.mode & ~RKC_MODE_RELAX) <= 3 &&
                  d.n_events <= g.max_events && d.n_chains >= 0 &&
                  d.n_chains <= g.max_chains && d.max_live_claims >= 0 && d.max_live_claims <= g.max_claims &&
                  d.max_live_requests >= 0 && d.max_live_requests <= g.max_reqs &&
                  d.n_claim_slots <= g.max_slots && d.defer_limit >= 0 && d.offload_blocks >= 0 &&
                  d.reserved[0] == 0 && d.reserved[1] == 0 && d.reserved[2] == 0;
  if (!ok) {
    if (ev_ok)
      for (i32 i = (i32)lane; i < d.n_events; i += 64) g.outcomes[ev_off + i] = rkc_outcome{{RKC_OC_INVALID, -1, 0, 0}};
    if (sl_ok)
      for (i32 i = (i32)lane; i < d.n_claim_slots; i += 64)
        g.claim_tel[slot_off + i] = rkc_claim_telemetry{{-1, 0, -1, -1, -1, -1, -1, -1, 0, 0}};
    g.pool_tel[pool].w[lane] = lane == 31 ? RKC_PS_DESCRIPTOR : (lane == RKC_OC_INVALID && ev_ok) ? d.n_events : 0;
    return;
  }
  const u32 mode = (u32)__builtin_amdgcn_readfirstlane(d.mode & ~RKC_MODE_RELAX);
  const u32 ext = (u32)__builtin_amdgcn_readfirstlane(d.defer_limit) > 0 || (d.mode & RKC_MODE_RELAX);
  if (mode == RKC_MODE_LRU) replay_pool<RKC_MODE_LRU, false>(g, d, pool, lds_raw);
  else if (mode == RKC_MODE_SOFT) replay_pool<RKC_MODE_SOFT, false>(g, d, pool, lds_raw);
  else if (mode == RKC_MODE_NOADMIT) replay_pool<RKC_MODE_NOADMIT, false>(g, d, pool, lds_raw);
  else if (!ext) replay_pool<RKC_MODE_HARD, false>(g, d, pool, lds_raw);
  else replay_pool<RKC_MODE_HARD, true>(g, d, pool, lds_raw);
}

u64 align_up(u64 v, u64 a) { return (v + a - 1) / a * a; }

}  // namespace

bool rkc_big_layout(const rkc_batch* b, rkc_big_args* g) {
  constexpr u32 kLds = 160 * 1024, kCUs = 256, kMinNodes = 128;
  if (b->max_usable_blocks >= (1 << 20) || b->max_events > 65536 || b->max_chains > (i32)kChains ||
      b->max_live_requests > 16384 || b->max_claim_slots > 65536)
    return false;
  const u64 reqs = b->max_live_requests > 0 ? (u64)b->max_live_requests : 1u;
  const u64 claims = b->max_live_claims > 0 ? (u64)b->max_live_claims : 1u;
  u32 ring = 64;
  while (ring < reqs) ring *= 2;
  g->ring = ring;
  g->node_cap = (u32)b->max_events + 2;
  // nodes in LDS: what a pool's share of its CU leaves (LDS comes in units of 1,280 bytes), at least
  // kMinNodes
  const u32 per_cu = (u32)(((u64)b->n_pools + kCUs - 1) / kCUs);
  const u32 fixed = L_RQ + 8 * ring, share = kLds / (per_cu > 0 ? per_cu : 1) / 1280 * 1280;
  u32 nodes = share > fixed ? (share - fixed) / 16 : 0;
  nodes = nodes < kMinNodes ? kMinNodes : nodes;
  g->nodes_lds = nodes < g->node_cap ? nodes : g->node_cap;
  g->lds_bytes = fixed + 16 * g->nodes_lds;
  if (g->lds_bytes > kLds) return false;
  u64 s = 0;
  auto take = [&](u64 bytes) { const u64 r = s; s = align_up(s + bytes, 256); return r; };
  g->scr_off_nodes = take(16ull * (g->node_cap - g->nodes_lds));
  g->scr_off_fifo = take(8ull * ((u64)b->max_events + 1));
  g->scr_off_slots = take(8ull * (u64)(b->max_claim_slots > 0 ? b->max_claim_slots : 1));
  g->scr_off_defer = take(16ull * reqs);
  g->scr_off_claims = take(claims > kClaimsLds ? 16ull * align_up(claims - kClaimsLds, 64) : 0);
  g->scr_off_cx = take(claims > kClaimsLds ? 8ull * align_up(claims - kClaimsLds, 64) : 0);
  g->scr_pool_bytes = s;
  return true;
}

#ifdef RKC_CHECK_UNIFORM
unsigned rkc_big_uniform_violations(void) {
  unsigned v = 0;
  if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_big_uniform_violations), sizeof v) != hipSuccess) return ~0u;
  return v;
}
#endif

rkc_status rkc_big_launch(const rkc_big_args* g, hipStream_t s) {
  if (g->lds_bytes > 64 * 1024 &&
      hipFuncSetAttribute((const void*)rkc_big, hipFuncAttributeMaxDynamicSharedMemorySize, (int)g->lds_bytes) != hipSuccess)
    return RKC_E_HIP;
  hipLaunchKernelGGL(rkc_big, dim3((unsigned)g->n_pools), dim3(64), g->lds_bytes, s, *g);
  return hipGetLastError() == hipSuccess ? RKC_OK : RKC_E_HIP;
}
