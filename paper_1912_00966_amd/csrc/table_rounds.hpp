// table_rounds.hpp -- the relaxation rounds of a query whose arrivals live in
// the on-chip table, one connection type per lane (included by relax.hpp).
//
// What bounds it: the instructions of one wave, one after the other.  A query has
// some tens of rounds of a few hundred connection types each; a wave takes about
// ten cycles an instruction whatever the other waves do (an LDS answer 65-90, a
// condition of its lanes 25: compare, mask, branch, restore), and the barrier
// waits for the wave with the longest path.  So the path from the barrier to the
// reads of the types is kept short, no work is prepared by one wave for another
// between two barriers, and lanes that have nothing to do go along (a neutral
// operand, a spare entry at a list's end) instead of being masked:
//   * A push books its place in the next round's list and the numbers of its
//     connection types in one 64-bit LDS atomic of its lane (the LDS serialises
//     the few lanes of a wave that push; a prefix sum over the wave was 30
//     instructions) and marks the windows of 64 types right away; the next round
//     starts with its windows.
//   * A wave issues the reads of its first window before it works out what the
//     round is (end, window base, sweep), which is then hidden behind them.
//   * Decisions that all waves take alike (end, overflow, window base, sweep)
//     are made from counters of the round that has ended.  A wave may already
//     relax in the next round while another still reads them, so every round
//     has a set of its own (three in turn) and none is shared across rounds.
//   * Arrivals past the arrival window go to a far list.  It is read only when
//     its earliest arrival has come inside the window, by the waves that have
//     the fewest windows, while the others relax; what it promotes is expanded
//     a round later.  So a query can take more rounds than with run_rounds, and
//     one that hits its limit of rounds runs again with those.
// Measured against the rounds with a take pass (relax.hpp's run_rounds, which
// the slab store, virtual warps and two or three types per lane still use): a
// query of 19 rounds alone on its CU 34 us instead of 54 (city of 50,000 stops),
// 256 queries on it 155 us a launch instead of 230 (1024 threads), 3,584 queries
// over seven cities 640 us instead of 850 (768 threads, two queries a CU).
#pragma once

// Flags of a table slot, in its low word with the stop's number.  NEAR_A /
// NEAR_B: the stop is in the list of an even / odd round.  FAR_FLAG: it has an
// entry in the far list.  They only keep a stop from being listed twice; a flag
// is set right before the entry it stands for is written.  FAR_FLAG is the
// highest: a stop that the full far list turns away gets a near flag instead
// (operator() below), and an equal arrival tried with FAR_FLAG then leaves the
// slot alone.
//   A round r clears the near flag of its own list's entries and its pushes use
//   the other one, so clearing needs no barrier against pushes: an improvement
//   of round r lists the stop for round r + 1 whether the stop's entry of round
//   r has been read yet or not.
constexpr uint32_t FAR_FLAG = 0x80000000u, NEAR_A = 0x40000000u, NEAR_B = 0x20000000u;
constexpr uint32_t STOP_MASK = 0x1fffffffu;
static_assert(kMaxTableStops == (int32_t)STOP_MASK, "an empty slot's low word is no stop");

// The on-chip table: one 64-bit word per slot, {arrival, flags, stop}.  One
// 64-bit atomic minimum lowers the arrival, sets the pushed list's flag, clears
// the others and returns what the flags were.  Two lanes never write equal
// arrivals with different flags to one slot: a round's candidates below its
// threshold all carry one flag, those at or past it the other.
struct TagTable {
  unsigned long long *kv;
  uint32_t mask;
  int32_t shift;
  // Even: a stop's first two slots are read together, which ends nearly every
  // probe.  (With one slot at a time, some lane of a wave of 64 had to go on, and
  // the wave with it, in more than half of the probes from a few hundred stops on.)
  __device__ __forceinline__ uint32_t home(int32_t v) const { return (((uint32_t)v * 2654435761u) >> shift) & ~1u; }
  __device__ __forceinline__ uint32_t *lo(int32_t p) const { return reinterpret_cast<uint32_t *>(kv + p); }
  __device__ __forceinline__ unsigned long long entry(int32_t p) const {
    return __hip_atomic_load(kv + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ int32_t value(int32_t p) const {
    return lds_ld(reinterpret_cast<const int32_t *>(kv + p) + 1);
  }
  // Arrival of stop v (INF if none); pos = its slot, or the empty slot where it
  // would go (slots are never freed).  No slot left: *full is told, and the
  // arrival is 0, which nothing improves.
  __device__ __forceinline__ int32_t find(int32_t v, int32_t &pos, uint32_t *full) const {
    uint32_t p = home(v);
    // Two reads of 8 bytes, each a slot as one atomic left it: other waves write
    // these slots meanwhile, and half a new slot beside half an old one would be
    // another stop's arrival.  (One read of 16 bytes measured the same: 256 queries on
    // city-50k 155.1 us, two reads 154.4; 3,584 over seven cities 647.5 and 646.5.)
    const unsigned long long e0 = entry((int32_t)p), e1 = entry((int32_t)p + 1);
    // 0: the slot is v's (the flags shifted out) or empty.  (Minima of numbers,
    // not conditions of lanes, which pass through scalar registers.)
    const uint32_t k0 = (uint32_t)e0, k1 = (uint32_t)e1;
    const uint32_t z0 = min((k0 ^ (uint32_t)v) << 3, ~k0), z1 = min((k1 ^ (uint32_t)v) << 3, ~k1);
    pos = (int32_t)(z0 == 0u ? p : p + 1u);
    int32_t av = z0 == 0u ? (int32_t)(e0 >> 32) : (int32_t)(e1 >> 32);  // an empty slot holds INF
    const uint32_t z = min(z0, z1);
    if (__builtin_expect(__ballot(z != 0u) != 0ull, 0)) {
      if (z != 0u) {
        ++p;
        for (uint32_t n = 2;; ++n) {
          if (n > mask) {
            atomicOr(full, kTableFull);
            av = 0;
            break;
          }
          p = (p + 1u) & mask;
          const unsigned long long e = entry((int32_t)p);
          const uint32_t key = (uint32_t)e;
          if (key == NO_KEY || (key & STOP_MASK) == (uint32_t)v) {
            pos = (int32_t)p;
            av = (int32_t)(e >> 32);
            break;
          }
        }
      }
    }
    return av;
  }
  // Tries to lower v's arrival to cand < av (av, pos from find).  Returns the
  // arrival before (cand is an improvement if it is later; INF for a new stop);
  // item = v's slot, old = the flags it had (0 for a new stop), fresh = it is
  // new.  No slot left: *full is told, 0 returned.
  __device__ __forceinline__ int32_t lower(int32_t v, int32_t pos, int32_t av, int32_t cand, uint32_t flag,
                                           int32_t &item, uint32_t &old, bool &fresh, uint32_t *full) const {
    const unsigned long long want = ((unsigned long long)(uint32_t)cand << 32) | flag | (uint32_t)v;
    item = pos;
    const bool insert = av == INF;  // every stored arrival is finite
    // Every lane does both, the one that is not meant for it without effect: no
    // slot holds all ones, and every slot is less.
    const uint32_t meant = insert ? (uint32_t)INF : ~0u;
    const unsigned long long wi = atomicCAS(kv + pos, ((unsigned long long)meant << 32) | NO_KEY, want);
    const unsigned long long wm = atomicMin(kv + pos, insert ? ~0ull : want);
    old = insert ? 0u : (uint32_t)wm;
    int32_t before = insert ? INF : (int32_t)(wm >> 32);
    fresh = insert;
    // a swap that lost a race for its slot: lower v's slot if it went there, else
    // probe on to it or to the next empty slot
    const bool lost = insert && wi != EMPTY_SLOT;
    if (__builtin_expect(__ballot(lost) != 0ull, 0)) {
      if (lost) {
        before = 0;
        fresh = false;
        uint32_t p = (uint32_t)pos, key = (uint32_t)wi;
        for (uint32_t n = 0;; ++n) {
          if (n > mask) {
            atomicOr(full, kTableFull);
            break;
          }
          if (key == NO_KEY) {
            const unsigned long long c = atomicCAS(kv + p, EMPTY_SLOT, want);
            if (c == EMPTY_SLOT) {
              item = (int32_t)p;
              fresh = true;
              before = INF;
              break;
            }
            key = (uint32_t)c;
          }
          if ((key & STOP_MASK) == (uint32_t)v) {
            const unsigned long long m = atomicMin(kv + p, want);
            item = (int32_t)p;
            old = (uint32_t)m;
            before = (int32_t)(m >> 32);
            break;
          }
          p = (p + 1u) & mask;
          key = (uint32_t)entry((int32_t)p);
        }
      }
    }
    return before;
  }
};

// The number of set bits of m below this lane.
__device__ __forceinline__ int32_t rank_below(uint64_t m) {
  return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// What a round pushes.  Near list entry: {first type, type count, number of the
// first type, slot}.  Far list entry: {slot | type count << 16, first type}
// (slots are below 2^16; a stop with more types is always pushed near).
struct TablePush {
  TagTable S;
  int4 *near;
  int2 *far;
  unsigned long long *wstart;
  uint16_t *wentry;
  RoundCtr *rc;
  int32_t fcap, farcap, far0;  // far0: entries the far list held when the round began
  uint32_t flag;               // the near flag of the next round

  // Entry `slot` of the near list, whose types are numbered from toff on.  What
  // lies past the list or the windows goes to the spare entry or word at their
  // end: a lane condition costs 25 cycles, a minimum 4.
  __device__ __forceinline__ void list_near(int32_t slot, int32_t toff, int32_t item, int32_t beg, int32_t cnt) {
    near[min(slot, fcap)] = make_int4(beg, cnt, toff, item);
    // bit i of wstart[w + 1]: an entry's types start at type 64 w + i + 1
    // (a lane counts the bits below it); word 0 takes what starts at type 0
    const int32_t q = toff - 1, w = (q >> 6) + 1;
    atomicOr(&wstart[min(w, kTabWin + 1)], 1ull << (q & 63));
    // the windows whose first type is one of this entry's
    wentry[(w << 6) < toff + cnt ? min(w, kTabWin) : kTabWin] = (uint16_t)slot;
  }
  __device__ __forceinline__ void list_more(int32_t slot, int32_t toff, int32_t cnt) {
    for (int32_t b = ((toff - 1) >> 6) + 2; b < kTabWin && (b << 6) < toff + cnt; ++b) wentry[b] = (uint16_t)slot;
  }
  // The far list is full: the stop is expanded in the next round already.
  __device__ __forceinline__ void spill(int32_t item, int32_t beg, int32_t cnt, int32_t val) {
    atomicAnd(S.lo(item), ~FAR_FLAG);
    if (atomicOr(S.lo(item), flag) & flag) return;
    const unsigned long long b = atomicAdd(&rc->near.cx, 1ull | ((unsigned long long)(uint32_t)cnt << 32));
    atomicMin(&rc->near.min, val);
    list_near((int32_t)(uint32_t)b, (int32_t)(uint32_t)(b >> 32), item, beg, cnt);
    list_more((int32_t)(uint32_t)b, (int32_t)(uint32_t)(b >> 32), cnt);
  }
  // Lists a stop (cnt > 0 types).
  __device__ __forceinline__ void operator()(bool isfar, int32_t item, int32_t beg, int32_t cnt, int32_t val) {
    PushCtr *const t = isfar ? &rc->far : &rc->near;
    const unsigned long long b = atomicAdd(&t->cx, 1ull | ((unsigned long long)(uint32_t)(isfar ? 0 : cnt) << 32));
    // both lists' writes for every lane, the other list's to its spare entry
    const int32_t slot = (int32_t)(uint32_t)b, toff = (int32_t)(uint32_t)(b >> 32);
    const int32_t place = isfar ? far0 + slot : farcap;
    list_near(isfar ? fcap : slot, isfar ? kTabWin * 64 + 1 : toff, item, beg, cnt);
    far[min(place, farcap)] = make_int2(item | (cnt << 16), beg);
    const bool rare = isfar ? place >= farcap : cnt > 64;
    if (__builtin_expect(__ballot(rare) != 0ull, 0)) {
      if (rare) {
        if (isfar) spill(item, beg, cnt, val);
        else list_more(slot, toff, cnt);
      }
    }
  }
};

// Waits until at most n vector memory operations of the wave are in flight.  The
// compiler counts with it: past wait_vector_memory(0) it knows of no pending
// read and does not put waits of its own into the round's other steps, which
// would also wait for the stores of the slab's fill.
template <int n>
__device__ __forceinline__ void wait_vector_memory() {
  static_assert(n < 16, "low bits of the counter");
  __builtin_amdgcn_s_waitcnt(0x0f70 | n);
}

// A connection type on its way: its record r (and r2, grid form excepted), the
// grid entry e of its tail stop's arrival x.  No type, or no departure at or
// after x: x = INF, from which nothing improves.
struct TypeRead {
  int4 r, r2, e;
  int32_t x;
};

// Issues the reads of the d-th type of a stop with types [b, b + n), reached at
// x.  in = false: no type (d = 0 then, so that the reads stay in the arrays).
template <int KIND>
__device__ __forceinline__ void issue_record(const GraphG &G, int32_t b, int32_t d, TypeRead &t) {
  if constexpr (KIND == kKindGrid) {
    t.r = G.side[(uint32_t)(b + d)];  // {v, lam, first type of v, type count of v}; fewer than 2^31 types
  } else {
    const int64_t j = (int64_t)b + d;
    t.r = G.ty[2 * j];
    t.r2 = G.ty[2 * j + 1];
  }
}
template <int KIND>
__device__ __forceinline__ void issue_entry(const GraphG &G, int32_t b, int32_t n, int32_t d, int32_t x, bool in,
                                            TypeRead &t) {
  t.x = in ? x : INF;
  if constexpr (KIND == kKindGrid) {
    t.x = x < G.horizon ? t.x : INF;
    // x < horizon <= 64 * 32767 < 2^21: x + 0.5 is exact in float and (x + 0.5) /
    // width is 2^-22 of itself or more away from every integer, more than the two
    // roundings of the product move it, so its integer part is the cluster of x
    const int32_t xc = min(x, G.horizon - 1);
    const uint32_t k = (uint32_t)(((float)xc + 0.5f) * G.inv_cw);
    // unconditional, so that the record and the entry are the two reads in
    // flight and the record can be waited for alone
    t.e = G.grid[(uint32_t)b * (uint32_t)G.n_clusters + k * (uint32_t)n + (uint32_t)d];
  }
}

// Relaxes the type whose reads have been issued.
template <int KIND, bool GOAL>
__device__ __forceinline__ void table_relax(const GraphG &G, const TagTable &S, const TypeRead &t, int32_t thr,
                                            int32_t bound, int32_t target, TablePush &P, Ctr &c) {
  const int32_t x = t.x;
  Look L;
  if constexpr (KIND == kKindGrid) {
    L.mode = 2;
    L.e = t.e;
    wait_vector_memory<1>();
  } else {
    look_locate<KIND>(G, t.r, KIND == EAT_LAYOUT_HYBRID ? (uint32_t)t.r2.z : 0u, x, L);
    look_fetch_headers<KIND>(G, t.r, L);
  }
  const int32_t v = t.r.x, lam = t.r.y;
  int32_t pos = 0;
  const int32_t av = S.find(v, pos, &P.rc->near.extra);
  wait_vector_memory<0>();
  c.tev += x != INF ? 1u : 0u;
  // any departure leaves at t_c >= x, so it arrives at >= x + lam: skip the
  // type when that cannot beat arr[v] (early termination, Section III-D)
  if (x >= av - lam) return;
  if constexpr (KIND != kKindGrid) {
    if (L.mode == 0) return;
  }
  count_fetch<KIND>(t.r, L, c);
  int32_t tc;
  if constexpr (KIND == kKindGrid) {
    // look_finish of a grid entry: the progression (also every empty cluster) is
    // worked out for all lanes, an array only where there is one
    const int32_t d = t.e.y & 0xffff, n = t.e.y >> 16;
    const uint32_t r = (uint32_t)(x - t.e.x - 1), hi = __umulhi(r, (uint32_t)t.e.w);
    const int32_t i = (int32_t)(t.e.w ? hi : r) + 1;
    tc = i < n ? t.e.x + i * d : t.e.z;
    tc = x <= t.e.x ? t.e.x : tc;
    const bool array = t.e.y < 0 && x > t.e.x;
    if (__ballot(array)) {
      if (array) {
        if (__builtin_expect(__ballot(grid_pool_array(t.e.y)) != 0ull, 0)) {  // more than five departures
          look_fetch_chunks<KIND>(G, x, L, c);
          wait_vector_memory<0>();
        }
        tc = look_finish<KIND>(G, t.r, x, L, c);
      }
    }
  } else {
    look_fetch_chunks<KIND>(G, x, L, c);
    wait_vector_memory<0>();
    tc = look_finish<KIND>(G, t.r, x, L, c);
  }
  // INF + lam is past every arrival as an unsigned number
  int32_t cand = (int32_t)((uint32_t)tc + (uint32_t)lam);
  if constexpr (GOAL) cand = cand < min(bound, lds_ld((const int32_t *)&P.rc->far.extra)) ? cand : -1;
  if ((uint32_t)cand >= (uint32_t)av) return;
  int32_t beg, cnt;
  if constexpr (KIND == kKindGrid) {
    beg = t.r.z;
    cnt = t.r.w;
  } else {
    beg = t.r2.x;
    cnt = t.r2.y;
  }
  const bool isfar = cand >= thr && cnt <= 0xffff;
  const uint32_t flag = isfar ? FAR_FLAG : P.flag;
  uint32_t old = 0;
  int32_t item = 0;
  bool fresh = false;
  const int32_t before = S.lower(v, pos, av, cand, flag, item, old, fresh, &P.rc->near.extra);
  if (cand >= before) return;
  c.imp++;
  atomicAdd(&P.rc->near.extra, fresh ? 1u : 0u);
  if constexpr (GOAL) {
    if (v == target) {  // the target is not expanded
      atomicMin((int32_t *)&P.rc->far.extra, cand);
      return;
    }
  }
  // also for a stop that is listed already: its arrival is earlier now
  atomicMin(isfar ? &P.rc->far.min : &P.rc->near.min, cand);
  if (((old & flag) | (cnt > 0 ? 0u : 1u)) == 0u) P(isfar, item, beg, cnt, cand);
}

// Rounds until no arrival improves.  On entry (thread 0's writes, no barrier
// since): the source's slot is in S with NEAR_A set; near0[0] is its entry;
// rc[2] counts it and holds its arrival, rc[0] is reset; the source's windows
// are marked in half 0.  reached = stops in the table.  Returns false if the table
// overflowed or the limit of rounds was hit: the query then runs again in the
// result slab.  (A stop that comes inside the window waits a round more here than
// in run_rounds, so only that one tells whether a limit is enough: of 96 queries of
// city-50k 65 took more rounds here than there, 30.3 on average against 29.5.)
template <int KIND, int B, bool GOAL>
__device__ __forceinline__ bool table_rounds(const RunArgs &a, const GraphG &G, const TagTable &S, int32_t H,
                                             int4 *near0, int4 *near1, int2 *far0, int2 *far1, int32_t far_entries,
                                             bool topo, int32_t max_rounds, int32_t bound, int32_t target, Shared &sh,
                                             QState &qs, int32_t &reached, Ctr &c) {
  constexpr int kWaves = B / 64;
  const int lane = __lane_id();
  const int32_t wave = uniform((int32_t)(threadIdx.x >> 6));
  // a round's list that is longer is a sweep; the lists' last entries are spare
  const int32_t fcap = topo ? 0 : a.fcap - 1, farcap = far_entries - 1;
  const int32_t window = a.table_window;
  const uint32_t limit = (uint32_t)(H - H / 4);
  uint32_t total = 1;  // stops in the table
  int32_t rounds = 0, nf = 0, fmin = INF;
  int32_t n = 0, types = 0, nw = 0;      // of the round's list: entries, types, windows
  int32_t thr = INF, sweep_thr = INF;    // arrivals from here on: to the far list; left by a topology sweep
  bool scan = false;  // the far list holds arrivals inside the window
  bool ended = false;
  int32_t maxf = 1;

  // The round's halves and counters: list and marks by rounds & 1, counters
  // (of the last round, of this one, of the next one) by three in turn.
  int32_t half = 0;
  RoundCtr *r0 = &sh.rc[2], *r1 = &sh.rc[0], *r2 = &sh.rc[1];
  auto near_of = [&](int32_t h) { return h ? near1 : near0; };
  auto marks_of = [&](int32_t h) { return sh.wstart + (h ? kTabWin + 2 : 0); };
  auto holders_of = [&](int32_t h) { return sh.wentry + (h ? kTabWin + 1 : 0); };
  auto flag_of = [&](int32_t h) { return h ? NEAR_B : NEAR_A; };
  auto pushes = [&]() {
    return TablePush{S,  near_of(half ^ 1), scan ? far1 : far0, marks_of(half ^ 1), holders_of(half ^ 1),
                     r1, fcap,              farcap,             scan ? 0 : nf,      flag_of(half ^ 1)};
  };
  // What the last round did (its counters, read as two 16-byte words), and what
  // this one is; false: the query is over.
  int4 last_near, last_far;
  auto read_last = [&]() {
    last_near = *reinterpret_cast<const int4 *>(&r0->near);
    last_far = *reinterpret_cast<const int4 *>(&r0->far);
    // whole words, one wait: not the single fields where they are used
    asm volatile("" : "+v"(last_near.x), "+v"(last_near.y), "+v"(last_near.z), "+v"(last_near.w));
    asm volatile("" : "+v"(last_far.x), "+v"(last_far.y), "+v"(last_far.z), "+v"(last_far.w));
  };
  // (In vector registers: a value that every lane computes alike costs one
  // instruction there, and two or three with scalar conditions.)
  auto decide = [&]() -> bool {
    nf = min(nf + last_far.x, farcap);
    fmin = min(fmin, last_far.z);
    if constexpr (GOAL) bound = min(bound, last_far.w);
    total += (uint32_t)last_near.w;
    const int32_t base = n > 0 ? last_near.z : fmin;
    const bool full = total > limit;  // or a stop found no slot: kTableFull is past any number of slots
    bool over = full || (n | nf) == 0;
    // nothing listed can lead to an earlier arrival at the target
    if constexpr (GOAL) over = over || min(base, nf > 0 ? fmin : INF) >= bound;
    maxf = max(maxf, n + nf);
    thr = window > 0 ? min(base, INF - window) + window : INF;
    const int32_t what = uniform((over ? 1 : 0) | (nf > 0 && fmin < thr ? 2 : 0));
    scan = (what & 2) != 0;
    if (topo) {
      sweep_thr = thr;
      thr = INF;
    }
    ++rounds;
    ended = (what & 1) != 0;
    return !ended && rounds <= max_rounds;
  };
  // The end of a round: the next round's counters are reset, the far list's
  // entries that have come inside the window move to the near list (the others
  // to the far list's other buffer), and the roles change.
  auto finish = [&]() {
    if (wave == kWaves - 1) *r2 = RoundCtr{{0ull, INF, 0u}, {0ull, INF, (uint32_t)INF}};
    if (scan) {
      TablePush P = pushes();
      for (int32_t i = (kWaves - 1 - wave) * 64 + lane; i < nf; i += B) {
        const int2 f = far0[i];
        const int32_t item = f.x & 0xffff;
        const unsigned long long e = S.entry(item);
        const int32_t x = (int32_t)(e >> 32);
        if (!((uint32_t)e & FAR_FLAG)) continue;  // pushed near meanwhile
        const bool prom = x < thr && (!GOAL || x < bound);
        if (prom) {
          atomicAnd(S.lo(item), ~FAR_FLAG);
          if (atomicOr(S.lo(item), P.flag) & P.flag) continue;
        }
        atomicMin(prom ? &P.rc->near.min : &P.rc->far.min, x);
        P(!prom, item, f.y, (int32_t)((uint32_t)f.x >> 16), x);
      }
      nf = 0;
      fmin = INF;
      int2 *f = far0;
      far0 = far1;
      far1 = f;
    }
    half ^= 1;
    RoundCtr *const r = r0;
    r0 = r1;
    r1 = r2;
    r2 = r;
    __syncthreads();  // all pushes of the round are in
  };

  bool go = true;
  __syncthreads();
  while (go) {
    // ---- rounds whose types the windows hold (nearly all) ------------------------
    // (One exit, and no read in flight on any way to it: the compiler then puts
    // no wait of its own before a round's first reads.)
    bool hot;
    do {
      // the marks of the wave's first window come with the counters
      const int4 *const cur = near_of(half);
      unsigned long long *const ws = marks_of(half) + 1;
      const uint16_t *const we = holders_of(half);
      const uint32_t keep_flags = ~flag_of(half);
      int32_t w = wave;
      unsigned long long starts;
      int32_t first;
      auto read_marks = [&]() {
        starts = __hip_atomic_load(ws + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        first = __hip_atomic_load(we + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      };
      read_marks();
      read_last();
      n = uniform(last_near.x);
      types = uniform(last_near.y);
      nw = (types + 63) >> 6;
      hot = n <= fcap && nw <= kTabWin;
      TypeRead t;
      // Lane i of window w relaxes type k = 64 w + i, of the entry that holds it:
      // we[w] plus the entries starting in (64 w, k].
      auto issue = [&]() {
        const int32_t k = (w << 6) + lane;
        const bool in = k < types;
        const int4 e = cur[first + rank_below(starts)];  // past the last type: the last entry
        ws[w] = 0ull;  // read by every lane: clear for the round after next
        const int32_t d = in ? k - e.z : 0;  // the type's place in its stop's range
        issue_record<KIND>(G, e.x, d, t);
        const int32_t x = S.value(e.w);
        if (k == e.z) {
          atomicAnd(S.lo(e.w), keep_flags);
          c.act++;
        }
        issue_entry<KIND>(G, e.x, e.y, d, x, GOAL ? in && x < bound : in, t);
      };
      if (hot) {
        if (w < nw) {
          // before the waves that scan, fill or end a round (1,000 goal-directed
          // queries, two on a CU: 284 -> 278 us; one on a CU: 173 -> 170)
          __builtin_amdgcn_s_setprio(2);
          do {
            if (w != wave) read_marks();
            issue();
            if (w == wave) go = decide();
            // the query's end included: the reads are waited for on every path, so
            // that none of them is in flight where the next window's are issued
            t.x = go ? t.x : INF;
            TablePush P = pushes();
            table_relax<KIND, GOAL>(G, S, t, thr, bound, target, P, c);
            w += kWaves;
          } while (go && w < nw);
          __builtin_amdgcn_s_setprio(0);
        } else {
          go = decide();
        }
        if (go) {
          // a wave with fewer windows than wave 0 issues part of the slab's fill meanwhile
          // (w - wave: the types of its windows' rows; two steps' worth at most)
          const int32_t left = nw - (w - wave);
          if (left > 0) fill_issue(sh, left > kWaves ? 2 * kFillPerStep : kFillPerStep);
          finish();
        }
      }
    } while (hot && go);
    if (!go) break;
    // ---- a sweep over the slots, or a list of more types than the windows hold.
    // A sweep lists the stops its flag marks, as many as the list takes at a time
    // (a stop past the list keeps its flag for the next pass); a list's types are
    // relaxed kTabWin windows at a time, with marks made from its entries.  So the
    // waves share the types evenly here too.  (A wave that took four listed stops,
    // or the marked ones of 64 slots, relaxed their types alone: a query through
    // stops of 750 and 30,000 types took 391 ms, now 42; 256 queries on a flat
    // city-50k in topology mode 1,038 us, now 472; with lists of 64 entries on its
    // grid 613 us, now 533.)
    const bool sweep = n > fcap;
    go = decide();
    if (!go) break;
    qs.sweeps += sweep ? 1 : 0;
    TablePush P = pushes();
    int4 *const list = near_of(half);
    unsigned long long *const ws = marks_of(half) + 1;
    uint16_t *const we = holders_of(half);
    const uint32_t flag = flag_of(half);
    const int32_t cap = a.fcap - 1;
    for (int32_t i = (int32_t)threadIdx.x; i < kTabWin; i += B) ws[i] = 0ull;  // the pushes' marks
    int32_t m = n;     // the list's entries, of all that there are
    bool more = false;
    do {
      if (sweep) {
        if (threadIdx.x == 0) sh.cx[0] = 0ull;
        __syncthreads();
        for (int32_t i0 = wave * 64; i0 < H; i0 += B) {
          const int32_t item = i0 + lane;
          const unsigned long long e = S.entry(item);
          const uint32_t key = (uint32_t)e;
          if (key == NO_KEY || !(key & flag)) continue;
          const int32_t x = (int32_t)(e >> 32);
          if (x >= sweep_thr) {  // left for the next round
            atomicAnd(S.lo(item), ~flag);
            if (!(atomicOr(S.lo(item), P.flag) & P.flag)) {
              atomicAdd(&r1->near.cx, 1ull);
              atomicMin(&r1->near.min, x);
            }
            continue;
          }
          const int2 rg = G.vt[key & STOP_MASK];
          if (rg.y == 0) {  // flagged when it improved, but never listed: entries start at types of their own
            atomicAnd(S.lo(item), ~flag);
            continue;
          }
          const unsigned long long at = atomicAdd(&sh.cx[0], 1ull | ((unsigned long long)(uint32_t)rg.y << 32));
          if ((int32_t)(uint32_t)at < cap) list[(uint32_t)at] = make_int4(rg.x, rg.y, (int32_t)(at >> 32), item);
        }
        __syncthreads();
        m = uniform((int32_t)(uint32_t)sh.cx[0]);
        more = m > cap;
        m = min(m, cap);
      }
      // one atomic books a place and the types' numbers: entries are in their order
      const int32_t listed = m > 0 ? uniform(list[m - 1].z + list[m - 1].y) : 0, upto = (listed + 63) >> 6;
      for (int32_t w0 = 0; w0 < upto; w0 += kTabWin) {
        __syncthreads();  // the marks of the windows before are read
        for (int32_t i = (int32_t)threadIdx.x; i < m; i += B) {
          const int4 e = list[i];
          const int32_t q = e.z - 1, w = (q >> 6) - w0;
          if (w >= 0 && w < kTabWin) atomicOr(&ws[w], 1ull << (q & 63));
          for (int32_t b = max(w + 1, 0); b < kTabWin && ((w0 + b) << 6) < e.z + e.y; ++b) we[b] = (uint16_t)i;
        }
        __syncthreads();
        for (int32_t w = wave; w < min(upto - w0, kTabWin); w += kWaves) {
          const unsigned long long starts = ws[w];
          const int32_t k = ((w0 + w) << 6) + lane;
          const bool in = k < listed;
          const int4 e = list[we[w] + rank_below(starts)];
          ws[w] = 0ull;
          const int32_t d = in ? k - e.z : 0;
          TypeRead t;
          issue_record<KIND>(G, e.x, d, t);
          const int32_t x = S.value(e.w);
          if (k == e.z) {
            atomicAnd(S.lo(e.w), ~flag);
            c.act++;
          }
          issue_entry<KIND>(G, e.x, e.y, d, x, GOAL ? in && x < bound : in, t);
          table_relax<KIND, GOAL>(G, S, t, thr, bound, target, P, c);
        }
      }
      if (more) __syncthreads();  // before the next pass's list
    } while (more);
    finish();
  }
  reached = (int32_t)total;
  if (!ended) return false;  // the limit of rounds
  qs.rounds += rounds - 1;   // the last decision began no round
  qs.maxf = max(qs.maxf, maxf);
  return uniform(total > limit ? 1 : 0) == 0;
}
