// Bounded per-target queues (FIFO, SORTED), closed loop: many time steps in ONE launch over the whole chip, one grid
// barrier per step.  Included by adseq.hip after ring_resident_forward.h, whose layout, barrier (rev_wait / rev_arrive) and
// synchronising wavefront it shares.
//
// Two launches per step (k_neurons, k_fanout_step) are bound by the launches and by the state they read again every time:
// 16 x 1,000 neurons with FIFO[32] 11.6 us per step by those, 4.4 here; 100,000 neurons 18.9 and 14.1; 256 x 4,096 neurons with
// sorted[128] 25.9 and 11.0.  Here a block owns the targets [rank * chunk, + chunk) for the whole launch; membrane and synaptic state and row
// bounds stay in registers, the queues' occupancy, front, first mask word and earliest stored arrival in LDS (the slots
// themselves in global memory, private to the block: they are touched only when something is due or admitted).  A step is
//   before the barrier   what is due at step n leaves the queues (its own state alone decides that), drive bits
//   behind it            contenders of step n - 1 (every block has registered its own): admission, update, spikes
//   then                 the rows of the block's spikes, cut into pieces of 64 entries that the wavefronts share out:
//                        tickets, contender records; then the arrival
// so that the fan-out of a step needs no barrier of its own: contenders are registered in two buffers in turn, the one
// being filled while the other one's are admitted.  For the same reason whether a target is full after its pop of step n is not
// known to the others in step n.  What is known a step ahead is that a full queue with nothing due at step n stays full: the
// owners leave that as one bit per target, every block takes all the bits into LDS behind the barrier (one target per
// thread: 16 KB at most), and events for such targets are dropped at once (100,000 neurons, FIFO[32], seven events in ten:
// 18.4 -> 16 us per step).  With several targets per thread there are too many bits for that, and looking them up in memory cost
// more (11.0 -> 12.2 us per step where no queue is full) than the tickets it saves below some 400,000 events per step at full queues; beyond
// that two launches per step are the faster ones (256,000 targets, 2 million events per step, 993 in 1,000 dropped: 332 against 122 us).
// All others are contenders, and the admission -- same rule, same canonical order -- drops what is left to drop;
// the overflow list has room for every synapse (that is what decides whether this kernel runs).  Admission flags are
// written once, by whoever decides.  The tape's places are claimed block by block, spikes
// and events in one 64-bit counter per step, so that their orders agree and the spikes of a 64-neuron word stay
// together and ascending, which k_tape_words relies on.  What a step is bound by now is the chain of a block with spikes: row
// entries, tickets, records, their acknowledgement, the barrier's two trips, count and records of the contenders: 5 us
// of waiting for memory, and where the queues are full (100,000 neurons) the instructions of pops and admissions.
//
// What crosses blocks -- tickets, contender records, overflow entries, the claim counters -- goes through atomics and
// agent-scope accesses.  Waits are bounded as in the ring's resident kernels (ERR_BARRIER).  After a wait that ran out --
// in whichever block -- blocks no longer run in step and may read records and list links that have not been
// written: so whatever is read of other blocks is checked against its range before it is used as an index, and every walk of a
// list is bounded by its count (k_queue_settle clears what such a run leaves behind).

constexpr int kQueueItems = 1024;   // row pieces of a step that are shared out at once
// A piece of a spike's row: its first entry, its entries, first state index of the trial; first admission flag and end of
// the row's flags, counted from the block's first event of the step.
struct QItem { long long p; int cnt, base, ev, evend; };

// TRIAL: per step of the launch, trial and 64 of its neurons, the spikes and where the first one's admission flags begin.
struct QTrial { unsigned long long* bits; long long* evb; int words; };
constexpr int kTrialQueueSteps = 256;   // steps of a launch

// Phase clocks (builds with ADSEQ_PHASE_CLOCK only): ticks of 10 ns that thread 0 of the first block spent in each phase of
// a step, in Counters::phase: [0] pops, [1] waiting, [2] admission, [3] update, [4] pieces written, [5] tickets and records,
// [6] until the arrival, [7] tape.
#ifdef ADSEQ_PHASE_CLOCK
#define QPH_BEGIN unsigned long long qpc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, qpt = wall_clock64();
#define QPH(i) { const unsigned long long t_ = wall_clock64(); qpc[i] += t_ - qpt; qpt = t_; }
#define QPH_END if (rank == 0 && tid == 0) for (int i = 0; i < 8; ++i) d.ctr->phase[i] += qpc[i];
#else
#define QPH_BEGIN
#define QPH(i) {}
#define QPH_END
#endif

// LS: the slots of FIFO targets are in LDS too, for up to 32 of them and one target per thread.
// LC (TRIAL): contender counts are in LDS too, so that a ticket is no trip to memory; 2: in the place of the synaptic current states (delta
// synapse, eight targets per thread).
template <int NPT, bool LS, int LC>
struct QueueLds {
  static constexpr int kTargets = NPT * kResThreads;
  int acc[kTargets];            // Q8.24 sum delivered in the step; from its spike to the step's end, a spiking neuron's membrane value
  unsigned mw[kTargets];        // FIFO: first mask word; SORTED: index of the front
  unsigned mn[kTargets];        // earliest stored arrival step (0xffffffff: none)
  int occ[kTargets];            // stored events | events popped in the step << 16; from its spike to the step's end, a spike's number in the block << 16
  float J[LC == 2 ? 1 : kTargets], Jf[LC == 2 ? 1 : kTargets];   // synaptic current states
  int cnt[LC ? 2 : 1][LC ? kTargets : 1];   // contenders, by buffer
  unsigned long long full[NPT == 1 ? 2048 : 1];   // the whole network's targets that stay full in this step (at most 256 x 512); TRIAL: the trial's, by step parity [2][8]
  int pool_n[2];                // TRIAL: entries taken of the block's shares of the overflow list, by buffer
  int2 list[kTargets];          // targets to work off: place, contenders; then by a spiking neuron's place: its first piece, its first event
  QItem item[kQueueItems];
  alignas(16) unsigned short key[LS ? kTargets : 1][32];
  int amp[LS ? kTargets : 1][32];
  int dead, n_list[2], items;
  unsigned long long claim;     // the block's spikes of the step << 40 | their events
  unsigned long long got;       // what the step's counter held when the block claimed its places
  long long sp_base, ev_base;   // spikes and events on the tape before the step
};

__device__ __forceinline__ uint4 cont_load(const Dev& d, const QBuf& qb, int x, int g) {
  const res_v4i v = __builtin_bit_cast(res_v4i, __builtin_amdgcn_raw_buffer_load_b128(res_rows(qb.cont, kCont * d.BN * 16), (x * d.BN + g) * 16, 0, kBufAgent));
  return make_uint4((unsigned)v[0], (unsigned)v[1], (unsigned)v[2], (unsigned)v[3]);
}
__device__ __forceinline__ void cont_store(const Dev& d, const QBuf& qb, int x, int g, const uint4& c) {
  const res_v4i v = {(int)c.x, (int)c.y, (int)c.z, (int)c.w};
  __builtin_amdgcn_raw_buffer_store_b128(v, res_rows(qb.cont, kCont * d.BN * 16), (x * d.BN + g) * 16, 0, kBufAgent);
}

template <int KIND, int NPT, bool LS, int LC>
__device__ __forceinline__ QState qstate_of(const QueueLds<NPT, LS, LC>& L, int t) {
  QState q;
  q.occ = L.occ[t] & 0xffff; q.mn = L.mn[t]; q.m0 = L.mw[t]; q.hd = (int)L.mw[t];
  return q;
}
// The events of target g (place t) that are due at step kn leave its queue.
template <int KIND, int NPT, bool LS, int LC>
__device__ __forceinline__ void pop_target(const Dev& d, QueueLds<NPT, LS, LC>& L, int t, int g, unsigned kn, StepAcc& r, long long& s_del) {
  QState q = qstate_of<KIND>(L, t);
  const int before = q.occ;
  r.acc = 0;
  if (LS) fifo_scan<true>(d, g, L.key[t], L.amp[t], kn, q, r);
  else if (KIND == ADSEQ_FIFO) fifo_scan<true>(d, g, kn, q, r);
  else sorted_pop(d, g, kn, q, r);
  L.occ[t] = q.occ | ((before - q.occ) << 16);
  L.mn[t] = q.mn; L.mw[t] = KIND == ADSEQ_FIFO ? q.m0 : (unsigned)q.hd;
  L.acc[t] = r.acc;
  s_del += r.acc;
}
// Admission of the K contenders of target g (place t): rule and order as in admit_contenders.  c0, c1: their first two
// records (the others are requested here, together).  deliver: an event that is due at step kn is delivered at once (false:
// the launch ends, everything is stored).  The winners are a bit mask over the record slots, so that there is one copy of the
// insertion and not one per slot: unrolled as in k_neurons this kernel spilled a hundred registers.  More contenders than
// record slots: if there is room for all, the records and the overflow list are walked once; if not, the smallest synapse index is
// selected as often as there is room.  (Selecting in either case, an entry and then the link to the next, took longer than
// two launches per step: 16,000 targets, 25 contenders for each in every step, us per step: SORTED[128] with room for all 1,002 -> 176,
// two launches 262; FIFO[32], one event in six dropped, 693 -> 496, two launches 530; 10 contenders 194 -> 60, two launches 103.)
// buf: the contender buffer's index.
template <int KIND, bool RECORD, int NPT, bool LS, int LC>
__device__ __forceinline__ void admit_target(const Dev& d, QueueLds<NPT, LS, LC>& L, const QBuf& qb, int buf, int t, int g, int K, unsigned kn, bool deliver,
                                             const uint4& c0, const uint4& c1, StepAcc& r, long long& s_del) {
  QState q = qstate_of<KIND>(L, t);
  const int room = d.C - q.occ - (L.occ[t] >> 16);   // what the contenders found when they were emitted
  const int take = K < room ? K : room;
  int acc = 0;
  if (LC) L.cnt[buf][t] = 0; else q_store<true>(&qb.cnt[g], 0);
  auto flag_it = [&](long long f, int won) { if (f >= 0 && f < d.event_cap) d.tape_adm[f] = (unsigned char)won; };
  auto linked = [&](int y) { return y >= 0 && y < d.pool_cap; };
  auto take_in = [&](unsigned k, int a) {
    r.c_adm += 1; r.s_adm += a;
    if (deliver && k == kn) { acc = wrap_add(acc, a); r.popped += 1; return; }
    if (LS) fifo_insert(d, g, L.key[t], L.amp[t], q, k, a);
    else if (KIND == ADSEQ_FIFO) fifo_insert(d, g, q, k, a);
    else sorted_insert(d, g, q, k, a);
    q.mn = k < q.mn ? k : q.mn;
    q.occ += 1;
  };
  if (K <= kCont) {
    uint4 cc[kCont];
    cc[0] = c0; cc[1] = c1;
#pragma unroll
    for (int x = 2; x < kCont; ++x) { cc[x] = make_uint4(0u, 0u, 0u, 0u); if (x < K) cc[x] = cont_load(d, qb, x, g); }
    unsigned won = take ? (1u << K) - 1u : 0u;
    if (take > 0 && take < K) {
      // a contender's rank among them decides (synapse indices below 2^30)
      int rank[kCont];
#pragma unroll
      for (int x = 0; x < kCont; ++x) rank[x] = 0;
#pragma unroll
      for (int x = 1; x < kCont; ++x)
#pragma unroll
        for (int y = 0; y < x; ++y) {
          const bool lt = x >= K || cc[y].x < cc[x].x;
          rank[x] += lt ? 1 : 0; rank[y] += lt ? 0 : 1;
        }
      won = 0u;
#pragma unroll
      for (int x = 0; x < kCont; ++x) won |= x < K && rank[x] < take ? 1u << x : 0u;
    }
#pragma unroll
    for (int x = 0; x < kCont; ++x) if (x < K) flag_it(cont_flag(cc[x]), (int)((won >> x) & 1u));
    for (; won; won &= won - 1u) {
      const int slot = __ffs((int)won) - 1;
      uint4 c = cc[0];
#pragma unroll
      for (int x = 1; x < kCont; ++x) if (slot == x) { c.z = cc[x].z; c.w = cc[x].w; }
      take_in(cont_arrival(c, kn), (int)c.w);
    }
  } else {
    const int head = q_load<true>(&qb.head[g]);   // beyond the record slots: overflow list
    q_store<true>(&qb.head[g], -1);
    const bool all = take == K;   // room for all of them: taken as they stand
    int at = head;
    long long last = -1;
    for (int rnd = 0; rnd <= take; ++rnd) {   // (the last round clears the flags of those that are left)
      const bool clear = rnd == take;
      long long bp = 0x7fffffffffffffffLL, flag = -1;
      unsigned k = 0; int a = 0;
      if (clear && (all || !RECORD)) break;
      if (all && rnd < kCont) {
        const uint4 c = cont_load(d, qb, rnd, g);
        k = cont_arrival(c, kn); a = (int)c.w; flag = cont_flag(c);
      } else if (all) {
        if (!linked(at)) break;
        const int next = q_load<true>(&d.pool_next[at]);
        k = q_load<true>(&d.pool_k[at]); a = q_load<true>(&d.pool_a[at]); flag = q_load<true>(&d.pool_t[at]);
        at = next;
      } else {
        // (requested together where there are registers for it -- four at a time: with all eight the FIFO[32] run of
        // 100,000 neurons took 19.5 ms forward and back where it takes 18.5 --; so are an entry of the list and the link to the next)
        constexpr int kAtOnce = NPT == 1 ? 4 : 1;
#pragma unroll 1
        for (int x0 = 0; x0 < kCont; x0 += kAtOnce) {
          uint4 cc[kAtOnce];
#pragma unroll
          for (int x = 0; x < kAtOnce; ++x) cc[x] = cont_load(d, qb, x0 + x, g);
#pragma unroll
          for (int x = 0; x < kAtOnce; ++x) {
            const long long p = cont_syn(cc[x]);
            if (clear) { if (p > last) flag_it(cont_flag(cc[x]), 0); }
            else if (p > last && p < bp) { bp = p; k = cont_arrival(cc[x], kn); a = (int)cc[x].w; flag = cont_flag(cc[x]); }
          }
        }
        int y = head, best = -1;
        for (int left = K - kCont; left > 0 && linked(y); --left) {
          const int next = q_load<true>(&d.pool_next[y]);
          const long long p = q_load<true>(&d.pool_p[y]);
          if (clear) { if (p > last) flag_it(q_load<true>(&d.pool_t[y]), 0); }
          else if (p > last && p < bp) { bp = p; best = y; }
          y = next;
        }
        if (best >= 0) { k = q_load<true>(&d.pool_k[best]); a = q_load<true>(&d.pool_a[best]); flag = q_load<true>(&d.pool_t[best]); }
        if (clear) break;
        last = bp;
      }
      take_in(k, a);
      flag_it(flag, 1);
    }
  }
  L.occ[t] = q.occ;
  L.mn[t] = q.mn; L.mw[t] = KIND == ADSEQ_FIFO ? q.m0 : (unsigned)q.hd;
  if (acc != 0) L.acc[t] = wrap_add(L.acc[t], acc);
  s_del += acc;
}

// Steps n0 .. n0 + nsteps - 1.  P taking-part blocks (every stride-th block of the grid), each owning `chunk` <= NPT * 512
// targets; thread t of a block owns the places t, t + 512, ... .  bar_base: sum of the arrival counters when the launch
// begins; every block arrives nsteps times.  RECORD: the tape is written (claims: one counter per step, zero).  No
// contender is pending when the launch begins, and none when it ends.
// TRIAL: every block owns one whole trial (rank: the trial, chunk = N), so that no block has anything to do with another one's events: the grid
// barrier goes -- a step then takes as long as a block's own, not as the longest of all blocks', whose spikes cost 5 us each time.  The tape's
// spike list is ordered by step over all trials, which nobody knows any more while the blocks run apart: a block claims places for its
// events' flags as it comes to them (claims[max_steps] counts the launch's; tape_evb says where they are, in whatever order) and leaves its
// spike words and where their events begin for k_trial_list.  The block has shares of its own of the overflow list.  RECORD only.
// 256 x 4,096 neurons, sorted[128]: 11.2 -> 6.7 us per step; queue_trial_plan.h has the sizes.
template <int KIND, bool RECORD, int NPT, bool LS, bool TRIAL, int LC>
__global__ __launch_bounds__(kResLaunch) void k_queue_run(long long n0, int nsteps, unsigned bar_base, int P, int chunk, int stride,
                                                          unsigned long long* __restrict__ claims, QTrial tr, Dev d) {
  static_assert(TRIAL || LC == 0, "counts in LDS: a block's own targets");
  __shared__ QueueLds<NPT, LS, LC> L;
  if (blockIdx.x % stride) return;
  const int rank = blockIdx.x / stride;
  if (rank >= P) return;
  if (threadIdx.x == 0) {
    L.dead = (ld_agent(&d.ctr->err) & ERR_BARRIER) ? 1 : 0;
    L.n_list[0] = 0; L.n_list[1] = 0; L.items = 0; L.claim = 0ull; L.got = 0ull;
    L.pool_n[0] = 0; L.pool_n[1] = 0;
    if (RECORD) { L.sp_base = d.step_off[n0]; L.ev_base = d.step_evoff[n0]; }
  }
  const bool worker = threadIdx.x < kResThreads;   // uniform per wavefront
  if (!worker) {
    // the block barriers of a step, in the workers' order
    __syncthreads();
    for (int k = 0; k <= nsteps; ++k) {
      const bool last = k == nsteps;
      if (!last && NPT > 1) { __syncthreads(); __syncthreads(); }          // step before written up; due targets listed
      if (!TRIAL && k > 0) rev_wait(d, bar_base + (unsigned)k * (unsigned)P, &L.dead); else __syncthreads();
      if (NPT > 1) __syncthreads();                                        // targets with contenders listed
      __syncthreads();                                                     // admitted
      if (last) break;
      __syncthreads();                                                     // spikes known
      const int total = L.items;
      const unsigned long long claim = L.claim;
      for (int b0 = 0; b0 < total || (RECORD && b0 == 0 && claim); b0 += kQueueItems) {
        __syncthreads();                                                   // pieces written
        if (RECORD && b0 == 0) {
          if (threadIdx.x == kResThreads && claim) {
            if (TRIAL) atomicAdd(&claims[n0 + k], claim);   // (what the step comes to, for k_trial_list)
            L.got = atomicAdd(&claims[TRIAL ? d.max_steps : n0 + k], claim);
          }
          __syncthreads();                                                 // places claimed
        }
        if (b0 + kQueueItems < total) __syncthreads();                     // pieces taken
      }
      if (TRIAL) __syncthreads(); else rev_arrive(d, true, rank);
    }
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kWaves = kResThreads / 64;
  const int lo = rank * chunk;
  const int hi = lo + chunk < d.BN ? lo + chunk : d.BN;
  const bool syn = LC != 2 && d.alpha_s > 0.0f, dexp = LC != 2 && d.alpha_r > 0.0f;
  const unsigned long long G64 = 0x9E3779B97F4A7C15ull;
  float V[NPT];
  int r0[NPT], rlen[NPT];   // (2 B S entries fit the overflow pool: B S < 2^30)
  unsigned long long zg[NPT];
  const int voff = (lo + tid) * 4;   // of the thread's first target in a row of 4-byte values; the others 2,048 bytes apart
  constexpr int kRow = kResThreads * 4;
  unsigned actmask = 0;
  StepAcc r; r.acc = 0; r.popped = 0; r.c_adm = 0; r.s_adm = 0;
  long long s_del = 0, c_off = 0, s_off = 0;
#pragma unroll
  for (int c = 0; c < NPT; ++c) {
    const int t = c * kResThreads + tid, g = lo + t;
    V[c] = 0.0f; r0[c] = 0; rlen[c] = 0; zg[c] = 0ull;
    if (LC) { L.cnt[0][t] = 0; L.cnt[1][t] = 0; }
    L.acc[t] = 0;
    if (LC != 2) { L.J[t] = 0.0f; L.Jf[t] = 0.0f; }
    L.mw[t] = 0u; L.mn[t] = 0xffffffffu; L.occ[t] = 0;
    if (g < hi) {
      actmask |= 1u << c;
      const int i = g - trial_of(d, g) * d.N;
      r0[c] = (int)d.row_ptr[i];
      rlen[c] = (int)d.row_ptr[i + 1] - r0[c];
      V[c] = d.V[g];
      if (syn) L.J[t] = d.J[g];
      if (dexp) L.Jf[t] = d.J[(size_t)d.BN + g];
      zg[c] = mix64(d.seed + G64 * ((unsigned long long)g + 1ull));
      QState q;
      q.occ = d.occ[g]; q.hd = 0; q.m0 = 0u; q.mn = 0xffffffffu;
      if (LS) for (int x = 0; x < d.C; ++x) { L.key[t][x] = d.fkey[(size_t)g * d.cpad + x]; L.amp[t][x] = d.famp[(size_t)g * d.C + x]; }
      if (KIND == ADSEQ_FIFO) { q.m0 = d.vmask[(size_t)g * d.nw]; if (q.occ > 0) fifo_scan<false>(d, g, (unsigned)n0, q, r); }
      else { q.hd = d.head[g]; q.mn = d.min_k[g]; }
      L.occ[t] = q.occ; L.mn[t] = q.mn; L.mw[t] = KIND == ADSEQ_FIFO ? q.m0 : (unsigned)q.hd;
    }
  }
  if (NPT == 1) for (int w = tid; w < (TRIAL ? 16 : d.words); w += kResThreads) L.full[w & 2047] = 0ull;
  // appends the lane's target (place t) to the block's list
  auto enlist = [&](int* n, bool want, int t, int K) {
    const unsigned long long m = __ballot(want);
    if (!m) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(n, __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
    if (want) L.list[at] = make_int2(t, K);
  };
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  QPH_BEGIN
  for (int k = 0; k <= nsteps; ++k) {
    const long long n = n0 + k;
    const unsigned kn = (unsigned)n;
    const bool last = k == nsteps;   // (only the contenders of the last step are left: admitted, nothing delivered)
    // ---- in front of the barrier: what is due leaves the queues
    unsigned xi = 0;
    if (!last) {
      if (d.p_thresh) {
#pragma unroll
        for (int c = 0; c < NPT; ++c)
          xi |= (mix64(zg[c] + G64 * ((unsigned long long)n + 1ull)) >> 32) < d.p_thresh ? 1u << c : 0u;
      }
      if (NPT == 1) {
        if ((actmask & 1u) && L.mn[tid] == kn) pop_target<KIND>(d, L, tid, lo + tid, kn, r, s_del);
      } else {
        __syncthreads();   // (the list still says where the last step's spikes are on the tape)
#pragma unroll
        for (int c = 0; c < NPT; ++c) {
          const int t = c * kResThreads + tid;
          enlist(&L.n_list[0], ((actmask >> c) & 1u) && L.mn[t] == kn, t, 0);
        }
        __syncthreads();
        const int due = L.n_list[0];
        for (int x = tid; x < due; x += kResThreads) { const int t = L.list[x].x; pop_target<KIND>(d, L, t, lo + t, kn, r, s_del); }
      }
    }
    QPH(0)
    // ---- every block has registered the contenders of step n - 1
    if (!TRIAL && k > 0) rev_wait(d, bar_base + (unsigned)k * (unsigned)P, &L.dead); else __syncthreads();
    QPH(1)
    QBuf in = queue_buf_half(d, (k & 1) ^ 1), out = queue_buf_half(d, k & 1);
    if (TRIAL) {   // (a trial's synapses fit a share)
      const int share = (int)d.S;
      in.pool0 += rank * share; in.pool_cap = share; in.pool_n = &L.pool_n[(k & 1) ^ 1];
      if (LC) { in.cnt = &L.cnt[(k & 1) ^ 1][0] - lo; out.cnt = &L.cnt[k & 1][0] - lo; }   // (generic pointers, for the way that is hardly ever taken)
      out.pool0 += rank * share; out.pool_cap = share; out.pool_n = &L.pool_n[k & 1];
    }
    unsigned long long before = 0ull;   // what the blocks claimed in step n - 1 (one thread)
    if (RECORD && !TRIAL && k > 0 && tid == kResThreads - 1) before = __hip_atomic_load(&claims[n - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long stay[4];   // targets that stay full in this step, as their owners saw it coming in the last one
    if (NPT == 1) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int w = tid + x * kResThreads;
        stay[x] = 0ull;
        if (!TRIAL && k > 0 && w < d.words) stay[x] = q_load<true>(&d.full_bits[(size_t)((k & 1) ^ 1) * d.words + w]);
      }
      if (k > 0 && (actmask & 1u)) {
        const int g = lo + tid;
        const int K = LC ? L.cnt[(k & 1) ^ 1][tid] : ld_agent(&in.cnt[g]);
        // (the first two records are requested beside the count: most targets that have contenders have no more)
        const uint4 c0 = cont_load(d, in, 0, g), c1 = cont_load(d, in, 1, g);
        if (K > 0) admit_target<KIND, RECORD>(d, L, in, (k & 1) ^ 1, tid, g, K, kn, !last, c0, c1, r, s_del);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) { const int w = tid + x * kResThreads; if (!TRIAL && w < d.words && w < 2048) L.full[w] = stay[x]; }
    } else {
      if (tid == 0) L.n_list[0] = 0;
      int K[NPT];
#pragma unroll
      for (int c = 0; c < NPT; ++c)   // (past the block's last target: zero)
        K[c] = LC ? (k > 0 ? L.cnt[(k & 1) ^ 1][c * kResThreads + tid] : 0) : __builtin_amdgcn_raw_buffer_load_b32(res_rows(in.cnt, k > 0 ? hi * 4 : 0), voff, c * kRow, kBufAgent);
#pragma unroll
      for (int c = 0; c < NPT; ++c) enlist(&L.n_list[1], K[c] > 0, c * kResThreads + tid, K[c]);
      __syncthreads();
      const int offered = L.n_list[1];
      for (int x = tid; x < offered; x += kResThreads) {
        const int t = L.list[x].x, Kt = L.list[x].y, g = lo + t;
        const uint4 c0 = cont_load(d, in, 0, g), c1 = cont_load(d, in, 1, g);
        admit_target<KIND, RECORD>(d, L, in, (k & 1) ^ 1, t, g, Kt, kn, !last, c0, c1, r, s_del);
      }
    }
    if (TRIAL) { if (tid == 0) L.pool_n[(k & 1) ^ 1] = 0; }
    else if (rank == 0 && tid == 0) q_store<true>(in.pool_n, 0);   // (its entries are being consumed; the next ones come a barrier later)
    if (RECORD && !TRIAL && k > 0 && tid == kResThreads - 1) {
      L.sp_base += (long long)(before >> 40); L.ev_base += (long long)(before & ((1ull << 40) - 1ull));
      if (rank == 0) { d.step_off[n] = L.sp_base; d.step_evoff[n] = L.ev_base; }
    }
    __syncthreads();
    if (last) break;
    if (tid == 0) L.n_list[1] = 0;
    QPH(2)
    // ---- drive, membrane, spikes; the pieces of the spikes' rows are numbered
    unsigned smask = 0;
#pragma unroll
    for (int c = 0; c < NPT; ++c) {
      const int t = c * kResThreads + tid;
      const int acc = L.acc[t], o = L.occ[t];
      if (acc != 0) L.acc[t] = 0;
      if (o >> 16) L.occ[t] = o & 0xffff;
      float I = (float)acc * 0x1p-24f;
      if (syn) {   // the jumps go into the synaptic current state(s)
        const float jump = I;
        I = __fmaf_rn(d.alpha_s, L.J[t], jump);
        L.J[t] = I;
        if (dexp) {
          const float fast = __fmaf_rn(d.alpha_r, L.Jf[t], jump);
          L.Jf[t] = fast;
          I = I - fast;
        }
      }
      if (d.p_thresh) I = I + (((xi >> c) & 1u) ? d.ext_w : 0.0f);
      const float U = __fmaf_rn(d.alpha, V[c], I);
      const bool s = ((actmask >> c) & 1u) && U >= d.theta;
      V[c] = s ? d.v_reset : U;
      smask |= s ? 1u << c : 0u;
      if (NPT == 1) {
        const unsigned long long f = __ballot((actmask & 1u) && (o & 0xffff) == d.C && L.mn[t] != kn + 1u);
        if (TRIAL) { if (lane == 0) L.full[(k & 1) * 8 + wave] = f; }
        else if (lane == 0 && lo + tid < hi) q_store<true>(&d.full_bits[(size_t)(k & 1) * d.words + ((lo + tid) >> 6)], f);
      }
      const unsigned long long m = __ballot(s);
      if (TRIAL && lane == 0 && c * 8 + wave < tr.words) tr.bits[((size_t)k * P + rank) * tr.words + c * 8 + wave] = m;
      if (m) {   // uniform
        const int seg = s ? (rlen[c] + 63) >> 6 : 0, len = s ? rlen[c] : 0;
        const int segs = dpp_scan_add(seg), lens = dpp_scan_add(len);
        int at = 0;
        unsigned long long cl = 0ull;
        if (lane == 63) {
          if (segs) at = atomicAdd(&L.items, segs);
          if (RECORD) cl = atomicAdd(&L.claim, ((unsigned long long)__popcll(m) << 40) | (unsigned long long)lens);
        }
        const int first = lane_get(at, 63) + segs - seg;
        const unsigned long long c0 = (unsigned long long)lane_get((long long)cl, 63);
        if (s) {
          L.list[t] = make_int2(first, (int)(c0 & 0x7fffffffull) + lens - len);
          L.occ[t] = (o & 0xffff) | (((int)(c0 >> 40) + __popcll(m & ((1ull << lane) - 1ull))) << 16);
          L.acc[t] = __float_as_int(U);
        }
      }
    }
    __syncthreads();
    QPH(3)
    // ---- fan-out: tickets and contender records
    const int total = L.items;
    const bool any = RECORD && L.claim != 0ull;
    for (int b0 = 0; b0 < total || (b0 == 0 && any); b0 += kQueueItems) {
      if (__ballot(smask != 0u) != 0ull) {
#pragma unroll
        for (int c = 0; c < NPT; ++c) {
          unsigned long long m = __ballot((smask >> c) & 1u);
          if (!m) continue;   // uniform
          const int t = c * kResThreads + tid;
          const int2 at = L.list[t];
          while (m) {   // (the pieces of one spike are written by as many lanes)
            const int src = __ffsll((long long)m) - 1;
            m &= m - 1;
            const int len = lane_get(rlen[c], src), p = lane_get(r0[c], src), first = lane_get(at.x, src) - b0, ev = lane_get(at.y, src);
            const int base = trial_of(d, lo + c * kResThreads + wave * 64 + src) * d.N;
            for (int x = lane, o = 64 * lane; o < len; x += 64, o += 4096)
              if (first + x >= 0 && first + x < kQueueItems) {
                QItem it;
                it.p = (long long)p + o; it.cnt = len - o < 64 ? len - o : 64; it.base = base;
                it.ev = ev + o; it.evend = ev + len;
                L.item[first + x] = it;
              }
          }
        }
      }
      __syncthreads();
      QPH(4)
      const int here = total - b0 < kQueueItems ? total - b0 : kQueueItems;
      bool first = RECORD && b0 == 0;   // (the block's places on the tape are being claimed by the synchronising wavefront)
      for (int x0 = wave; first || x0 < here; x0 += 4 * kWaves) {
        QItem it[4]; unsigned pk[4]; int a[4], tk[4], gt[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          it[u].cnt = 0; it[u].p = 0; it[u].base = 0; it[u].ev = 0; it[u].evend = 0; pk[u] = 0u; a[u] = 0;
          if (x0 + u * kWaves < here) {   // (the same in every lane)
            it[u] = L.item[x0 + u * kWaves];
            if (lane < it[u].cnt) { pk[u] = d.packed[it[u].p + lane]; a[u] = d.a_q[it[u].p + lane]; }
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          tk[u] = -1;
          gt[u] = it[u].base + (int)(pk[u] >> d.dbits);
          bool open = lane < it[u].cnt;
          if (NPT == 1 && open) {
            const int at = TRIAL ? gt[u] - lo : gt[u], w = TRIAL ? ((k & 1) ^ 1) * 8 + (at >> 6) : (at >> 6) & 2047;
            open = !((L.full[w] >> (at & 63)) & 1ull);
          }
          if (open) tk[u] = LC ? atomicAdd(&L.cnt[k & 1][gt[u] - lo], 1) : atomicAdd(&out.cnt[gt[u]], 1);
        }
        if (first) { __syncthreads(); first = false; }
        const long long ev0 = RECORD ? L.ev_base + (long long)(L.got & ((1ull << 40) - 1ull)) : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (it[u].cnt == 0) continue;   // uniform
          const int D = (int)(pk[u] & d.dmask);
          const long long flag = RECORD && ev0 + it[u].evend <= d.event_cap ? ev0 + it[u].ev + lane : -1;
          if (NPT == 1 && RECORD && tk[u] < 0 && lane < it[u].cnt && flag >= 0) d.tape_adm[flag] = 0;   // (dropped: the target stays full)
          if (tk[u] >= 0 && tk[u] < kCont) cont_store(d, out, tk[u], gt[u], cont_pack(it[u].p + lane, flag, (unsigned)(n + D) & 0xffffu, a[u]));
          const bool over = tk[u] >= kCont;   // beyond the record slots: overflow list
          if (__ballot(over)) overflow_push<true>(d, out, over, gt[u], it[u].p + lane, flag, (unsigned)(n + D), a[u]);
        }
      }
      if (b0 + kQueueItems < total) __syncthreads();
    }
    QPH(5)
    if (TRIAL) { __builtin_amdgcn_s_waitcnt(0x0F70); __syncthreads(); } else rev_arrive(d, true, rank);
    QPH(6)
    // ---- after the arrival, off the chain: tape, counts
    if (RECORD) {
#pragma unroll
      for (int c = 0; c < NPT; ++c)
        __builtin_amdgcn_raw_buffer_store_b32((smask >> c) & 1u ? L.acc[c * kResThreads + tid] : __float_as_int(V[c]),
                                              res_rows(d.tapeU + (size_t)n * d.BN, hi * 4), voff, c * kRow, kBufNonTemporal);
    }
    if (__ballot(smask != 0u) != 0ull) {
#pragma unroll
      for (int c = 0; c < NPT; ++c) {
        if (!((smask >> c) & 1u)) continue;
        const int t = c * kResThreads + tid, g = lo + t;
        const int o = L.occ[t];
        L.acc[t] = 0; L.occ[t] = o & 0xffff;
        c_off += rlen[c]; s_off += d.rowsum[g - trial_of(d, g) * d.N];
        if (RECORD) {
          atomicAdd(&d.spk_count[g], 1);
          const long long at = L.sp_base + (long long)(L.got >> 40) + (o >> 16);
          if (TRIAL) {   // where the events of the word's first spike begin; that all find room is looked at with the list
            const unsigned long long m = __ballot((smask >> c) & 1u);
            if (lane == __ffsll((long long)m) - 1)
              tr.evb[((size_t)k * P + rank) * tr.words + c * 8 + wave] = L.ev_base + (long long)(L.got & ((1ull << 40) - 1ull)) + L.list[t].y;
            continue;
          }
          long long evb = L.ev_base + (long long)(L.got & ((1ull << 40) - 1ull)) + L.list[t].y;
          if (evb + rlen[c] > d.event_cap) { evb = -1; atomicOr(&d.ctr->err, ERR_TAPE_EVENTS); }
          if (at < d.spike_cap) {
            d.tape_spk[at] = g; d.tape_evb[at] = evb;
            if (!d.sorted_rev) { RowSpan rs; rs.r0 = r0[c]; rs.r1 = (long long)r0[c] + rlen[c]; d.tape_row[at] = rs; }
          } else atomicOr(&d.ctr->err, ERR_TAPE_SPIKES);
        }
      }
    }
    QPH(7)
    if (tid == 0) L.items = 0;
    if (tid == 64) L.claim = 0ull;
  }
  QPH_END
  // ---- the state goes back to memory, the counters to the block's private lines
#pragma unroll
  for (int c = 0; c < NPT; ++c)
    if ((actmask >> c) & 1u) {
      const int t = c * kResThreads + tid, g = lo + t;
      d.V[g] = V[c];
      if (syn) d.J[g] = L.J[t];
      if (dexp) d.J[(size_t)d.BN + g] = L.Jf[t];
      d.occ[g] = L.occ[t] & 0xffff;
      if (LS) for (int x = 0; x < d.C; ++x) { d.fkey[(size_t)g * d.cpad + x] = L.key[t][x]; d.famp[(size_t)g * d.C + x] = L.amp[t][x]; }
      if (KIND == ADSEQ_FIFO) d.vmask[(size_t)g * d.nw] = L.mw[t];
      else { d.head[g] = (int)L.mw[t]; d.min_k[g] = L.mn[t]; }
    }
  if (RECORD && !TRIAL && rank == 0 && tid == kResThreads - 1) { d.ctr->tape_spikes = L.sp_base; d.ctr->tape_events = L.ev_base; }
  const long long t_pop = wave_total64(r.popped), t_adm = wave_total64(r.c_adm), t_sadm = wave_total64(r.s_adm), t_del = wave_total64(s_del);
  const long long t_off = wave_total64(c_off), t_soff = wave_total64(s_off);
  if (lane == 0) {
    BlkCtr& bc = d.blk[TRIAL ? rank % d.nblk : rank];
    if (t_pop) atomicAdd(&bc.delivered, (unsigned long long)t_pop);
    if (t_adm) { atomicAdd(&bc.admitted, (unsigned long long)t_adm); atomicAdd((unsigned long long*)&bc.sum_admitted, (unsigned long long)t_sadm); }
    if (t_del) atomicAdd((unsigned long long*)&bc.sum_delivered, (unsigned long long)t_del);
    if (t_off) { atomicAdd(&bc.offered, (unsigned long long)t_off); atomicAdd((unsigned long long*)&bc.sum_offered, (unsigned long long)t_soff); }
  }
}

// The spike list of steps n0 .. n0 + gridDim.x - 1, run by k_queue_run<TRIAL> in one launch: a block per step.  Spikes ascend within a step.
__global__ __launch_bounds__(kBlock) void k_trial_list(Dev d, long long n0, QTrial tr) {
  __shared__ long long s_red[2][kBlock / 64];
  __shared__ int s_wave[kBlock / 64];
  const int k = (int)blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long n = n0 + k;
  constexpr unsigned long long kEvents = (1ull << 40) - 1ull;
  // spikes and events of the steps before
  long long sp = 0, ev = 0;
  for (int j = threadIdx.x; j < k; j += kBlock) { const unsigned long long c = d.claims[n0 + j]; sp += (long long)(c >> 40); ev += (long long)(c & kEvents); }
  sp = wave_total64(sp); ev = wave_total64(ev);
  if (lane == 0) { s_red[0][wave] = sp; s_red[1][wave] = ev; }
  __syncthreads();
  sp = d.step_off[n0]; ev = d.step_evoff[n0];
  for (int w = 0; w < kBlock / 64; ++w) { sp += s_red[0][w]; ev += s_red[1][w]; }
  const unsigned long long mine = d.claims[n];
  if (threadIdx.x == 0) {
    d.step_off[n + 1] = sp + (long long)(mine >> 40); d.step_evoff[n + 1] = ev + (long long)(mine & kEvents);
    if (k + 1 == (int)gridDim.x) {
      d.ctr->tape_spikes = sp + (long long)(mine >> 40); d.ctr->tape_events = ev + (long long)(mine & kEvents);
      d.claims[d.max_steps] = 0ull;   // (of the next launch)
    }
  }
  if (mine == 0ull) return;
  const int all = d.B * tr.words;
  const unsigned long long* const bits = tr.bits + (size_t)k * all;
  long long at = sp;
  for (int x0 = 0; x0 < all; x0 += kBlock) {
    const int x = x0 + (int)threadIdx.x;
    unsigned long long m = x < all ? bits[x] : 0ull;
    const int c = __popcll(m), incl = dpp_scan_add(c);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < kBlock / 64; ++w) { if (w < wave) before += s_wave[w]; total += s_wave[w]; }
    __syncthreads();
    if (m) {
      long long p = at + before + incl - c, e = tr.evb[(size_t)k * all + x];
      const int b = x / tr.words, i0 = (x - b * tr.words) * 64;
      for (; m; m &= m - 1ull, ++p) {
        const int i = i0 + __ffsll((long long)m) - 1;
        const long long len = d.row_ptr[i + 1] - d.row_ptr[i];
        const bool fits = e + len <= d.event_cap;
        if (!fits) atomicOr(&d.ctr->err, ERR_TAPE_EVENTS);
        if (p < d.spike_cap) { d.tape_spk[p] = b * d.N + i; d.tape_evb[p] = fits ? e : -1; }
        else atomicOr(&d.ctr->err, ERR_TAPE_SPIKES);
        e += len;
      }
    }
    at += total;
  }
}

// After the launches of a run: nothing, unless one of their waits ran out -- then the contender buffers are emptied, so that
// the launches that follow find what a run leaves behind otherwise (the run stays void).
__global__ __launch_bounds__(kBlock) void k_queue_settle(Dev d) {
  if (!(d.ctr->err & ERR_BARRIER)) return;
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < 2 * (size_t)d.BN; i += (size_t)gridDim.x * kBlock) { d.cnt[i] = 0; d.c_head[i] = -1; }
  if (blockIdx.x == 0 && threadIdx.x < 2) d.ctr->pool_n[threadIdx.x] = 0;
}
