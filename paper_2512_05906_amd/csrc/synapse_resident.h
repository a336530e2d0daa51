// One queue per synapse (SYN_FIFO, SYN_LATEST, SYN_BINS), closed loop with a tape: many time steps in ONE launch over the
// whole chip, and no queue is looked at.  Included by adseq.hip after ring_resident_forward.h, whose barrier
// (rev_wait / rev_arrive) and synchronising wavefront it shares.
//
// By three launches per step (k_synq_pop, k_neurons, k_fanout_step) a step streams the heads of all the queues, whatever is in
// flight: 10,000 neurons x 1,000 synapses 8.2 + 3.6 + 7.7 us per step.  But what a queue holds follows from its source alone:
// every synapse has one delay D, so a queue's events are its source's spikes of the last D steps, less those that were refused
// or replaced -- and that, too, depends on nothing but the source's spikes and D:
//   SYN_FIFO    the spike of step n is refused where the queue holds C events: where C of the source's spikes m with
//               n - m < D were admitted to a queue of delay D.  A source with fewer than C spikes in the last d_max steps is
//               admitted everywhere; for any other spike a bit per D says where (syn_mask, made in the order of the spikes).
//   SYN_LATEST  the event of spike m is replaced by the source's next spike n, where m + D > n;
//   SYN_BINS    by the next spike n with n = m mod C.
// So a block owns `chunk` neurons AS SOURCES AND AS TARGETS, keeps their spikes of the last R steps as words in LDS (replaced
// spikes cleared), and a time step is
//   behind the barrier   cells of the step (all that is due has been added), update, spikes; the spikes' entries that arrive one to
//                        three steps later (the front of the sorted row, kept in LDS) are added to those steps' cells; entries of
//                        replaced spikes that are there already are taken back; arrival
//   behind the arrival   off the chain: tape; the entries of all held spikes that arrive two steps later (D of a spike is known steps
//                        ahead; [dstart[D], dstart[D + 1]) of its sorted row) are added to that step's cells.  Spike words, row
//                        positions and entries are three dependent accesses, each made a step before the next, so that none is
//                        waited for: the list is made for arrivals four steps later, hence the three steps of the front.
// A FIFO of one or two events may refuse an event of delay 2 or 3: there the front is that of one step, and the three accesses
// follow one another (first version, every kind: 5.2 instead of 4.3 us per step of the network below).
// Cells are eight rows of Q8.24 sums, by arrival step mod 8: the one being read, those that are added to, those being cleared.
// Sums are integers, so results do not depend on the order of the adds.
// The queue arrays are not touched.  Another entry point that needs them gets them from the spike words (k_syn_queues).
// Spike list and admission flags are written from the tape's spike words when the launch is over (k_syn_list, k_syn_flags).
// A step is bound by its barrier and by two trips to memory (cells, adds): 1.9 us while nothing spikes; then by the adds of the step's
// events (27 per ns at best).  Measured, SYN_FIFO[4], 10,000 x 1,000 synapses at 20 spikes and 20,000 events per step: 19.4 us per step
// by launches, 4.3 so (1,000 steps forward and back 21.0 -> 7.3 ms); 54 trials x 1,396 x 16, 31 spikes per step 14.5 -> 3.6 us.
// Under load a FIFO is bound by what its sources hold, most of it refused: pieces are looked up one per lane and sifted before their rows
// are (eight lanes per piece and three trips after one another took 2 to 3 times the step below), and a mask is made of set bits, 64 held
// spikes at a time (each bit of each delay by a ballot: five times the step below at d_max 1,000).  SYN_FIFO[1], 4,000 x 100, us per step by
// launches / so at 0.2, 2, 10 and 30 % of the neurons firing: d_max 250 13.7 18.7 34 68 / 3.8 7.0 12.1 26; 512 13.5 18.6 34 70 / 4.9 9.8 19 49;
// 1,000 13.5 18.5 34 71 / 6.3 12.4 27 94, hence kSynFifoDelay.  SYN_LATEST and SYN_BINS, which hold one spike per source or bin, are faster than
// launches at all of these (1.6 to 10 times).
//
// What crosses blocks are the cells (atomic adds, agent-scope loads and clears) and the claim counters.  Waits are bounded as in
// the ring's resident kernels; a run whose waits ran out is void, and reads nothing of other blocks that is used as an index.

constexpr int kSynChunk = 128;         // steps of one launch: FIFO masks are kept for R + kSynChunk steps
constexpr int kSynLdsWords = 16384;    // 8-byte words of LDS for spike words (FIFO: twice) and the rows' fronts
constexpr int kSynFifoDelay = 512;     // SYN_FIFO: largest delay (see above)
constexpr int kSynNear = 64;           // entries of a row's front kept in LDS, at most
constexpr int kSynList = 256;          // pieces a wavefront collects before it takes them
constexpr int kSynAhead = 4;           // accesses per lane that are under way between two steps

__device__ __forceinline__ int* syn_cells_of(const Dev& d, long long n) { return d.syn_cells + (size_t)(n & 7) * d.BN; }
__device__ __forceinline__ unsigned long long syn_mask_load(const Dev& d, int slot2, int g, int w) {
  return __hip_atomic_load(&d.syn_mask[((size_t)slot2 * d.BN + g) * d.syn_mw + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int NPT>
struct SynLds {
  alignas(16) unsigned long long words[kSynLdsWords];   // [R][wpb] spikes; FIFO: [R][wpb] spikes with a mask; fronts [near][chunk]
  unsigned list[kResThreads / 64][kSynList];            // pieces of a wavefront: D << 12 | place
  unsigned short spk[NPT * kResThreads];                // places of the step's spikes
  unsigned char front[NPT * kResThreads];               // entries in the front of a neuron's row (255: as many or more)
  unsigned long long claim[2];                          // the block's spikes of the step << 40 | their events, by step parity
  int dead, n_spk[2];                                   // spikes of the step, by step parity
};

// Collects the pieces (D, place) of all spikes with dlo <= D <= d_max into the wavefront's list and hands them to
// take(number of pieces, whether these are the last) whenever the list may be full and at the end; it returns how many it leaves at the
// list's front, kSynList - 64 at most, none of the last.  slot0: row of the spike words that D = 0 would have.
// Returns the number of pieces; most >= 0: gives up, with -1, when there are more than that (take is not called then).
template <int NPT, class Take>
__device__ __forceinline__ int syn_walk(const Dev& d, SynLds<NPT>& L, int wpb, int dlo, int slot0, int most, Take take) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // (lane by lane over the wavefronts: pieces are shared out evenly, which is worth more than the LDS banks that meet -- sixteen words
  // at a time 7.6 instead of 7.3 ms for 1,000 steps of 10,000 x 1,000 synapses)
  const int t = lane * (kResThreads / 64) + wave;
  unsigned* list = L.list[wave];
  const int items = (d.d_max - dlo + 1) * wpb;
  const int dj = kResThreads / wpb, dw = kResThreads - dj * wpb;
  int j = t / wpb, w = t - j * wpb, np = 0;
  for (int it0 = 0; it0 < items; it0 += kResThreads) {
    unsigned long long bits = 0ull;
    const int D = dlo + j;
    if (it0 + t < items) {
      int s = slot0 - D;
      if (s < 0) s += d.R;
      bits = L.words[s * wpb + w];
    }
    for (;;) {
      const unsigned long long m = __ballot(bits != 0ull);
      if (!m) break;
      if (most >= 0 && np + __popcll(m) > most) return -1;
      if (np > kSynList - 64) np = take(np, false);
      if (bits) {
        list[np + __popcll(m & ((1ull << lane) - 1ull))] = ((unsigned)D << 12) | (unsigned)(w * 64 + __ffsll((long long)bits) - 1);
        bits &= bits - 1;
      }
      np += __popcll(m);
    }
    j += dj; w += dw;
    if (w >= wpb) { w -= wpb; j += 1; }
  }
  if (most < 0 && np) take(np, true);
  return np;
}

// Steps n0 .. n0 + nsteps - 1 (at most kSynChunk).  P taking-part blocks (every stride-th block of the grid), each owning `chunk` <=
// NPT * 512 neurons (a multiple of 64); thread t of a block owns the places t, t + 512, ... .  near: entries of a row's front in
// LDS.  bar_base: sum of the arrival counters when the launch begins.
// DEEP: the front is that of three steps, and what a step adds off the chain was requested in the two steps before.
// (No counters here: the events are counted by k_syn_list, k_syn_flags and k_syn_in_flight.  With them, and the kind a run-time
// value, the kernel spilled 26 vector and 108 scalar registers, and a step of the network above took 5.7 us.)
template <int NPT, bool FIFO, bool DEEP>
__global__ __launch_bounds__(kResLaunch) void k_syn_run(long long n0, int nsteps, unsigned bar_base, int P, int chunk, int stride,
                                                        int near, Dev d) {
  __shared__ SynLds<NPT> L;
  if (blockIdx.x % stride) return;
  const int rank = blockIdx.x / stride;
  if (rank >= P) return;
  const int wpb = chunk >> 6;
  if (threadIdx.x == 0) {
    L.dead = (ld_agent(&d.ctr->err) & ERR_BARRIER) ? 1 : 0;
    L.n_spk[0] = 0; L.n_spk[1] = 0; L.claim[0] = 0ull; L.claim[1] = 0ull;
  }
  const bool worker = threadIdx.x < kResThreads;   // uniform per wavefront
  if (!worker) {
    // the block barriers of a step, in the workers' order
    __syncthreads();
    for (int k = 0; k < nsteps; ++k) {
      if (k > 0) rev_wait(d, bar_base + (unsigned)k * (unsigned)P, &L.dead);
      __syncthreads();                                          // spikes known
      rev_arrive(d, k + 1 < nsteps, rank);
      if (FIFO && !DEEP && L.n_spk[k & 1] > 0) __syncthreads();  // masks made
    }
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kWaves = kResThreads / 64;
  constexpr int kFront = DEEP ? 3 : 1;                          // delays of the front: 1 .. kFront
  const int lo = rank * chunk;
  const int hi = lo + chunk < d.BN ? lo + chunk : d.BN;
  const int nb = d.d_max + 2;
  const int fcol = kFront + 1 < nb - 1 ? kFront + 1 : nb - 1;   // dstart column behind the front
  const int every = d.kind == ADSEQ_SYN_BINS ? d.C : 1;         // LATEST, BINS: a spike replaces those this many steps before it, or a multiple
  const bool syn = d.alpha_s > 0.0f, dexp = d.alpha_r > 0.0f;
  const unsigned long long G64 = 0x9E3779B97F4A7C15ull;
  const int voff = (lo + tid) * 4;   // of the thread's first neuron in a row of 4-byte values; the others 2,048 bytes apart
  constexpr int kRow = kResThreads * 4;
  unsigned long long* const flagged = L.words + (size_t)d.R * wpb;                        // FIFO: spikes with a mask
  uint2* const fronts = reinterpret_cast<uint2*>(L.words + (size_t)d.R * wpb * (FIFO ? 2 : 1));
  // lane c < NPT stores the wavefront's spike word c of the step
  const int blk_word = (lane < NPT && lane * kWaves + wave < wpb) ? lane * kWaves + wave : -1;             // in the block's LDS words
  const int my_word = (blk_word >= 0 && (lo >> 6) + blk_word < d.words) ? (lo >> 6) + blk_word : -1;   // on the tape
  // ---- what outlives a launch
  for (int x = tid; x < d.R * wpb; x += kResThreads) {
    const int s = x / wpb, w = (lo >> 6) + (x - s * wpb);
    L.words[x] = w < d.words ? d.spike_bits[(size_t)s * d.words + w] : 0ull;
    if (FIFO) {   // (of the steps n0 - R .. n0 - 1)
      const int slot_n0 = (int)(n0 % d.R);
      const long long m = n0 - (s < slot_n0 ? slot_n0 - s : slot_n0 - s + d.R);
      flagged[x] = m >= 0 && w < d.words ? d.syn_flagged[(size_t)(m % d.syn_R2) * d.words + w] : 0ull;
    }
  }
  float V[NPT], J[NPT], Jf[NPT];
  unsigned long long zg[NPT];
  int rlen[NPT];
  unsigned actmask = 0;
#pragma unroll
  for (int c = 0; c < NPT; ++c) {
    const int t = c * kResThreads + tid, g = lo + t;
    V[c] = 0.0f; J[c] = 0.0f; Jf[c] = 0.0f; zg[c] = 0ull; rlen[c] = 0;
    int front = 0;
    if (g < hi) {
      actmask |= 1u << c;
      const int i = g - trial_of(d, g) * d.N;
      const long long r0 = d.row_ptr[i];
      rlen[c] = d.rowlen[i];
      front = (int)d.dstart[(size_t)i * nb + fcol];
      V[c] = d.V[g];
      if (syn) J[c] = d.J[g];
      if (dexp) Jf[c] = d.J[(size_t)d.BN + g];
      zg[c] = mix64(d.seed + G64 * ((unsigned long long)g + 1ull));
      for (int q = 0; q < near && q < front; ++q) fronts[q * chunk + t] = d.synf[r0 + q];
    }
    L.front[t] = (unsigned char)(front < 255 ? front : 255);
  }
  int slot = (int)(n0 % d.R), slot2 = (int)(n0 % d.syn_R2);   // rows of the circular words and masks that belong to the step
  if (FIFO && my_word >= 0) q_store<true>(&d.syn_flagged[(size_t)slot2 * d.words + my_word], 0ull);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  // ---- the three accesses for what is added off the chain, each for four pieces at a time.  gsize lanes take a piece.
  const int gshift = d.syn_gshift, per = 64 >> gshift, group = lane >> gshift, sub = lane & ((1 << gshift) - 1);
  auto refused = [&](int D, int place, int slot0, int slot20) {   // FIFO: the spike D steps before slot0's is not admitted at delay D
    int s = slot0 - D;
    if (s < 0) s += d.R;
    if (!((flagged[s * wpb + (place >> 6)] >> (place & 63)) & 1ull)) return false;
    int t = slot20 - D;
    if (t < 0) t += d.syn_R2;
    return !((syn_mask_load(d, t, lo + place, (D - 1) >> 6) >> ((D - 1) & 63)) & 1ull);
  };
  unsigned pcA[kSynAhead], qA0[kSynAhead], qA1[kSynAhead], pcB[kSynAhead];
  long long rA[kSynAhead];
  int npA = 0, npB = -1, leftB[kSynAhead];   // pieces under way (-1: not requested, or more than there is room for; taken in one go when they are due)
#pragma unroll
  for (int u = 0; u < kSynAhead; ++u) { pcA[u] = 0u; qA0[u] = 0u; qA1[u] = 0u; pcB[u] = 0u; rA[u] = 0; leftB[u] = 0; }
  uint2 eB[kSynAhead];
#pragma unroll
  for (int u = 0; u < kSynAhead; ++u) eB[u] = make_uint2(0u, 0u);
  // positions of the row pieces list[t0 ..] requested
  auto request_rows = [&](int t0, int np, int slot0, int slot20) {
    const unsigned* list = L.list[wave];
#pragma unroll
    for (int u = 0; u < kSynAhead; ++u) {
      pcA[u] = 0u; qA0[u] = 0u; qA1[u] = 0u; rA[u] = 0;
      if (t0 + u * per >= np) continue;   // uniform
      const int x = t0 + u * per + group;
      if (x < np) {
        pcA[u] = list[x];
        const int D = (int)(pcA[u] >> 12), place = (int)(pcA[u] & 0xfffu), g = lo + place;
        const int i = g - trial_of(d, g) * d.N;
        if (!(FIFO && !DEEP && refused(D, place, slot0, slot20))) {
          const unsigned* ds = d.dstart + (size_t)i * nb + D;
          qA0[u] = ds[0]; qA1[u] = ds[1];
          rA[u] = d.row_ptr[i];
        }
      }
    }
  };
  // their entries requested (DEEP: the masks of the spikes in question were made at least a step ago, with a block barrier since)
  auto request_entries = [&](int np, int slot0, int slot20) {
#pragma unroll
    for (int u = 0; u < kSynAhead; ++u) {
      if (u * per >= np) continue;   // uniform
      pcB[u] = pcA[u]; leftB[u] = (int)(qA1[u] - qA0[u]) - sub;
      if (FIFO && DEEP && leftB[u] > 0 && refused((int)(pcA[u] >> 12), (int)(pcA[u] & 0xfffu), slot0, slot20)) leftB[u] = 0;
      if (leftB[u] > 0) eB[u] = load_stream(&d.synf[rA[u] + qA0[u] + sub]);
    }
  };
  // and added to the cells of the step they arrive in (slot0: row of the spike words of that step; replaced spikes are left out)
  auto add_entries = [&](int np, int* cells, int slot0) {
#pragma unroll
    for (int u = 0; u < kSynAhead; ++u) {
      if (u * per >= np) continue;   // uniform
      const int place = (int)(pcB[u] & 0xfffu), base = trial_of(d, lo + place) * d.N;
      if (!FIFO && leftB[u] > 0) {
        int s = slot0 - (int)(pcB[u] >> 12);
        if (s < 0) s += d.R;
        if (!((L.words[s * wpb + (place >> 6)] >> (place & 63)) & 1ull)) leftB[u] = 0;
      }
      if (leftB[u] > 0) atomicAdd(&cells[base + (int)(eB[u].x >> d.dbits)], (int)eB[u].y);
      const int more = 1 << gshift;
      if (__ballot(leftB[u] > more) && leftB[u] > more) {   // a piece of more entries than lanes
        const int i = lo + place - base;
        const long long end = d.row_ptr[i] + d.dstart[(size_t)i * nb + (pcB[u] >> 12) + 1];
        for (long long p = end - (leftB[u] - more); p < end; p += more) {
          const uint2 e = load_stream(&d.synf[p]);
          atomicAdd(&cells[base + (int)(e.x >> d.dbits)], (int)e.y);
        }
      }
    }
  };
  auto none = [](int, bool) { return 0; };
  // more pieces than are requested ahead: list[0 .. np) added to the cells of step n + 2 in one go
  auto take_all = [&](int np, int* cells, int slot0, int slot20) {
    for (int t0 = 0; t0 < np; t0 += kSynAhead * per) {
      request_rows(t0, np, slot0, slot20);
      request_entries(np - t0, slot0, slot20);
      add_entries(np - t0, cells, slot0);
    }
  };
  // FIFO, where a source may hold many spikes that were refused: a lane looks one piece up, and only those that are admitted and not empty stay
  // in list[kept ..].  Returns their number.
  auto sift = [&](int kept, int np, int slot0, int slot20) {
    unsigned* const list = L.list[wave];
    unsigned pc[kSynList / 64];
    bool in[kSynList / 64];
#pragma unroll
    for (int u = 0; u < kSynList / 64; ++u) {
      const int x = kept + 64 * u + lane;
      pc[u] = 0u; in[u] = x < np;
      if (in[u]) {
        pc[u] = list[x];
        const int D = (int)(pc[u] >> 12), place = (int)(pc[u] & 0xfffu), g = lo + place;
        const unsigned* ds = d.dstart + (size_t)(g - trial_of(d, g) * d.N) * nb + D;
        const unsigned q0 = ds[0], q1 = ds[1];
        in[u] = !refused(D, place, slot0, slot20) && q1 > q0;
      }
    }
#pragma unroll
    for (int u = 0; u < kSynList / 64; ++u) {
      const unsigned long long m = __ballot(in[u]);
      if (in[u]) list[kept + __popcll(m & ((1ull << lane) - 1ull))] = pc[u];
      kept += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return kept;
  };
  for (int k = 0; k < nsteps; ++k) {
    const long long n = n0 + k;
    const int par = k & 1;
    unsigned xi = 0;
    if (d.p_thresh) {
#pragma unroll
      for (int c = 0; c < NPT; ++c)
        xi |= (mix64(zg[c] + G64 * ((unsigned long long)n + 1ull)) >> 32) < d.p_thresh ? 1u << c : 0u;
    }
    // ---- the adds for step n are in place once every block has arrived
    if (k > 0) rev_wait(d, bar_base + (unsigned)k * (unsigned)P, &L.dead);
    const __amdgpu_buffer_rsrc_t cells = res_rows(syn_cells_of(d, n), hi * 4);
    float U[NPT];
    unsigned smask = 0;
    {
      int acc[NPT];
#pragma unroll
      for (int c = 0; c < NPT; ++c) acc[c] = __builtin_amdgcn_raw_buffer_load_b32(cells, voff, c * kRow, kBufAgent);   // (past the block's last neuron: zero)
#pragma unroll
      for (int c = 0; c < NPT; ++c) {
        float I = (float)acc[c] * 0x1p-24f;
        if (syn) {   // the jumps go into the synaptic current state(s)
          const float jump = I;
          I = __fmaf_rn(d.alpha_s, J[c], jump);
          J[c] = I;
          if (dexp) {
            const float fast = __fmaf_rn(d.alpha_r, Jf[c], jump);
            Jf[c] = fast;
            I = I - fast;
          }
        }
        if (d.p_thresh) I = I + (((xi >> c) & 1u) ? d.ext_w : 0.0f);
        U[c] = __fmaf_rn(d.alpha, V[c], I);
        const bool s = U[c] >= d.theta;
        V[c] = s ? d.v_reset : U[c];
        smask |= s ? 1u << c : 0u;
      }
      smask &= actmask;
    }
    unsigned long long wbits = 0ull;
    if (__ballot(smask != 0u) != 0ull) {
      unsigned long long m[NPT];
      int total = 0, len = 0;
#pragma unroll
      for (int c = 0; c < NPT; ++c) {
        m[c] = __ballot((smask >> c) & 1u);
        if (lane == c) wbits = m[c];
        total += __popcll(m[c]);
        len += ((smask >> c) & 1u) ? rlen[c] : 0;
      }
      const long long lens = wave_total(len);
      int at = 0;
      if (lane == 0) {
        at = atomicAdd(&L.n_spk[par], total);
        atomicAdd(&L.claim[par], ((unsigned long long)total << 40) | (unsigned long long)lens);
      }
      at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
      for (int c = 0; c < NPT; ++c) {
        if ((m[c] >> lane) & 1ull) L.spk[at + __popcll(m[c] & ((1ull << lane) - 1ull))] = (unsigned short)(c * kResThreads + tid);
        at += __popcll(m[c]);
      }
    }
    if (blk_word >= 0) {
      L.words[slot * wpb + blk_word] = wbits;
      if (FIFO) flagged[slot * wpb + blk_word] = 0ull;
    }
    __syncthreads();
    const int nspk = L.n_spk[par];
    if (tid == 0) { L.n_spk[par ^ 1] = 0; L.claim[par ^ 1] = 0ull; }   // (the last step's have been read)
    // ---- what arrives in the next steps; what the spikes replace
    auto add_front = [&](const uint2& e, int base) {   // an entry that arrives at most kFront steps from now
      const int D = kFront == 1 ? 1 : (int)(e.x & d.dmask);
      atomicAdd(&syn_cells_of(d, n + D)[base + (int)(e.x >> d.dbits)], (int)e.y);
    };
    for (int x = wave; x < nspk; x += kWaves) {
      const int place = L.spk[x], g = lo + place;   // (the same in every lane)
      const int b = trial_of(d, g), i = g - b * d.N, base = b * d.N;
      int front = L.front[place];
      if (lane < near && lane < front) add_front(fronts[lane * chunk + place], base);
      if (front > near) {   // the rest of the front from memory
        if (front == 255) front = (int)d.dstart[(size_t)i * nb + fcol];
        const long long r0 = d.row_ptr[i];
        for (int q = near + lane; q < front; q += 64) add_front(load_stream(&d.synf[r0 + q]), base);
      }
      if (!FIFO) {
        // the spike that this one replaces (there is one at most: the others have been replaced by it)
        int age = 0;
        for (int a0 = 0; a0 < d.d_max - 1 && age == 0; a0 += 64 * every) {
          const int a = a0 + every * (lane + 1);
          int s = slot - a;
          if (s < 0) s += d.R;
          const bool held = a < d.d_max && ((L.words[(a < d.d_max ? s : 0) * wpb + (place >> 6)] >> (place & 63)) & 1ull);
          const unsigned long long m = __ballot(held);
          if (m) age = a0 + every * __ffsll((long long)m);
        }
        if (age) {
          int s = slot - age;
          if (s < 0) s += d.R;
          if (lane == 0) atomicAnd(&L.words[s * wpb + (place >> 6)], ~(1ull << (place & 63)));
          // its entries that have been added already: those that arrive in the next step (age + 1 <= d_max) and those of its front
          int last = age + 2 > kFront ? age + 2 : kFront + 1;
          if (last > nb - 1) last = nb - 1;
          const unsigned* ds = d.dstart + (size_t)i * nb;
          const unsigned q0 = ds[age + 1], q1 = ds[last];
          const long long r0 = d.row_ptr[i];
          for (unsigned q = q0 + lane; q < q1; q += 64) {
            const uint2 e = load_stream(&d.synf[r0 + q]);
            const int later = (int)(e.x & d.dmask) - age;   // 1 .. kFront - 1
            atomicAdd(&syn_cells_of(d, n + later)[base + (int)(e.x >> d.dbits)], (int)(0u - e.y));
          }
        }
      }
    }
    rev_arrive(d, k + 1 < nsteps, rank);
    // ---- off the chain: the popped cells cleared (for step n + 8: nobody adds to them before every block has arrived twice
    // more), tape, counts
#pragma unroll
    for (int c = 0; c < NPT; ++c) __builtin_amdgcn_raw_buffer_store_b32(0, cells, voff, c * kRow, kBufAgent);
    {
      const __amdgpu_buffer_rsrc_t tape = res_rows(d.tapeU + (size_t)n * d.BN, hi * 4);
#pragma unroll
      for (int c = 0; c < NPT; ++c) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(U[c]), tape, voff, c * kRow, kBufNonTemporal);
    }
    if (my_word >= 0) d.tape_bits[(size_t)n * d.words + my_word] = wbits;
    if (__ballot(smask != 0u) != 0ull) {
#pragma unroll
      for (int c = 0; c < NPT; ++c)
        if ((smask >> c) & 1u) atomicAdd(&d.spk_count[lo + c * kResThreads + tid], 1);
    }
    if (nspk > 0 && tid == 0) atomicAdd(&d.claims[n], L.claim[par]);
    if (FIFO) {
      if (nspk > 0) {
        // spikes of sources that have C or more in the last d_max - 1 steps: which delays admit them
        for (int x = wave; x < nspk; x += kWaves) {
          const int place = L.spk[x], g = lo + place, pw = place >> 6, pb = place & 63;
          auto held = [&](int a) {   // the source's spike of step n - a is in the words
            int s = slot - a;
            if (s < 0) s += d.R;
            return a < d.d_max && ((L.words[(a < d.d_max ? s : 0) * wpb + pw] >> pb) & 1ull);
          };
          int count = 0;
          for (int a0 = 0; a0 < d.d_max - 1; a0 += 64) count += __popcll(__ballot(held(a0 + lane + 1)));
          if (__builtin_expect(count < d.C, 1)) continue;   // (uniform)
          // The held spikes, 64 at a time: by the list of their ages where that has room for them, else as they come.  A lane has one spike
          // and 64 delays of its mask; each spike's word is then handed to the whole wavefront, whose lanes are the delays.
          const bool listed = count <= kSynList;
          if (listed) {
            int at = 0;
#pragma unroll 1
            for (int a0 = 0; a0 < d.d_max - 1; a0 += 64) {
              const bool has = held(a0 + lane + 1);
              const unsigned long long m = __ballot(has);
              if (has) L.list[wave][at + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned)(a0 + lane + 1);
              at += __popcll(m);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          }
          const int chunks = ((listed ? count : d.d_max - 1) + 63) >> 6;
#pragma unroll 1
          for (int r = 0; r < d.syn_mw; ++r) {
            int mine = 0;   // events in the queues of delay 64 r + lane + 1
#pragma unroll 1
            for (int x = 0; x < chunks; ++x) {
              const int a = !listed ? 64 * x + lane + 1 : (64 * x + lane < count ? (int)L.list[wave][64 * x + lane] : d.d_max);
              const int gone = a - 64 * r;   // (in the queue of delay D while a < D)
              const bool has = gone < 64 && (listed ? a < d.d_max : held(a));
              if (!__ballot(has)) continue;
              unsigned long long w = 0ull;
              if (has) {
                int s = slot - a, t = slot2 - a;
                if (s < 0) s += d.R;
                if (t < 0) t += d.syn_R2;
                w = ((flagged[s * wpb + pw] >> pb) & 1ull) ? syn_mask_load(d, t, g, r) : ~0ull;
                if (gone > 0) w &= ~0ull << gone;
              }
#pragma unroll 1
              for (unsigned long long m = __ballot(w != 0ull); m; m &= m - 1) {
                const int j = __ffsll((long long)m) - 1;
                const unsigned lo32 = lane_get((unsigned)w, j), hi32 = lane_get((unsigned)(w >> 32), j);
                mine += (int)(((lane < 32 ? lo32 : hi32) >> (lane & 31)) & 1u);
              }
            }
            const unsigned long long in = __ballot(mine < d.C && 64 * r + lane < d.d_max);
            if (lane == 0) __hip_atomic_store(&d.syn_mask[((size_t)slot2 * d.BN + g) * d.syn_mw + r], in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (lane == 0) {
            atomicOr(&flagged[slot * wpb + pw], 1ull << pb);
            atomicOr(&d.syn_flagged[(size_t)slot2 * d.words + (g >> 6)], 1ull << pb);
          }
        }
        if (!DEEP) {   // (DEEP: no mask is looked at before the next step's arrival)
          __builtin_amdgcn_s_waitcnt(0x0F70);
          __syncthreads();
        }
      }
      // (the next step's word: acknowledged before that step's masks are made)
      if (my_word >= 0) q_store<true>(&d.syn_flagged[(size_t)(slot2 + 1 == d.syn_R2 ? 0 : slot2 + 1) * d.words + my_word], 0ull);
    }
    // ---- what arrives two steps later
    int* const after = syn_cells_of(d, n + 2);
    if (d.d_max > kFront) {
      const bool due = DEEP && npB >= 0;
      if (due) add_entries(npB, after, slot + 2);
      else {
        int kept = 0;
        syn_walk<NPT>(d, L, wpb, kFront + 1, slot + 2, -1, [&](int np, bool last) {
          if (FIFO) np = kept = sift(kept, np, slot + 2, slot2 + 2);
          if (FIFO && !last && np <= kSynList - 64) return np;
          take_all(np, after, slot + 2, slot2 + 2);
          kept = 0;
          return 0;
        });
      }
      if (DEEP) {
        // (what was under way for the next step is requested anew where the registers were needed)
#pragma unroll 1
        for (int x = due ? 4 : 3; x <= 4; ++x) {
          if (x == 4) { npB = npA; if (npB > 0) request_entries(npB, slot + 3, slot2 + 3); }
          npA = syn_walk<NPT>(d, L, wpb, kFront + 1, slot + x, kSynAhead * per, none);
          if (npA > 0) request_rows(0, npA, slot + x, slot2 + x);
        }
      }
    }
    if (++slot == d.R) slot = 0;
    if (++slot2 == d.syn_R2) slot2 = 0;
  }
  // ---- what outlives the launch
  // (the words were last written before the last step's arrival, which had a block barrier)
  for (int x = tid; x < d.R * wpb; x += kResThreads) {
    const int s = x / wpb, w = (lo >> 6) + (x - s * wpb);
    if (w < d.words) d.spike_bits[(size_t)s * d.words + w] = L.words[x];
  }
#pragma unroll
  for (int c = 0; c < NPT; ++c)
    if ((actmask >> c) & 1u) {
      const int g = lo + c * kResThreads + tid;
      d.V[g] = V[c];
      if (syn) d.J[g] = J[c];
      if (dexp) d.J[(size_t)d.BN + g] = Jf[c];
    }
}

// After a launch of k_syn_run: one block per step writes the step's spikes, in ascending order, and where their admission flags
// begin, and counts the events offered, as admitted for the time being (k_syn_flags takes off what was refused or replaced).
__global__ __launch_bounds__(kBlock) void k_syn_list(Dev d, long long n0) {
  __shared__ long long s_c[kBlock / 64], s_e[kBlock / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const long long n = n0 + blockIdx.x;
  constexpr unsigned long long kEvents = (1ull << 40) - 1ull;
  long long sp = 0, ev = 0;
  for (int k = t; k < (int)blockIdx.x; k += kBlock) { const unsigned long long c = d.claims[n0 + k]; sp += (long long)(c >> 40); ev += (long long)(c & kEvents); }
  // sum over the block
  auto total = [&](long long v, long long* s) {
    const long long w = wave_total64(v);
    __syncthreads();
    if (lane == 0) s[wave] = w;
    __syncthreads();
    long long r = 0;
    for (int x = 0; x < kBlock / 64; ++x) r += s[x];
    return r;
  };
  sp = d.step_off[n0] + total(sp, s_c);
  ev = d.step_evoff[n0] + total(ev, s_e);
  const unsigned long long own = d.claims[n];
  if (t == 0) {
    d.step_off[n + 1] = sp + (long long)(own >> 40);
    d.step_evoff[n + 1] = ev + (long long)(own & kEvents);
    if (blockIdx.x + 1 == gridDim.x) { d.ctr->tape_spikes = sp + (long long)(own >> 40); d.ctr->tape_events = ev + (long long)(own & kEvents); d.ctr->syn_live = 1u; }
  }
  if (own == 0ull) return;   // (uniform)
  const int nw = (d.BN + 63) >> 6;
  for (int w0 = 0; w0 < nw; w0 += kBlock) {
    unsigned long long bits = w0 + t < nw ? d.tape_bits[(size_t)n * d.words + w0 + t] : 0ull;
    long long c = __popcll(bits), e = 0, s = 0;
    for (unsigned long long b = bits; b; b &= b - 1) { const int g = (w0 + t) * 64 + __ffsll((long long)b) - 1; const int i = g - trial_of(d, g) * d.N; e += d.rowlen[i]; s += d.rowsum[i]; }
    s = wave_total64(s);
    // exclusive prefixes over the block
    long long ic = c, ie = e;
    for (int o = 1; o < 64; o <<= 1) {
      const long long uc = __shfl_up(ic, o, 64), ue = __shfl_up(ie, o, 64);
      if (lane >= o) { ic += uc; ie += ue; }
    }
    __syncthreads();
    if (lane == 63) {
      s_c[wave] = ic; s_e[wave] = ie;
      if (ic) {
        BlkCtr& bc = d.blk[blockIdx.x];   // (at most kSynChunk blocks, fewer than there are lines)
        atomicAdd(&bc.offered, (unsigned long long)ie); atomicAdd(&bc.admitted, (unsigned long long)ie);
        atomicAdd((unsigned long long*)&bc.sum_offered, (unsigned long long)s); atomicAdd((unsigned long long*)&bc.sum_admitted, (unsigned long long)s);
      }
    }
    __syncthreads();
    long long at = sp + ic - c, evb = ev + ie - e;
    for (int x = 0; x < kBlock / 64; ++x) {
      if (x < wave) { at += s_c[x]; evb += s_e[x]; }
      sp += s_c[x]; ev += s_e[x];
    }
    for (; bits; bits &= bits - 1, ++at) {
      const int g = (w0 + t) * 64 + __ffsll((long long)bits) - 1;
      const int len = d.rowlen[g - trial_of(d, g) * d.N];
      const bool fits = evb + len <= d.event_cap;
      if (!fits) atomicOr(&d.ctr->err, ERR_TAPE_EVENTS);
      if (at < d.spike_cap) { d.tape_spk[at] = g; d.tape_evb[at] = fits ? evb : -1; }
      else atomicOr(&d.ctr->err, ERR_TAPE_SPIKES);
      evb += len;
    }
  }
}

// Index of the first admission flag of the spike of neuron g at step n, from the tape's spike words: for spikes that the tape's list
// had no room for.  -1: its flags do not fit.  Whole wavefront.
__device__ __forceinline__ long long syn_flag_base(const Dev& d, long long n, int g) {
  long long e = 0;
  for (int w = threadIdx.x & 63; w <= (g >> 6); w += 64) {
    unsigned long long bits = d.tape_bits[(size_t)n * d.words + w];
    if (w == (g >> 6)) bits &= (1ull << (g & 63)) - 1ull;
    for (; bits; bits &= bits - 1) { const int q = w * 64 + __ffsll((long long)bits) - 1; e += d.rowlen[q - trial_of(d, q) * d.N]; }
  }
  e = d.step_evoff[n] + wave_total64(e);
  return e + d.rowlen[g - trial_of(d, g) * d.N] <= d.event_cap ? e : -1;
}

// The age at which the spike of neuron g at step n is replaced (SYN_LATEST, SYN_BINS), by the tape's spike words of steps below
// n_end; 0: it is not, or none of its events is left then.  Whole wavefront.
__device__ __forceinline__ int syn_replaced(const Dev& d, long long n, int g, long long n_end) {
  const int lane = threadIdx.x & 63, every = d.kind == ADSEQ_SYN_BINS ? d.C : 1;
  for (int a0 = 0; a0 < d.d_max - 1; a0 += 64 * every) {
    const int a = a0 + every * (lane + 1);
    const bool hit = a < d.d_max && n + a < n_end && ((d.tape_bits[(size_t)(n + a) * d.words + (g >> 6)] >> (g & 63)) & 1ull);
    const unsigned long long m = __ballot(hit);
    if (m) return a0 + every * __ffsll((long long)m);
  }
  return 0;
}

// The admission flags of the spikes of steps [n0, n1), in the caller's order of the rows, and those of the spikes since n_lo that
// were replaced in these steps.  One wavefront per spike; blockIdx.y: share of a step's spikes.
__global__ __launch_bounds__(kBlock) void k_syn_flags(Dev d, long long n_lo, long long n0, long long n1) {
  const int lane = threadIdx.x & 63;
  const int wave = (int)(blockIdx.y * (kBlock / 64)) + (threadIdx.x >> 6), nwaves = (int)gridDim.y * (kBlock / 64);
  const long long n = n_lo + blockIdx.x;
  int lost = 0;          // events of these spikes that were refused or replaced, and their amplitudes
  long long s_lost = 0;
  auto one = [&](int g, long long evb) {
    const int i = g - trial_of(d, g) * d.N;
    const long long r0 = d.row_ptr[i];
    const int len = d.rowlen[i];
    if (len == 0) return;
    unsigned char* const flag = d.tape_adm + evb;
    bool some = false;
    int age = 0, slot2 = 0;
    if (d.kind == ADSEQ_SYN_FIFO) {
      slot2 = (int)(n % d.syn_R2);
      some = (d.syn_flagged[(size_t)slot2 * d.words + (g >> 6)] >> (g & 63)) & 1ull;
    } else {
      age = syn_replaced(d, n, g, n1);
      some = age > 0;
      if (n < n0 && (!some || n + age < n0)) return;   // (as it was)
    }
    if (!some && evb >= 0) {
      // all ones: whole words in the middle
      int head = (int)((0u - (unsigned)(uintptr_t)flag) & 3u);
      if (head > len) head = len;
      const int mid = (len - head) >> 2, tail = head + 4 * mid;
      if (lane < head) flag[lane] = 1;
      unsigned* const f4 = reinterpret_cast<unsigned*>(flag + head);
      for (int x = lane; x < mid; x += 64) f4[x] = 0x01010101u;
      if (tail + lane < len) flag[tail + lane] = 1;
    }
    if (!some) return;
    for (int q = lane; q < len; q += 64) {
      const int D = (int)(d.packed[r0 + q] & d.dmask);
      const bool in = d.kind == ADSEQ_SYN_FIFO ? (syn_mask_load(d, slot2, g, (D - 1) >> 6) >> ((D - 1) & 63)) & 1ull : D <= age;
      if (evb >= 0) flag[q] = in ? 1 : 0;
      if (!in) { lost += 1; s_lost += d.a_q[r0 + q]; }
    }
  };
  const long long lo = d.step_off[n], hi = d.step_off[n + 1];
  if (hi <= d.spike_cap) {
    for (long long e = lo + wave; e < hi; e += nwaves) one(d.tape_spk[e], d.tape_evb[e]);
  } else {   // (the list is full: the step's spikes from the tape's words)
    for (int w = wave; w < (d.BN + 63) >> 6; w += nwaves)
      for (unsigned long long bits = d.tape_bits[(size_t)n * d.words + w]; bits; bits &= bits - 1) {
        const int g = w * 64 + __ffsll((long long)bits) - 1;
        one(g, syn_flag_base(d, n, g));
      }
  }
  if (__ballot(lost != 0)) {
    const long long t = wave_total(lost), ts = wave_total64(s_lost);
    BlkCtr& bc = d.blk[(blockIdx.x + blockIdx.y * gridDim.x) & (kSynqBlocks - 1)];   // (there are more lines than that)
    if (lane == 0) { atomicAdd(&bc.admitted, 0ull - (unsigned long long)t); atomicAdd((unsigned long long*)&bc.sum_admitted, 0ull - (unsigned long long)ts); }
  }
}

// Events in flight before step n_end (arrival n_end or later) and their amplitudes, added to out[0], out[1]: the tails of the held
// spikes' rows.  One wavefront per spike word.  This and the next two do nothing unless the events are in the spike words.
__global__ __launch_bounds__(kBlock) void k_syn_in_flight(Dev d, long long n_end, unsigned long long* out) {
  if (!d.ctr->syn_live) return;
  const int lane = threadIdx.x & 63;
  const long long items = (long long)d.d_max * d.words, waves = (long long)gridDim.x * (kBlock / 64);
  int c = 0;
  long long s = 0;
  for (long long x = (long long)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); x < items; x += waves) {
    const int age = 1 + (int)(x / d.words), word = (int)(x - (long long)(age - 1) * d.words);
    if (age > n_end) break;
    const long long m = n_end - age;
    unsigned long long bits = d.spike_bits[(size_t)(m % d.R) * d.words + word];
    if (!bits) continue;
    const int t = (int)(m % d.syn_R2);
    const unsigned long long masked = d.kind == ADSEQ_SYN_FIFO ? d.syn_flagged[(size_t)t * d.words + word] : 0ull;
    for (; bits; bits &= bits - 1) {
      const int bit = __ffsll((long long)bits) - 1, g = word * 64 + bit, i = g - trial_of(d, g) * d.N;
      const long long r0 = d.row_ptr[i];
      const int len = d.rowlen[i];
      for (int q = (int)d.dstart[(size_t)i * (d.d_max + 2) + age] + lane; q < len; q += 64) {
        const uint2 e = load_stream(&d.synf[r0 + q]);
        const int D = (int)(e.x & d.dmask);
        if (((masked >> bit) & 1ull) && !((syn_mask_load(d, t, g, (D - 1) >> 6) >> ((D - 1) & 63)) & 1ull)) continue;
        c += 1; s += (int)e.y;
      }
    }
  }
  const long long tc = wave_total(c), ts = wave_total64(s);
  if (lane == 0 && tc) { atomicAdd(&out[0], (unsigned long long)tc); atomicAdd(&out[1], (unsigned long long)ts); }
}
// The queue arrays as three launches per step would have left them before step n_end, from the spike words (the arrays are as a
// reset leaves them).  One wavefront per neuron and trial.
__global__ __launch_bounds__(kBlock) void k_syn_queues(Dev d, long long n_end) {
  __shared__ unsigned short s_age[kBlock / 64][1024];
  if (!d.ctr->syn_live) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned short* const ages = s_age[wave];
  const long long qpad = (((long long)d.B * d.S + 7) >> 3) << 3;
  for (int g = (int)blockIdx.x * (kBlock / 64) + wave; g < d.BN; g += (int)gridDim.x * (kBlock / 64)) {
    // ages n_end - m of the held spikes, the oldest first
    int cnt = 0;
    for (int a0 = (d.d_max + 63) / 64 * 64; a0 > 0; a0 -= 64) {
      const int a = a0 - lane;
      const bool held = a <= d.d_max && a <= n_end && ((d.spike_bits[(size_t)((n_end - a) % d.R) * d.words + (g >> 6)] >> (g & 63)) & 1ull);
      const unsigned long long m = __ballot(held);
      if (held) ages[cnt + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)a;
      cnt += __popcll(m);
    }
    if (cnt == 0) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // the spikes' first admission flags (BINS: of every spike; LATEST: of the last one)
    auto evb_of = [&](int age) {
      long long a = d.step_off[n_end - age], b = d.step_off[n_end - age + 1];
      if (b > d.spike_cap) b = d.spike_cap;
      while (a < b) { const long long mid = (a + b) >> 1; if (d.tape_spk[mid] < g) a = mid + 1; else b = mid; }
      return a < d.spike_cap && d.tape_spk[a] == g ? d.tape_evb[a] : syn_flag_base(d, n_end - age, g);
    };
    const int b = trial_of(d, g), i = g - b * d.N;
    const long long r0 = d.row_ptr[i];
    const int len = d.rowlen[i];
    if (d.kind == ADSEQ_SYN_LATEST) {
      const long long evb = evb_of(ages[cnt - 1]);
      if (lane == 0) d.last_evb[(size_t)(d.spk_count[g] & 1) * d.BN + g] = evb;
    }
    for (int x = 0; x < (d.kind == ADSEQ_SYN_FIFO ? 1 : cnt); ++x) {
      const int age0 = ages[x];
      const long long evb = d.kind == ADSEQ_SYN_BINS ? evb_of(age0) : -1;
      for (int p = lane; p < len; p += 64) {
        const int D = (int)(d.packed[r0 + p] & d.dmask);
        const long long q = (long long)b * d.S + r0 + p;
        if (d.kind == ADSEQ_SYN_FIFO) {
          int size = 0;
          for (int y = 0; y < cnt; ++y) {
            const int age = ages[y];
            if (age > D) continue;
            const long long m = n_end - age;
            const int t = (int)(m % d.syn_R2);
            if (((d.syn_flagged[(size_t)t * d.words + (g >> 6)] >> (g & 63)) & 1ull) &&
                !((syn_mask_load(d, t, g, (D - 1) >> 6) >> ((D - 1) & 63)) & 1ull)) continue;
            if (size >= d.C) break;   // (never: a void run)
            const unsigned short key = (unsigned short)synq_key(m + D);
            if (size == 0) d.sq_next[q] = key;
            d.sq_key[(size_t)q * d.C + size] = key;
            size += 1;
          }
          if (size) d.sq_hs[q] = (unsigned short)size;
        } else if (age0 <= D) {
          const long long k = n_end - age0 + D;
          const long long at = d.kind == ADSEQ_SYN_BINS ? (k % d.C) * qpad + q : q;
          d.sq_next[at] = (unsigned short)synq_key(k);
          if (d.kind == ADSEQ_SYN_BINS && d.sq_flag && evb >= 0) d.sq_flag[at] = evb + p;   // (once the flags are full, none is looked at)
        }
      }
    }
  }
}

// Delivered so far: admitted and no longer in flight.  (The last of the three: from here on the queue arrays hold the events, and are popped
// by kernels that count for themselves.)
__global__ void k_syn_delivered(Dev d, int lines, const unsigned long long* in_flight) {
  if (!d.ctr->syn_live) return;
  long long c = 0, s = 0;
  for (int x = threadIdx.x; x < lines; x += 64) { c += (long long)d.blk[x].admitted; s += d.blk[x].sum_admitted; }
  c = wave_total64(c); s = wave_total64(s);
  if (threadIdx.x == 0) {
    d.blk[0].delivered += (unsigned long long)c - in_flight[0];
    d.blk[0].sum_delivered += s - (long long)in_flight[1];
    d.ctr->syn_live = 0u;
  }
}
