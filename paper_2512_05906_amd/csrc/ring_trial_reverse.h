// Reverse sweep, small networks: a whole sweep in ONE launch, one workgroup per trial, no synchronisation outside the workgroup
// (delta synapse, or one synaptic current state; all queue kinds).  Included by adseq.hip after ring_trial.h.
//
// Trials share nothing in the reverse sweep but the per-synapse sums, so a workgroup that keeps the adjoint rows its spikes gather from in
// LDS needs one block barrier per step, two where there is a spike, where k_bwd_flow needs rows written through to memory, gathers from there and a far gather per
// window (k_bwd_win).  Where the rows of d_max steps do not fit, a spike's row is taken in pieces of H offsets: the piece with the offsets
// (q H, (q + 1) H] is gathered q H steps before the spike's own step, when the rows n + q H + 1 .. n + (q + 1) H are there, and its sum
// waits in Gacc; the spikes are known from the tape.  So a step works on the spikes of up to P steps, listed a step ahead, whose entries
// (the leading 64 of a piece, four pieces per wavefront) are requested then.  Two more wavefronts load what the steps read of the tape,
// four steps ahead: one hands the rows over in LDS, one makes the lists: memory operations complete in order, and the compiler waits for all
// of them where it cannot count them, so that a wavefront which requests tape rows and uses entries waits for memory in every step
// (1.09 us per step so).  A thread owns two neurons: half the wavefronts, half the instructions that every wavefront spends.
// A step without a spike is bound by the barrier and what the reading wavefronts do (0.6 us), one with spikes by the chain barrier ->
// gather -> sum -> barrier -> update (0.9 us more), beyond 32 pieces by the rounds of four per wavefront.  Measured, us per reverse
// step at 0.2 / 1 / 3 / 8 / 20 spikes per step and trial, the kernels over the whole chip / so (400 steps, with everything around them):
//   8 x 1,000 x 100, d_max 50, ring   1.62 1.84 2.10 2.44 2.92 / 0.99 1.37 1.60 2.20 3.91     the same, FIFO   1.83 2.05 2.31 2.72 3.23 / 1.24 1.80 2.18 3.18 5.57
//   8 x 600 x 300, 250 (P = 3)        1.64 1.85 2.16 2.51 3.15 / 1.22 1.74 2.46 4.20 8.26
//   1 x 1,000 x 100, 50               1.94 3.69 5.31 6.06 7.46 / 1.02 1.37 1.63 2.20 3.88     64 x 100 x 100, 50   1.93 2.47 3.21 5.00 11.8 / 0.88 1.53 2.13 3.10 5.72
// Hence a line on the spikes of the run, which the host reads with the error word: a spike weighs a piece more or less, its entries and,
// in the bounded kinds, their admission bits; where it lies, and why, is in reverse_trial_plan.h.
#include "reverse_trial_plan.h"

// A listed piece: first entry, entries, neuron | piece << 16; ADM: first word of the row's admission bits.
struct RevPiece { int p0, len, iq; unsigned adm; };

// T steps of the tape; H adjoint rows in LDS, P = ceil(d_max / H) pieces of a row.  Workers: all wavefronts but the last two.
template <bool HAS_DU, int SURR, int SYN, bool ADM>
__global__ __launch_bounds__(640) void k_bwd_trial(long long T, int H, int P, const float* __restrict__ dL_dcount, const float* __restrict__ dL_dU, Dev d) {
  __shared__ alignas(16) unsigned char lds[kRevTrialLds];
  __shared__ int s_items[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int threads = (int)blockDim.x, waves = (threads >> 6) - 2, half = waves * 64;   // worker wavefronts, worker threads
  const int N = d.N, base = (int)blockIdx.x * N;
  const int w_lo = base >> 6, nwg = ((base + N - 1) >> 6) - w_lo + 1;   // the trial's spike words (the first and the last shared with other trials)
  const int nwords = P * nwg, most = P * ((N + 63) / 64 + 1);
  // ---- LDS
  RevPiece* const items = reinterpret_cast<RevPiece*>(lds);                                    // [2][kRevTrialItems]
  unsigned long long* const words = reinterpret_cast<unsigned long long*>(items + 2 * kRevTrialItems);   // [2][most]
  unsigned* const word_adm = reinterpret_cast<unsigned*>(words + 2 * most);                    // [2][most]
  int* const row0 = reinterpret_cast<int*>(word_adm + 2 * most);                               // [N + 1]
  float* const near = reinterpret_cast<float*>(row0 + N + 1);                                  // [N] queue terms of the step's spikes
  const int NS = (N + 63) & ~63;
  float* const tape = near + N;                                                                // [2][NS] membrane values of a step
  float* const tape_dU = tape + 2 * NS;                                                        // [2][NS] dL/dU
  float* const rows = tape_dU + 2 * NS;                                                        // [H][N] by step mod H
  int* const cut = reinterpret_cast<int*>(rows + (size_t)H * N);                               // [P + 1][N] where the pieces of a row begin
  for (int x = tid; x <= N; x += threads) row0[x] = (int)d.row_ptr[x];
  for (int x = tid; x < H * N; x += threads) rows[x] = 0.0f;
  for (int x = tid; x < 4 * NS; x += threads) tape[x] = 0.0f;
  for (int x = tid; x < (P + 1) * N; x += threads) {
    const int q = x / N, i = x - q * N, D = q * H + 1;
    cut[x] = (int)d.dstart[(size_t)i * (d.d_max + 2) + (D < d.d_max + 1 ? D : d.d_max + 1)];
  }
  __syncthreads();
  if (wave == waves) {
    // ---- the wavefront that loads the rows: 16 values per lane
    constexpr int kAhead = HAS_DU ? 2 : 4;   // (steps whose values are on their way, in registers)
    struct Ahead { float U[16], dU[HAS_DU ? 16 : 1]; };
    // (Every request is made whatever is there to load -- past the end of its descriptor it gives zero --, so that it can be counted what is
    // waited for: requests behind branches were waited for in the next step.)
    auto load_rows = [&](long long m, Ahead& f) {   // (past the trial's end zero)
      const size_t at = (size_t)(m > 0 ? m : 0) * d.BN + base;
      const __amdgpu_buffer_rsrc_t ru = res_rows(d.tapeU + at, N * 4);
#pragma unroll
      for (int c = 0; c < 16; ++c) f.U[c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ru, lane * 4 + 256 * c, 0, kBufNonTemporal));
      if constexpr (HAS_DU) {
        const __amdgpu_buffer_rsrc_t rd = res_rows(dL_dU + at, N * 4);
#pragma unroll
        for (int c = 0; c < 16; ++c) f.dU[c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, lane * 4 + 256 * c, 0, kBufNonTemporal));
      }
    };
    auto store_rows = [&](long long m, const Ahead& f) {
      float* const to = tape + (m & 1) * NS + lane;
#pragma unroll
      for (int c = 0; c < 16; ++c) if (64 * c < N) to[64 * c] = f.U[c];
      if constexpr (HAS_DU) {
        float* const tod = tape_dU + (m & 1) * NS + lane;
#pragma unroll
        for (int c = 0; c < 16; ++c) if (64 * c < N) tod[64 * c] = f.dU[c];
      }
    };
    Ahead F[kAhead];
#pragma unroll
    for (int x = 0; x < kAhead; ++x) load_rows(T - 1 - x, F[x]);
    store_rows(T - 1, F[0]);
    load_rows(T - 1 - kAhead, F[0]);
    __syncthreads();
    int here = s_items[(T - 1) & 1];   // pieces of the step being run
    auto one = [&](long long m, Ahead& f) {   // f: of step m - 1, which there is
      __syncthreads();
      store_rows(m - 1, f);
      load_rows(m - 1 - kAhead, f);
      const int next = s_items[(m - 1) & 1];
      if (here) __syncthreads();
      here = next;
    };
    // (no branch around the requests in the loop, see above)
    long long m = T - 1;
    for (; m >= kAhead; m -= kAhead) {
#pragma unroll
      for (int x = 0; x < kAhead; ++x) one(m - x, F[(x + 1) % kAhead]);
    }
#pragma unroll
    for (int x = 0; x < kAhead; ++x) if (m - x > 0) one(m - x, F[(x + 1) % kAhead]);
    __syncthreads();   // step 0
    if (here) __syncthreads();
    return;
  }
  if (wave == waves + 1) {
    // ---- the wavefront that lists the pieces: up to two spike words per lane
    constexpr int kAhead = 4;
    struct Ahead { unsigned long long W[2]; unsigned A[2]; };
    int wq[2], first[2];
    unsigned long long own[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int t = lane + 64 * c;
      wq[c] = t / nwg; first[c] = (w_lo + t - wq[c] * nwg) << 6;
      own[c] = t < nwords ? (first[c] < base ? ~0ull << (base - first[c]) : ~0ull) & (first[c] + 64 > base + N ? ~0ull >> (first[c] + 64 - base - N) : ~0ull) : 0ull;
    }
    auto load_words = [&](long long m, Ahead& f) {   // of sweep step m
      const long long top = m >= 0 ? m : 0, low = top - (long long)(P - 1) * H > 0 ? top - (long long)(P - 1) * H : 0;   // rows read: low .. top
      const int have = m >= 0 ? (int)(top - low + 1) * d.words : 0;
      const __amdgpu_buffer_rsrc_t rw = res_rows(d.tape_bits + (size_t)low * d.words, have * 8);
      const __amdgpu_buffer_rsrc_t ra = res_rows(d.adm_base + (ADM ? (size_t)low * d.words : 0), have * 4);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const long long n = m - (long long)wq[c] * H;
        const int at = lane + 64 * c < nwords && n >= low ? (int)(n - low) * d.words + (first[c] >> 6) : kFlowNowhere / 8;
        f.W[c] = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(rw, at * 8, 0, 0));
        f.A[c] = ADM ? (unsigned)__builtin_amdgcn_raw_buffer_load_b32(ra, at * 4, 0, 0) : 0u;
      }
    };
    // the pieces of sweep step m, into the list of its parity
    auto list = [&](long long m, const Ahead& f) {
      const int par = (int)(m & 1);
      int count = 0;   // (the same in every lane)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (64 * c >= nwords) break;   // uniform
        const int t = lane + 64 * c;
        if (t < nwords) { words[par * most + t] = f.W[c]; if (ADM) word_adm[par * most + t] = f.A[c]; }
        unsigned adm = f.A[c];
        unsigned long long b = f.W[c] & own[c];
        if (ADM && b) {   // another trial's spikes in front of the trial's: only their words count
          for (unsigned long long o = f.W[c] & ~own[c] & ((b & (0ull - b)) - 1ull); o; o &= o - 1ull) {
            const int i = ((first[c] + __ffsll((long long)o) - 1 - base) % N + N) % N;
            adm += (unsigned)((row0[i + 1] - row0[i] + 63) >> 6);
          }
        }
        while (__ballot(b != 0ull)) {
          bool put = false;
          RevPiece p; p.p0 = 0; p.len = 0; p.iq = 0; p.adm = 0u;
          if (b) {
            const int i = first[c] + __ffsll((long long)b) - 1 - base;
            b &= b - 1ull;
            const int c0 = cut[wq[c] * N + i], c1 = cut[(wq[c] + 1) * N + i];
            // (the first piece is listed even if it is empty: it takes the other pieces' sums in, and a step with a spike has its second
            // barrier, without which the tape row of the step before, which the spike-time rule reads, could still be on its way)
            put = c1 > c0 || wq[c] == 0;
            p.p0 = row0[i] + c0; p.len = c1 - c0; p.iq = i | wq[c] << 16; p.adm = adm;
            if (ADM) adm += (unsigned)((row0[i + 1] - row0[i] + 63) >> 6);
          }
          const unsigned long long m64 = __ballot(put);
          const int at = count + __popcll(m64 & ((1ull << lane) - 1ull));
          if (put && at < kRevTrialItems) items[par * kRevTrialItems + at] = p;
          count += __popcll(m64);
        }
      }
      if (lane == 0) s_items[par] = count;
      return count;
    };
    Ahead F[kAhead];
#pragma unroll
    for (int x = 0; x < kAhead; ++x) load_words(T - 1 - x, F[x]);
    int here = list(T - 1, F[0]);
    load_words(T - 1 - kAhead, F[0]);
    __syncthreads();
    auto one = [&](long long m, Ahead& f) {
      const int next = list(m - 1, f);
      load_words(m - 1 - kAhead, f);
      __syncthreads();
      if (here) __syncthreads();
      here = next;
    };
    long long m = T - 1;
    for (; m >= kAhead; m -= kAhead) {
#pragma unroll
      for (int x = 0; x < kAhead; ++x) one(m - x, F[(x + 1) % kAhead]);
    }
#pragma unroll
    for (int x = 0; x < kAhead; ++x) if (m - x > 0) one(m - x, F[(x + 1) % kAhead]);
    __syncthreads();   // step 0
    if (here) __syncthreads();
    return;
  }
  // ---- workers: thread t owns the neurons t and t + half
  float carry[2], cj[2], dLc[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = tid + c * half;
    carry[c] = 0.0f; cj[c] = 0.0f;
    dLc[c] = i < N && dL_dcount ? dL_dcount[base + i] : 0.0f;
  }
  int mslot = (int)((T - 1) % H), rslot = (int)((T - 1) % d.R);
  constexpr int kAt = 4;   // pieces of a wavefront that are under way together
  uint2 e[kAt]; unsigned long long bits[kAt]; RevPiece pc[kAt];   // the step's first pieces of this wavefront
  float far[kAt];                                            // lane 0: what the other pieces of their spikes add up to
#pragma unroll
  for (int u = 0; u < kAt; ++u) { e[u] = make_uint2(0u, 0u); bits[u] = 0ull; far[u] = 0.0f; pc[u].p0 = 0; pc[u].len = -1; pc[u].iq = 0; pc[u].adm = 0u; }
  auto row_entry = [&](size_t p) {   // (one 8-byte load, and not a non-temporal one: the rows stay in the L2)
    const unsigned long long v = reinterpret_cast<const unsigned long long*>(d.synb)[p];
    return make_uint2((unsigned)v, (unsigned)(v >> 32));
  };
  auto bits_at = [&](const RevPiece& p, int q) {   // the admission bit of the piece's entry q (the lane's)
    const int at = p.p0 - row0[p.iq & 0xffff] + q;
    return q < p.len ? (d.adm_bits[p.adm + (unsigned)(at >> 6)] >> (at & 63)) & 1ull : 0ull;
  };
  auto far_of = [&](const RevPiece& p, int sl) {   // taken out: the slot is another step's R steps on, whose sums begin to arrive two steps later at the earliest
    float v = 0.0f;
    if (P > 1 && (p.iq >> 16) == 0 && lane == 0) v = __hip_atomic_exchange(&d.Gacc[(size_t)sl * d.BN + base + (p.iq & 0xffff)], 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return v;
  };
  auto piece_of = [&](int par, int x) {
    const RevPiece r = items[par * kRevTrialItems + x];
    RevPiece p;
    p.p0 = __builtin_amdgcn_readfirstlane(r.p0); p.len = __builtin_amdgcn_readfirstlane(r.len);
    p.iq = __builtin_amdgcn_readfirstlane(r.iq); p.adm = (unsigned)__builtin_amdgcn_readfirstlane((int)r.adm);
    return p;
  };
  auto request = [&](int par, int count, int sl, int x0) {   // pieces x0, x0 + waves, ...; sl: the step's slot in Gacc
#pragma unroll
    for (int u = 0; u < kAt; ++u) {
      pc[u].len = -1;   // (none)
      if (x0 + u * waves < count) {   // (the same in every lane)
        pc[u] = piece_of(par, x0 + u * waves);
        e[u] = make_uint2(0u, 0u);
        if (lane < pc[u].len) e[u] = row_entry((size_t)pc[u].p0 + lane);
        if (ADM) bits[u] = bits_at(pc[u], lane);
        far[u] = far_of(pc[u], sl);
      }
    }
  };
  __syncthreads();
  int cur_n = s_items[(T - 1) & 1];   // pieces of the step being run
  request((int)((T - 1) & 1), cur_n <= kRevTrialItems ? cur_n : 0, rslot, wave);
  for (long long m = T - 1; m >= 0; --m) {
    const int par = (int)(m & 1);
    const int rslot1 = rslot == 0 ? d.R - 1 : rslot - 1;
    __syncthreads();   // the rows above this step's are complete; so are the step's tape row and the next step's list
    const long long tail = T - 1 - m;   // offsets (beyond q H) up to this arrive within the run
    auto gather = [&](const uint2& x, int q, bool have, float& t) {   // the lane's entry: its adjoint; t: amplitude * adjoint
      const int off = (int)(x.x & d.dmask) - q * H;
      float gv = 0.0f;
      t = 0.0f;
      if (have && off <= tail) {
        int row = mslot + off;
        if (row >= H) row -= H;
        gv = rows[row * N + (int)(x.x >> d.dbits)];
        t = __uint_as_float(x.y) * gv;
      }
      return gv;
    };
    auto finish = [&](const RevPiece& p, float part, float far_sum) {   // the sum of a piece
      const int i = p.iq & 0xffff, q = p.iq >> 16;
      if (lane != 0) return;
      if (q == 0) near[i] = part + far_sum;
      else {
        int sl = rslot - q * H % d.R;
        if (sl < 0) sl += d.R;
        unsafeAtomicAdd(&d.Gacc[(size_t)sl * d.BN + base + i], part);
      }
    };
    auto rest = [&](const RevPiece& p, int q0, float part) {   // entries from q0 on, four times 64 in flight
      for (; q0 < p.len; q0 += 256) {   // uniform
        uint2 x[4]; unsigned long long b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q0 + 64 * u + lane;
          x[u] = make_uint2(0u, 0u); b[u] = 1ull;
          if (q < p.len) { x[u] = row_entry((size_t)p.p0 + q); if (ADM) b[u] = bits_at(p, q); }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = q0 + 64 * u + lane;
          float t;
          const float gv = gather(x[u], p.iq >> 16, q < p.len && b[u], t);
          if (gv != 0.0f) unsafeAtomicAdd(&d.gsum[(size_t)p.p0 + q], gv);
          part += t;
        }
      }
      return wave_sum_f(part);
    };
    const int n_here = cur_n;
    cur_n = m > 0 ? s_items[par ^ 1] : 0;
    if (n_here) {
      float sum[kAt], gvs[kAt], fars[kAt]; RevPiece done[kAt];
      auto take = [&]() {   // what has been requested, so that the registers are free
#pragma unroll
        for (int u = 0; u < kAt; ++u) {
          done[u] = pc[u]; fars[u] = far[u];
          gvs[u] = sum[u] = 0.0f;
          if (pc[u].len > 0) gvs[u] = gather(e[u], pc[u].iq >> 16, lane < pc[u].len && (!ADM || bits[u]), sum[u]);   // (uniform)
        }
      };
      auto put = [&]() {   // (the adds to memory behind the next requests)
#pragma unroll
        for (int u = 0; u < kAt; ++u) {
          if (done[u].len < 0) continue;   // uniform
          if (gvs[u] != 0.0f) unsafeAtomicAdd(&d.gsum[(size_t)done[u].p0 + lane], gvs[u]);
          finish(done[u], done[u].len > 64 ? rest(done[u], 64, sum[u]) : wave_sum_f(sum[u]), fars[u]);
        }
      };
      take();
      if (n_here <= kRevTrialItems) {
        for (int x = wave + kAt * waves; x < n_here; x += kAt * waves) { request(par, n_here, rslot, x); put(); take(); }   // uniform
        request(par ^ 1, cur_n <= kRevTrialItems ? cur_n : 0, rslot1, wave);
        put();
      } else {
        // more than the list holds: the words, one by one
        request(par ^ 1, cur_n <= kRevTrialItems ? cur_n : 0, rslot1, wave);
        for (int x = wave; x < nwords; x += waves) {
          const int q = x / nwg, first = (w_lo + x - q * nwg) << 6;
          unsigned adm = ADM ? word_adm[par * most + x] : 0u;
          for (unsigned long long b = words[par * most + x]; b; b &= b - 1ull) {
            int i = first + __ffsll((long long)b) - 1 - base;
            const bool mine = i >= 0 && i < N;
            if (!mine) i = (i % N + N) % N;
            i = __builtin_amdgcn_readfirstlane(i);
            RevPiece p;
            p.p0 = __builtin_amdgcn_readfirstlane(row0[i] + cut[q * N + i]);
            p.len = __builtin_amdgcn_readfirstlane(cut[(q + 1) * N + i] - cut[q * N + i]);
            p.iq = i | q << 16; p.adm = adm;
            if (ADM) adm += (unsigned)((row0[i + 1] - row0[i] + 63) >> 6);
            if (mine && (p.len > 0 || q == 0)) {
              const float f = far_of(p, rslot);
              finish(p, rest(p, 0, 0.0f), f);
            }
          }
        }
      }
      __syncthreads();   // the sums of the step's spikes are there, the rows it replaces used up
    } else {
      request(par ^ 1, cur_n <= kRevTrialItems ? cur_n : 0, rslot1, wave);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = tid + c * half;
      if (i < N) {
        const float U = tape[par * NS + i], dU = HAS_DU ? tape_dU[par * NS + i] : 0.0f;
        float gu;
        if (U >= d.theta) {
          const float G = near[i];
          // (the membrane value the step started from: that of the step before; only the spike-time rule looks at it)
          const float before = SURR == ADSEQ_GRAD_SPIKE_TIME && m > 0 ? tape[(par ^ 1) * NS + i] : 0.0f;
          carry[c] = bwd_update_as<SURR>(d, m, U, before, true, 0.0f, dLc[c], G, dU, &gu);
        } else {
          carry[c] = bwd_update_as<SURR>(d, m, U, 0.0f, false, carry[c], dLc[c], 0.0f, dU, &gu);
        }
        if (SYN) { cj[c] = __fmaf_rn(d.alpha_s, cj[c], gu); gu = cj[c]; }
        rows[mslot * N + i] = gu;
      }
    }
    if (P > 1 && (m & 7) == 0) __builtin_amdgcn_s_waitcnt(0x0F70);   // (far sums are read at least 16 steps after they were sent: they are there)
    mslot = mslot == 0 ? H - 1 : mslot - 1;
    rslot = rslot1;
  }
}

// RING: spikes on the tape, where the host reads them together with the error word.  One block stores the sum, several (tape_total_blocks) add
// to zero: a block's loop over the cells is a chain of trips to memory (512 x 1,000 cells, us per adseq_backward of 10 steps: by one
// block of 4-byte loads 296, without the sum at all 159, so 162).
__global__ __launch_bounds__(1024) void k_tape_total(Dev d) {
  __shared__ unsigned long long s_sum;
  if (threadIdx.x == 0) s_sum = 0ull;
  __syncthreads();
  const int whole = d.BN >> 2;   // (the counts begin on 256 bytes)
  long long c = 0;
  for (int x = (int)(blockIdx.x * 1024 + threadIdx.x); x < whole; x += (int)gridDim.x * 1024) {
    const int4 v = reinterpret_cast<const int4*>(d.spk_count)[x];
    c += (long long)v.x + v.y + v.z + v.w;
  }
  if (blockIdx.x == 0 && threadIdx.x < (d.BN & 3)) c += d.spk_count[4 * whole + (int)threadIdx.x];
  c = wave_total64(c);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(&s_sum, (unsigned long long)c);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (gridDim.x == 1) d.ctr->in_flight[0] = s_sum;
    else if (s_sum) atomicAdd(&d.ctr->in_flight[0], s_sum);
  }
}
// A block up to 16,384 cells, four loads of a thread; beyond, one for every 8,192.
inline unsigned tape_total_blocks(int BN) { return BN <= 16384 ? 1u : (unsigned)((BN + 8191) / 8192); }
