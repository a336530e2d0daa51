// Ring queue, forward, small networks: a whole run in ONE launch, one workgroup per trial, no synchronisation outside the
// workgroup.  Included by adseq.hip after synapse_resident.h.
//
// Trials do not exchange anything, and where a trial's whole delay line [R][N] fits LDS a spike adds its entries there at once: a
// step needs two block barriers where the kernels over one XCD or the whole chip need a barrier through memory, the cells' trip from
// the L2, the adds' acknowledgement, and the window's expansion besides.  The front of every row is in LDS too, as far as there
// is room; what is behind it is one trip to the L2.  A step is bound by the instructions of the one compute unit (drive hash, update)
// and by its LDS.  Measured, us per forward step, by launches per window / so: 100 neurons x 10 synapses 2.3 / 0.43; 3 trials x 212 x 253
// 3.4 / 0.48; 756 x 95 2.2 / 0.63; 100 x 10 with 50 spikes per step 9.1 / 5.4.  Faster at all of 0.2 to 50 % of the neurons firing, 10 to 1,000 synapses
// per neuron, 100 to 1,000 neurons, 1 to 512 trials (see trial_long).
// (An earlier form kept a window of eight rows in LDS and added the entries of all held spikes two steps ahead, as k_syn_run does; it
// took 16 x 1,000 neurons, d_max 50, from 2.0 to 1.7 us per step, but with 500 spikes per step and trial from 21 to 71.)
//
// Between launches there is nothing but what the other forward kernels leave, too: circular spike words, the window of the next step,
// counters, barrier arrivals.  A launch rebuilds its cells from the spike words and hands everything back at its end, so any other
// entry point, captured or not, may come before or after it.

constexpr int kTrialNeurons = 1024;
constexpr int kTrialMost = 512;                  // trials: a workgroup fills a compute unit's LDS, so that 256 run at a time, two rounds of 0.5 us per step
// Long rows: a step with many spikes is a chain of trips to the L2 for every wavefront, so there sixteen share them, and each requests a row's
// next piece before it adds the last one.  One trial, us per step at 0.2, 2, 10, 30 and 50 % of the neurons firing, by launches per window / short
// rows' way / long rows': 250 x 1,000, d_max 50: 3.1 10.6 24 41 54 / 1.1 4.7 17 54 86 / 1.1 2.2 4.3 11 17; 1,000 x 262, d_max 30: 3.7 8.6 21 46 70 /
// 1.5 3.1 12 35 58 / 1.3 2.5 7.9 22 36; 250 x 130: 1.9 3.0 6.7 10 13.6 / 0.68 1.4 3.9 10 16 / 0.74 1.2 2.0 3.9 5.8; 100 x 262: 2.2 4.4 11 15 20 /
// 0.53 1.2 3.4 9.1 15 / 0.62 1.05 1.5 2.3 3.1.  The line: where the short rows' way could be slower than launches (100 x 1,000 and 250 x 130 at half the
// neurons firing, 4 trials of 1,000 x 260 at 30 %), and no lower, since it is up to a sixth faster while little spikes.
constexpr bool trial_long(int N, long long synapses) { return synapses > (N <= 128 ? 512 : (N <= 256 ? 128 : 256)) * (long long)N; }
// (what every wavefront does costs the compute unit as often as there are wavefronts)
constexpr int trial_threads(int N, bool long_rows) { return long_rows ? 1024 : (N <= 128 ? 128 : (N <= 256 ? 256 : 1024)); }
constexpr int kTrialLdsWords = 18432;            // 8-byte words of LDS for cells, spike words and fronts
constexpr long long kTrialSynapses = 262144;     // synapses of a trial at most: 2 MB of rows, which the L2 holds
constexpr long long kTrialSteps = 64;            // steps of a call at least: a launch takes in the fronts and rebuilds the cells (100 neurons, in
                                                 // calls of 64 steps 1.7 / 0.63 us per step)

// Where the R rows do not fit, H rows are held and a spike's row is taken in up to kTrialPieces pieces of H offsets: the piece with the offsets
// (q H, (q + 1) H] is added q H steps after the spike, when the rows it adds to are those of the next H steps.  The spikes of those steps
// back are in the spike words, so that a step just lists them beside its own.  (With windows of eight rows, see above, the pieces were seven.)
// us per forward step by launches per window / so, 0.2, 2, 10, 30 and 50 % of the neurons firing:
//   1,000 x 100, d_max 50 (P = 2), 16 trials 2.40 3.15 8.3 21 34 / 1.24 2.38 6.3 15.5 24.5, one 2.74 3.76 7.0 15.6 23.7 / 1.23 2.34 6.3 15.5 24.4
//   1,024 x 50, 45 (2), 16 trials 2.39 2.73 5.9 14.0 21.6 / 1.17 2.24 5.7 13.8 22.0, one 2.48 3.28 5.6 12.1 18.2 / 1.16 2.20 5.6 13.7 22.0
//   1,000 x 262, 50 (2), 64 trials 3.8 9.6 52 167 282 / 1.39 2.95 9.1 24 39, 4 2.39 3.77 9.1 21.8 34.5 / 1.39 2.95 9.1 24.1 39.1
//   700 x 300, 120 (3), 16 trials 2.39 4.1 8.6 16.3 24.6 / 1.38 2.95 8.9 22.9 37.0;  1,000 x 20, 100 (4), 16 trials 2.05 2.32 4.2 9.2 14.0 / 1.35 3.62 9.9 24.6 39.2
// (16 x 1,000 x 100 at 0.2 spikes per step and trial: 2.06 / 0.83.)  A piece is a trip to the L2 whatever it holds, and one compute unit has
// only so many under way: two pieces of 24 entries and more, and long rows or single trials only where that was no slower, or hardly,
// with a third of the neurons firing in every step (trial_pieces_pay).  At 0.2, 2, 10, 30 and 60 % of them, other sizes: 500 x 100, 100 (2), one trial 1.7 3.1 5.6 11.7 20.4 / 1.0 2.1 4.4 9.8
// 17.7, 16 1.8 2.5 5.9 13.9 25.4 / 1.0 2.1 4.5 9.8 17.8; 500 x 400, 100 (2), 32 trials 2.4 5.3 20.5 62.5 127 / 1.2 2.5 6.4 15.4 28.8; 250 x 1,000, 200 (2), 32 2.4 7.8 19.8 61 124 / 1.3 3.0 5.3
// 12.8 23.8; 300 x 50, 200 (2), 32 1.9 2.5 4.2 9.7 17.7 / 1.0 1.9 2.7 5.2 8.8; 1,000 x 100, 50 (2), 256 3.2 7.7 84 267 542 / 1.2 2.1 7.8 19.6 36.5, 512 3.8 13.7 174 543 1,095 / 2.1 3.9 15.5 38.5 72.9.
inline bool trial_pieces_pay(int P, double row, int batch) { return P == 2 && row >= 48.0 && (batch >= 32 || (row <= 128.0 && (batch >= 16 || row >= 90.0))); }
// Fewer than 16 trials only in calls of so many steps: the other kernels have few blocks then, and taking in the state and adding what is under way is most of a
// short call.  us per step by launches per window / so, 1 x 1,000 x 100 in calls of 64, 128, 256 steps: 5 spikes per step 3.1 3.0 3.0 / 2.1 1.8 1.7, 100 6.9 6.9 6.8 / 8.3 7.0 6.4, 400 19.2
// 19.1 19.1 / 26.1 21.8 19.6 (in one call of 300: 300 16.0 / 17.0, 600 28.2 / 31.7); 16 trials in calls of 64: 100 8.2 / 8.5, 400 26.5 / 26.6.
// (From 256 steps on would cost calls of 128 to 255 more at loads up to a twentieth of the neurons than it gives at a third.)
inline long long trial_steps_least(int P, int batch) { return P > 1 && batch < 16 ? 128 : kTrialSteps; }
constexpr int kTrialPieces = 4;

template <int kMost>
struct TrialLds {
  alignas(16) unsigned long long words[kTrialLdsWords];   // spikes [R][wpb]; fronts [near][N]; cells [R][N] by step mod R
  unsigned short spk[kMost];                            // the step's spikes; PIECES: see there
  int row[kMost + 1];                                   // LONG: where the rows begin
  int n_spk[2];                                         // spikes of the step, by step parity
};

// Steps n0 .. n0 + nsteps - 1 of trial blockIdx.x; N <= blockDim.x <= kMost, thread t owns neuron t.  LONG: see trial_long.  near: entries of a row's
// front in LDS.  record: the tape is written; its spike words of these steps are zero when the launch begins.
// Spikes of steps [fold_lo, fold_hi) and the events they emit are counted: fold_lo <= n0, fold_hi the last window boundary of these
// steps (fold_lo if there is none), as where the other kernels stop counting, so that what is listed on top of the last step is still
// counted later.  Both n0 - fold_lo and n0 + nsteps - fold_hi are at most W < R.
// arrivals: what the barriers of these steps would have added to the arrival counter that the host counts along with (arrive_bar: that
// of the kernels over one XCD).
// PIECES: H rows of cells, P pieces of a row (else H = R, P = 1, near > 0); in LDS behind the cells where the pieces of every row begin, and
// the step's list: neuron | piece << 10, P N entries.
template <int kMost, bool LONG, bool PIECES>
__global__ __launch_bounds__(kMost) void k_trial_run(long long n0, int nsteps, int near, int record, long long fold_lo, long long fold_hi,
                                                     unsigned arrivals, int arrive_bar, Dev d, int H_, int P) {
  __shared__ TrialLds<kMost> L;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int threads = (int)blockDim.x, waves = threads >> 6;
  const int N = d.N, wpb = (N + 63) >> 6, R = d.R;
  const int base = (int)blockIdx.x * N, g = base + tid;
  const bool act = tid < N;
  const int H = PIECES ? H_ : R;
  const bool syn = d.alpha_s > 0.0f, dexp = d.alpha_r > 0.0f;
  const unsigned long long G64 = 0x9E3779B97F4A7C15ull;
  uint2* const fronts = reinterpret_cast<uint2*>(L.words + (size_t)R * wpb);
  int* const cells = reinterpret_cast<int*>(L.words + (size_t)R * wpb + (size_t)near * N);
  int* const cut = cells + (size_t)H * N;                                                     // PIECES: [P + 1][N]
  unsigned short* const spk = PIECES ? reinterpret_cast<unsigned short*>(cut + (size_t)(P + 1) * N) : &L.spk[0];
  // offsets up to this have been added for a spike `age` steps ago
  auto added = [&](int age) { return ((age - 1) / H + 1) * H; };
  // The trial's spike word x = step slot * wpb + word: bits [sh, ..) of the circular words' at[0], the rest in at[1] (hi: there is a
  // rest).  Trials share words: of such a word only the trial's own bits are looked at or changed.
  struct Place { unsigned long long* at; int sh; unsigned long long own; bool hi; };
  auto place = [&](int x) {
    const int s = x / wpb, w = x - s * wpb, n = N - w * 64 < 64 ? N - w * 64 : 64, g0 = base + w * 64;
    Place p;
    p.at = d.spike_bits + (size_t)s * d.words + (g0 >> 6);
    p.sh = g0 & 63;
    p.own = n < 64 ? (1ull << n) - 1ull : ~0ull;
    p.hi = p.sh + n > 64;
    return p;
  };
  auto held = [&](const Place& p) { return ((p.at[0] >> p.sh) | (p.hi ? p.at[1] << (64 - p.sh) : 0ull)) & p.own; };
  for (int x = tid; x < R * wpb; x += threads) L.words[x] = held(place(x));
  for (int x = tid; x < H * N; x += threads) cells[x] = 0;
  if (PIECES)
    for (int x = tid; x < (P + 1) * N; x += threads) {
      const int q = x / N, i = x - q * N, D = q * H + 1;
      cut[x] = (int)d.row_ptr[i] + (int)d.dstart[(size_t)i * (d.d_max + 2) + (D < d.d_max + 1 ? D : d.d_max + 1)];
    }
  if (tid < 2) L.n_spk[tid] = 0;
  if (LONG) for (int x = tid; x <= N; x += threads) L.row[x] = (int)d.row_ptr[x];
  float V = 0.0f, J = 0.0f, Jf = 0.0f;
  unsigned long long zg = 0ull;
  int count = 0;
  if (act) {
    const long long r0 = d.row_ptr[tid], len = d.row_ptr[tid + 1] - r0;
    V = d.V[g];
    if (syn) J = d.J[g];
    if (dexp) Jf = d.J[(size_t)d.BN + g];
    zg = mix64(d.seed + G64 * ((unsigned long long)g + 1ull));
    for (int q = 0; q < near && q < len; ++q) fronts[q * N + tid] = d.synf[r0 + q];
  }
  int slot = (int)(n0 % R);   // row of spike words that belongs to the step
  int piece_row = PIECES ? (int)(n0 % H) : 0;
  int& crow = PIECES ? piece_row : slot;   // and of cells
  __syncthreads();
  // the thread's spikes of the last `steps` steps before the one of `slot`
  auto recent = [&](int steps) {
    int c = 0;
    for (int a = 1; a <= steps; ++a) {
      int s = slot - a;
      if (s < 0) s += R;
      c += (int)((L.words[s * wpb + (tid >> 6)] >> (tid & 63)) & 1ull);
    }
    return c;
  };
  const int before = act ? recent((int)(n0 - fold_lo)) : 0;
  // ---- the cells as the steps before n0 left them: the tails of the held spikes' rows, a wavefront per spike word
  if (n0 > 0)
    for (int x = wave; x < d.d_max * wpb; x += waves) {
      const int age = 1 + x / wpb, w = x - (age - 1) * wpb;
      int s = slot - age;
      if (s < 0) s += R;
      unsigned long long bits = L.words[s * wpb + w];
      for (; bits; bits &= bits - 1) {
        const int i = w * 64 + __ffsll((long long)bits) - 1;
        const int r0 = (int)d.row_ptr[i];
        const int last = PIECES && added(age) < d.d_max ? added(age) + 1 : d.d_max + 1;   // (first offset that has not been added)
        const int r1 = r0 + (int)d.dstart[(size_t)i * (d.d_max + 2) + last];
        for (int q = r0 + (int)d.dstart[(size_t)i * (d.d_max + 2) + age] + lane; q < r1; q += 64) {
          const uint2 e = load_stream(&d.synf[q]);
          int row = crow + (int)(e.x & d.dmask) - age;
          if (row >= H) row -= H;
          atomicAdd(&cells[row * N + (int)(e.x >> d.dbits)], (int)e.y);
        }
      }
    }
  for (int k = 0; k < nsteps; ++k) {
    const long long n = n0 + k;
    const int par = k & 1;
    const bool xi = d.p_thresh && (mix64(zg + G64 * ((unsigned long long)n + 1ull)) >> 32) < d.p_thresh;
    __syncthreads();   // everything due at step n has been added
    float U = 0.0f;
    bool spike = false;
    if (act) {
      int* const cell = &cells[crow * N + tid];
      float I = (float)*cell * 0x1p-24f;
      *cell = 0;   // (for step n + H)
      if (syn) {   // the jumps go into the synaptic current state(s)
        const float jump = I;
        I = __fmaf_rn(d.alpha_s, J, jump);
        J = I;
        if (dexp) {
          const float fast = __fmaf_rn(d.alpha_r, Jf, jump);
          Jf = fast;
          I = I - fast;
        }
      }
      if (d.p_thresh) I = I + (xi ? d.ext_w : 0.0f);
      U = __fmaf_rn(d.alpha, V, I);
      spike = U >= d.theta;
      V = spike ? d.v_reset : U;
      count += spike ? 1 : 0;
    }
    const unsigned long long m = __ballot(spike);
    if (lane == 0 && wave < wpb) L.words[slot * wpb + wave] = m;
    if (m) {   // uniform
      int at = 0;
      if (lane == 0) at = atomicAdd(&L.n_spk[par], __popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      if (spike) spk[at + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)tid;
      if (record && lane < 2) {
        // the tape's words count from the first trial's first neuron
        const int gw = base + wave * 64, sh = gw & 63;
        const unsigned long long part = lane == 0 ? m << sh : (sh ? m >> (64 - sh) : 0ull);
        if (part) atomicOr(&d.tape_bits[(size_t)n * d.words + (gw >> 6) + lane], part);
      }
    }
    if (PIECES && tid < (P - 1) * wpb) {   // the spikes q H steps ago
      const int q = 1 + tid / wpb, w = tid - (q - 1) * wpb;
      if (q * H < d.d_max) {   // (never more than R - 1 steps back)
        int s = slot - q * H;
        if (s < 0) s += R;
        unsigned long long b = L.words[s * wpb + w];
        if (b) {
          int at = atomicAdd(&L.n_spk[par], __popcll(b));
          for (; b; b &= b - 1ull) spk[at++] = (unsigned short)((w * 64 + __ffsll((long long)b) - 1) | q << 10);
        }
      }
    }
    __syncthreads();   // spikes known, cells of the step taken
    const int nspk = __builtin_amdgcn_readfirstlane(L.n_spk[par]);
    if (tid == 0) L.n_spk[par ^ 1] = 0;   // (the last step's has been read)
    auto add = [&](const uint2& e) {
      int row = crow + (int)(e.x & d.dmask);
      if (row >= H) row -= H;
      atomicAdd(&cells[row * N + (int)(e.x >> d.dbits)], (int)e.y);
    };
    if (LONG && wave < nspk) {   // uniform
      // the rows of every waves-th spike, 64 at most: lane j has the j-th one's neuron and row
      int own = 0, first = 0, length = 0;
      if (wave + lane * waves < nspk) { own = spk[wave + lane * waves]; first = L.row[own]; length = L.row[own + 1] - first; }
      // What is behind the front, 256 entries at a time: a piece is requested before the one ahead of it is added.  (A request is four
      // loads whatever is left of the row, so that it can be counted what is waited for.)
      int x = wave, j = 0, r0 = lane_get(first, 0), len = lane_get(length, 0), q0 = near;
      auto request = [&](uint2 (&e)[4], int& left) {
        while (x < nspk && q0 >= len) {
          x += waves; ++j;
          if (x < nspk) { r0 = lane_get(first, j); len = lane_get(length, j); q0 = near; }
        }
        const int here = x < nspk ? len - q0 : 0;
        const __amdgpu_buffer_rsrc_t piece = res_rows(d.synf + r0 + q0, here * 8);
        left = here - lane;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const unsigned long long v = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(piece, lane * 8 + 512 * u, 0, 0));
          e[u] = make_uint2((unsigned)v, (unsigned)(v >> 32));
        }
        q0 += 256;
        return here > 0;
      };
      auto put = [&](const uint2 (&e)[4], int left) {
#pragma unroll
        for (int u = 0; u < 4; ++u) if (64 * u < left) add(e[u]);
      };
      auto add_fronts = [&]() {
        for (int y = wave, f = 0; y < nspk; y += waves, ++f)
          if (lane < near && lane < lane_get(length, f)) add(fronts[lane * N + lane_get(own, f)]);
      };
      if (__ballot(length > near) == 0ull) {
        add_fronts();
      } else {
        uint2 ea[4], eb[4];
        int la = 0, lb = 0;
        bool more = request(ea, la);
        add_fronts();
        while (more) {
          more = request(eb, lb);
          put(ea, la);
          if (!more) break;
          more = request(ea, la);
          put(eb, lb);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // (vmcnt(0): else it is waited for, and the tape's store with it, before every use of the registers)
      }
    }
    if constexpr (PIECES) {
      // four pieces of a wavefront under way together (eight: 0.83 -> 0.98 us per step of 16 x 1,000 at 0.2 spikes)
      for (int x0 = wave; x0 < nspk; x0 += 4 * waves) {   // uniform
        int p0[4], p1[4], back[4]; uint2 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int x = x0 + u * waves;
          p0[u] = 0; p1[u] = 0; back[u] = 0; e[u] = make_uint2(0u, 0u);
          if (x < nspk) {
            const int v = __builtin_amdgcn_readfirstlane((int)spk[x]), i = v & 1023, q = v >> 10;
            p0[u] = __builtin_amdgcn_readfirstlane(cut[q * N + i]); p1[u] = __builtin_amdgcn_readfirstlane(cut[(q + 1) * N + i]); back[u] = q * H;
            const __amdgpu_buffer_rsrc_t piece = res_rows(d.synf + p0[u], (p1[u] - p0[u] < 64 ? p1[u] - p0[u] : 64) * 8);
            const unsigned long long r = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(piece, lane * 8, 0, 0));
            e[u] = make_uint2((unsigned)r, (unsigned)(r >> 32));
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          auto put = [&](const uint2& x) {
            int row = crow + (int)(x.x & d.dmask) - back[u];
            if (row >= H) row -= H;
            atomicAdd(&cells[row * N + (int)(x.x >> d.dbits)], (int)x.y);
          };
          if (p0[u] + lane < p1[u]) put(e[u]);
          for (int p = p0[u] + 64 + lane; p < p1[u]; p += 256) {
            uint2 t[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { t[c] = make_uint2(0u, 0u); if (p + 64 * c < p1[u]) t[c] = d.synf[p + 64 * c]; }
#pragma unroll
            for (int c = 0; c < 4; ++c) if (p + 64 * c < p1[u]) put(t[c]);
          }
        }
      }
    } else if constexpr (!LONG)
      for (int x = wave; x < nspk; x += waves) {
        const int i = spk[x];   // (the same in every lane)
        const int r0 = (int)d.row_ptr[i], len = (int)d.row_ptr[i + 1] - r0;
        if (lane < near && lane < len) add(fronts[lane * N + i]);
        for (int q0 = near + lane; q0 < len; q0 += 256) {   // what is behind the front: four loads under way
          uint2 e[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) { e[u] = make_uint2(0u, 0u); if (q0 + 64 * u < len) e[u] = load_stream(&d.synf[r0 + q0 + 64 * u]); }
#pragma unroll
          for (int u = 0; u < 4; ++u) if (q0 + 64 * u < len) add(e[u]);
        }
      }
    if (record && act) __builtin_nontemporal_store(U, &d.tapeU[(size_t)n * d.BN + g]);
    if (++slot == R) slot = 0;
    if (PIECES && ++piece_row == H) piece_row = 0;
  }
  __syncthreads();
  // ---- what outlives the launch.  Spike words: the bits that have changed
  for (int x = tid; x < R * wpb; x += threads) {
    const Place p = place(x);
    const unsigned long long flip = held(p) ^ L.words[x];
    if (flip << p.sh) atomicXor(&p.at[0], flip << p.sh);
    if (p.hi && (flip >> (64 - p.sh))) atomicXor(&p.at[1], flip >> (64 - p.sh));
  }
  // the window of the next step from there on (if that step opens a window, it is empty as yet), and nothing in the one this launch began in
  const long long end = n0 + nsteps;
  const int phi = (int)(end & (long long)(d.W - 1));
  int* const win = win_of(d, end);
  int* const first = n0 > 0 ? win_of(d, n0 - 1) : win;
  for (int x = tid; x < d.W * N; x += threads) {
    const int r = x / N, i = x - r * N;
    int s = crow + r - phi;
    if (s >= H) s -= H;
    if (phi) win[(size_t)r * d.BN + base + i] = r >= phi && r - phi < H ? cells[s * N + i] : 0;
    if (first != win || !phi) first[(size_t)r * d.BN + base + i] = 0;
  }
  if (PIECES && phi) {
    // what of the held spikes' rows has not been added yet and arrives in this window
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();   // (the cells are in memory)
    for (int x = wave; x < d.d_max * wpb; x += waves) {
      const int age = 1 + x / wpb, w = x - (age - 1) * wpb, lo = added(age) + 1;   // offsets lo .. hi - 1
      int hi = age + d.W - phi;
      if (hi > d.d_max + 1) hi = d.d_max + 1;
      int s = slot - age;
      if (s < 0) s += R;
      if (lo >= hi) continue;   // uniform
      for (unsigned long long b = L.words[s * wpb + w]; b; b &= b - 1ull) {
        const int i = w * 64 + __ffsll((long long)b) - 1, r0 = (int)d.row_ptr[i];
        const unsigned* const ds = d.dstart + (size_t)i * (d.d_max + 2);
        for (int p = r0 + (int)ds[lo] + lane; p < r0 + (int)ds[hi]; p += 64) {
          const uint2 e = load_stream(&d.synf[p]);
          atomicAdd(&win[(size_t)(phi + (int)(e.x & d.dmask) - age) * d.BN + base + (int)(e.x >> d.dbits)], (int)e.y);
        }
      }
    }
  }
  if (blockIdx.x == 0 && tid == 0 && arrivals) atomicAdd(arrive_bar ? &d.ctr->bar[0] : &d.ctr->rev_arrivals[0][0], arrivals);
  // spikes and the events they emit, into the counters that the window's expansion keeps
  long long c0 = 0, c1 = 0, c2 = 0;
  if (act) {
    d.V[g] = V;
    if (syn) d.J[g] = J;
    if (dexp) d.J[(size_t)d.BN + g] = Jf;
    if (record) d.spk_count[g] += count;
    c0 = before + count - recent((int)(n0 + nsteps - fold_hi)); c1 = c0 * (d.row_ptr[tid + 1] - d.row_ptr[tid]); c2 = c0 * d.rowsum[tid];
  }
  c0 = wave_total64(c0); c1 = wave_total64(c1); c2 = wave_total64(c2);
  if (lane == 0 && c0) {
    BlkCtr& bc = d.blk[blockIdx.x & (kMaxBinBlocks - 1)];
    atomicAdd((unsigned long long*)&bc.pad[0], (unsigned long long)c0);
    atomicAdd(&bc.offered, (unsigned long long)c1);
    atomicAdd((unsigned long long*)&bc.sum_offered, (unsigned long long)c2);
  }
}
