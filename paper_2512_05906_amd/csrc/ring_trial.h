// Ring queue, forward, small networks: a whole run in ONE launch, one workgroup per trial, no synchronisation outside the
// workgroup.  Included by adseq.hip after synapse_resident.h.
//
// Trials do not exchange anything, and where a trial's whole delay line [R][N] fits LDS a spike adds its entries there at once: a
// step needs two block barriers where the kernels over one XCD or the whole chip need a barrier through memory, the cells' trip from
// the L2, the adds' acknowledgement, and the window's expansion besides.  The front of every row is in LDS too, as far as there
// is room; what is behind it is one trip to the L2.  A step is bound by the instructions of the one compute unit (drive hash, update)
// and by its LDS.  Measured, us per forward step, by launches per window / so: 100 neurons x 10 synapses 2.3 / 0.43; 3 trials x 212 x 253
// 3.4 / 0.48; 756 x 95 2.2 / 0.63; 4 x 200 x 1,000 with 3 spikes per step 3.5 / 1.3, with 142 18.7 / 13.3; 100 x 10 with 62 8.5 / 6.6.
// (An earlier form kept a window of eight rows in LDS and added the entries of all held spikes two steps ahead, as k_syn_run does; it
// took 16 x 1,000 neurons, d_max 50, from 2.0 to 1.7 us per step, but with 500 spikes per step and trial from 21 to 71.)
//
// Between launches there is nothing but what the other forward kernels leave, too: circular spike words, the window of the next step,
// counters, barrier arrivals.  A launch rebuilds its cells from the spike words and hands everything back at its end, so any other
// entry point, captured or not, may come before or after it.

constexpr int kTrialNeurons = 1024;
constexpr int kTrialMost = 512;                  // trials: a workgroup fills a compute unit's LDS, so that 256 run at a time, two rounds of 0.5 us per step
// (what every wavefront does costs the compute unit as often as there are wavefronts)
constexpr int trial_threads(int N) { return N <= 128 ? 128 : (N <= 256 ? 256 : 1024); }
constexpr int kTrialLdsWords = 18432;            // 8-byte words of LDS for cells, spike words and fronts
constexpr long long kTrialSynapses = 262144;     // synapses of a trial at most: 2 MB of rows, which the L2 holds
constexpr long long kTrialSteps = 64;            // steps of a call at least: a launch takes in the fronts and rebuilds the cells (100 neurons, in
                                                 // calls of 64 steps 1.7 / 0.63 us per step)

template <int kMost>
struct TrialLds {
  alignas(16) unsigned long long words[kTrialLdsWords];   // spikes [R][wpb]; fronts [near][N]; cells [R][N] by step mod R
  unsigned short spk[kMost];                            // the step's spikes
  int n_spk[2];                                         // spikes of the step, by step parity
};

// Steps n0 .. n0 + nsteps - 1 of trial blockIdx.x; N <= blockDim.x <= kMost, thread t owns neuron t.  near: entries of a row's
// front in LDS.  record: the tape is written; its spike words of these steps are zero when the launch begins.
// Spikes of steps [fold_lo, fold_hi) and the events they emit are counted: fold_lo <= n0, fold_hi the last window boundary of these
// steps (fold_lo if there is none), as where the other kernels stop counting, so that what is listed on top of the last step is still
// counted later.  Both n0 - fold_lo and n0 + nsteps - fold_hi are at most W < R.
// arrivals: what the barriers of these steps would have added to the arrival counter that the host counts along with (arrive_bar: that
// of the kernels over one XCD).
template <int kMost>
__global__ __launch_bounds__(kMost) void k_trial_run(long long n0, int nsteps, int near, int record, long long fold_lo, long long fold_hi,
                                                     unsigned arrivals, int arrive_bar, Dev d) {
  __shared__ TrialLds<kMost> L;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int threads = (int)blockDim.x, waves = threads >> 6;
  const int N = d.N, wpb = (N + 63) >> 6, R = d.R;
  const int base = (int)blockIdx.x * N, g = base + tid;
  const bool act = tid < N;
  const bool syn = d.alpha_s > 0.0f, dexp = d.alpha_r > 0.0f;
  const unsigned long long G64 = 0x9E3779B97F4A7C15ull;
  uint2* const fronts = reinterpret_cast<uint2*>(L.words + (size_t)R * wpb);
  int* const cells = reinterpret_cast<int*>(L.words + (size_t)R * wpb + (size_t)near * N);
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
  for (int x = tid; x < R * N; x += threads) cells[x] = 0;
  if (tid < 2) L.n_spk[tid] = 0;
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
  int slot = (int)(n0 % R);   // row of spike words and cells that belongs to the step
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
        const int r0 = (int)d.row_ptr[i], r1 = (int)d.row_ptr[i + 1];
        for (int q = r0 + (int)d.dstart[(size_t)i * (d.d_max + 2) + age] + lane; q < r1; q += 64) {
          const uint2 e = load_stream(&d.synf[q]);
          int row = slot + (int)(e.x & d.dmask) - age;
          if (row >= R) row -= R;
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
      int* const cell = &cells[slot * N + tid];
      float I = (float)*cell * 0x1p-24f;
      *cell = 0;   // (for step n + R)
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
      if (spike) L.spk[at + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)tid;
      if (record && lane < 2) {
        // the tape's words count from the first trial's first neuron
        const int gw = base + wave * 64, sh = gw & 63;
        const unsigned long long part = lane == 0 ? m << sh : (sh ? m >> (64 - sh) : 0ull);
        if (part) atomicOr(&d.tape_bits[(size_t)n * d.words + (gw >> 6) + lane], part);
      }
    }
    __syncthreads();   // spikes known, cells of the step taken
    const int nspk = L.n_spk[par];
    if (tid == 0) L.n_spk[par ^ 1] = 0;   // (the last step's has been read)
    auto add = [&](const uint2& e) {
      int row = slot + (int)(e.x & d.dmask);
      if (row >= R) row -= R;
      atomicAdd(&cells[row * N + (int)(e.x >> d.dbits)], (int)e.y);
    };
    for (int x = wave; x < nspk; x += waves) {
      const int i = L.spk[x];   // (the same in every lane)
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
    int s = slot + r - phi;
    if (s >= R) s -= R;
    if (phi) win[(size_t)r * d.BN + base + i] = r >= phi ? cells[s * N + i] : 0;
    if (first != win || !phi) first[(size_t)r * d.BN + base + i] = 0;
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
