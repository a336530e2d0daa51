// Ring queue, forward, crowded windows: events pulled by their targets.  Included by ring_window.h and ring_resident_forward.h.
//
// Where a large share of the network spikes in every step, handing events out spike by spike costs an atomic add each (in-window
// events: 27 G/s over the chip) or a trip through a tile of all targets per share of the spikes (role_dense).  The targets' own lists
// are the cheaper way then: for every part of `pull_pt` targets all incoming synapses, sorted by arrival offset, and for every neuron
// the spikes of a window as the bits of one word (k_fwd_chip leaves them).  A synapse of offset D takes the bits of its source's
// word shifted by D, and a block adds its part's events in LDS: no staging, no atomic outside the block but one per cell.
//   far:  role_pull, in the first pass of the window's expansion: all spikes before the window
//   near: fwd_pull_steps, inside k_fwd_chip: spikes of the window itself, a step at a time; the part's synapses with offsets inside
//         a window are held in LDS, those of two steps and more are looked at while the block waits for the grid barrier
// A pass costs its look at every synapse (8 bytes, one LDS read) whatever spikes, hence only from a number of spikes on (pull_at).
// Measured, 10,000 neurons x 1,000 synapses, d_max 200, us per window of 32 steps at 5,000 / 2,000 / 20 spikes per step: by the spikes
// steps 583 / 267 / 67, expansion 276 / 127 / 21; pulled steps 88 / 78 / 92, expansion 91 / 48 / 38 (10,000 steps 269 / 124 / 27.8 ms ->
// 56 / 40 ms, and 27.9: not pulled).  What bounds them then: the grid barrier and the look at up to 10,000 synapses per block and
// step (near), the adds to LDS and 80 MB of lists (far: 2.4 TB/s with nothing to add).

// A synapse in its part's list: x = source << (dbits + lb) | offset << lb | target's place in the part, y = Q8.24 amplitude.
__device__ __forceinline__ int pull_part_of(const Dev& d, const Pull& p, unsigned pk) { return (int)(pk >> d.dbits) / p.pt; }

// Lists, made once: entries per (part, offset), where they begin, the entries (in no particular order within one offset: sums of integers).
__global__ __launch_bounds__(kBlock) void k_pull_count(Dev d, Pull L, unsigned* __restrict__ cnt) {
  for (long long p = (long long)blockIdx.x * kBlock + threadIdx.x; p < d.S; p += (long long)gridDim.x * kBlock) {
    const unsigned pk = d.synf[p].x;
    atomicAdd(&cnt[(size_t)pull_part_of(d, L, pk) * (d.d_max + 2) + (pk & d.dmask)], 1u);
  }
}
// (one block; cnt in, pull_pos out: both [parts][d_max + 2], pull_pos with one more at the end)
__global__ __launch_bounds__(1024) void k_pull_scan(Dev d, Pull L, unsigned* __restrict__ cnt) {
  __shared__ unsigned s_sum[1024];
  const int n = L.parts * (d.d_max + 2), per = (n + 1023) / 1024, lo = per * (int)threadIdx.x, hi = lo + per < n ? lo + per : n;
  unsigned sum = 0;
  for (int x = lo; x < hi; ++x) sum += cnt[x];
  s_sum[threadIdx.x] = sum;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const unsigned v = (int)threadIdx.x >= o ? s_sum[threadIdx.x - o] : 0u;
    __syncthreads();
    s_sum[threadIdx.x] += v;
    __syncthreads();
  }
  unsigned run = s_sum[threadIdx.x] - sum;
  for (int x = lo; x < hi; ++x) { const unsigned c = cnt[x]; L.pos[x] = run; cnt[x] = run; run += c; }
  if (threadIdx.x == 1023) L.pos[n] = s_sum[1023];
}
__global__ __launch_bounds__(kBlock) void k_pull_fill(Dev d, Pull L, unsigned* __restrict__ cur) {
  const int lane = threadIdx.x & 63;
  for (long long i = (long long)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); i < d.N; i += (long long)gridDim.x * (kBlock / 64)) {
    const long long r1 = d.row_ptr[i + 1];
    for (long long p = d.row_ptr[i] + lane; p < r1; p += 64) {
      const uint2 e = d.synf[p];
      const int part = pull_part_of(d, L, e.x);
      const unsigned D = e.x & d.dmask, place = (e.x >> d.dbits) - (unsigned)(part * L.pt);
      const unsigned at = atomicAdd(&cur[(size_t)part * (d.d_max + 2) + D], 1u);
      L.list[at] = make_uint2((unsigned)i << (d.dbits + L.lb) | D << L.lb | place, e.y);
    }
  }
}

__host__ __device__ __forceinline__ unsigned* pull_words(const Dev& d, const Pull& L, long long window) { return L.hist + (size_t)(window & L.hmask) * d.BN; }

// Virtual block x of nvb: (trial, part, share of the offsets) in turn.  lds: a pair of window words per source, a tile [W][pull_pt].
// Spikes of steps from count_from on are counted: count_from >= k0 - W.
__device__ __forceinline__ void role_pull(const Dev& d, const Pull& L, unsigned long long* lds, int* s_count, long long k0, int vb, int nvb, long long count_from) {
  const int N = d.N, W = d.W, nb = d.d_max + 2, shift = d.dbits + L.lb;
  const unsigned lmask = (1u << L.lb) - 1u;
  const unsigned wmask = W < 32 ? (1u << W) - 1u : ~0u;
  unsigned long long* const pair = lds;
  int* const tile = reinterpret_cast<int*>(lds + N);
  const int cells = W * L.pt;
  const long long w0 = k0 >> d.wshift;
  int* __restrict__ win = win_of(d, k0);
  int seen = 0;   // spikes in the words taken in with a trial's first share, by its first part's block
  bool counting = false;
  for (int x = vb; x < d.B * L.parts * L.K; x += nvb) {
    const int part = x % L.parts, rest = x / L.parts, share = rest % L.K, base = rest / L.K * N;
    const int q_lo = 1 + share * L.Q / L.K, q_hi = 1 + (share + 1) * L.Q / L.K;   // windows back from k0
    const unsigned* __restrict__ pos = L.pos + (size_t)part * nb;
    const bool counted = part == 0 && share == 0;
    counting |= counted;
    for (int c = threadIdx.x; c < cells; c += kRingThreads) tile[c] = 0;
    for (int q = q_lo; q < q_hi && w0 - q >= -1; ++q) {
      const unsigned* lo = w0 - q >= 0 ? pull_words(d, L, w0 - q) + base : nullptr;
      const unsigned* hi = q > 1 ? pull_words(d, L, w0 - q + 1) + base : nullptr;
      __syncthreads();   // (the words before are used up)
      for (int i = threadIdx.x; i < N; i += kRingThreads) {
        const unsigned a = lo ? lo[i] : 0u;
        const unsigned long long b = q == q_lo ? (hi ? hi[i] : 0u) : pair[i] & wmask;
        pair[i] = (unsigned long long)a | b << W;
        if (counted) seen += __popc(a);
      }
      __syncthreads();
      const int d1 = q * W < d.d_max ? q * W : d.d_max, top = q * W;
      const unsigned e0 = pos[(q - 1) * W + 1], e1 = pos[d1 + 1];
      for (unsigned e = e0 + threadIdx.x; e < e1; e += 4 * kRingThreads) {
        uint2 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { v[u] = make_uint2(0u, 0u); if (e + u * kRingThreads < e1) v[u] = load_stream(&L.list[e + u * kRingThreads]); }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (e + u * kRingThreads >= e1) break;
          const int D = (int)((v[u].x >> L.lb) & d.dmask);
          unsigned m = (unsigned)(pair[v[u].x >> shift] >> (top - D)) & wmask;
          int* const at = tile + (v[u].x & lmask);
          for (; m; m &= m - 1u) atomicAdd(at + (__ffs((int)m) - 1) * L.pt, (int)v[u].y);
        }
      }
    }
    __syncthreads();
    const int t0 = part * L.pt, have = N - t0 < L.pt ? N - t0 : L.pt;
    for (int c = threadIdx.x; c < cells; c += kRingThreads) {
      const int r = c / L.pt, j = c - r * L.pt, v = tile[c];
      if (v != 0 && j < have) atomicAdd(&win[(size_t)r * d.BN + base + t0 + j], v);
    }
    __syncthreads();
  }
  // which way the next window goes (k_win_acc, which has left `pieces` zero): the windows of the first shares stand for all
  if (counting) {   // uniform
    if (threadIdx.x == 0) *s_count = 0;
    __syncthreads();
    const long long mine = wave_total(seen);
    if ((threadIdx.x & 63) == 0) atomicAdd(s_count, (int)mine);
    __syncthreads();
    const int windows = L.Q / L.K > 0 ? L.Q / L.K : 1;
    if (threadIdx.x == 0 && *s_count) atomicAdd((unsigned long long*)&d.ctr->pieces, (unsigned long long)((long long)*s_count * L.Q / windows));
  }
  // spikes of the window just finished, their events and amplitudes
  long long cnt[3] = {0, 0, 0};
  if (count_from < k0) {
    const unsigned* const last = pull_words(d, L, w0 - 1);
    const int from = (int)(count_from - (k0 - W));
    for (int g = vb * kRingThreads + (int)threadIdx.x; g < d.BN; g += nvb * kRingThreads) {
      const int c = __popc(last[g] >> from);
      if (c) { const int i = g - trial_of(d, g) * N; cnt[0] += c; cnt[1] += c * (d.row_ptr[i + 1] - d.row_ptr[i]); cnt[2] += c * d.rowsum[i]; }
    }
  }
  for (int k = 0; k < 3; ++k) {
    const long long v = wave_total64(cnt[k]);
    if ((threadIdx.x & 63) == 0 && v) {
      BlkCtr& bc = d.blk[vb & (kMaxBinBlocks - 1)];
      atomicAdd(k == 0 ? (unsigned long long*)&bc.pad[0] : k == 1 ? &bc.offered : (unsigned long long*)&bc.sum_offered, (unsigned long long)v);
    }
  }
}
