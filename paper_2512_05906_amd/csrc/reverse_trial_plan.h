// Which reverse sweeps go by k_bwd_trial (ring_trial_reverse.h), and how: sizes, LDS, pieces.  Host code only.
#ifndef ADSEQ_REVERSE_TRIAL_PLAN_H
#define ADSEQ_REVERSE_TRIAL_PLAN_H

constexpr int kRevTrialLds = 160000;     // bytes
constexpr int kRevTrialItems = 384;      // listed pieces of a step
constexpr int kRevTrialWords = 128;      // spike words of a step at most: two per lane of the loading wavefront
constexpr int kRevTrialPieces = 16;      // P at most
constexpr int kRevTrialNeurons = 1024;   // two per worker thread, 16 per lane of the wavefront that loads the rows
constexpr int kRevTrialMost = 512;       // trials

// LDS of a workgroup: bytes besides the adjoint rows.
inline long long rev_trial_fixed(int N, int P) {
  const long long words = (long long)P * ((N + 63) / 64 + 1);
  return (2LL * kRevTrialItems * 16) + 2 * words * 8 + 2 * words * 4 + 4LL * (N + 1) + 4LL * N + 16LL * ((N + 63) & ~63) + 4LL * (P + 1) * N + 64;
}

// H adjoint rows that fit, P pieces of a row (0: the sweep goes by the other kernels).  Positions in the rows are 32 bits there.
struct RevTrialPlan { int H, P; };
inline RevTrialPlan rev_trial_plan(int N, int B, long long S, int d_max) {
  if (N > kRevTrialNeurons || B > kRevTrialMost || S > 0x7fffffffLL) return {0, 0};
  for (int P = 1; P <= kRevTrialPieces; ++P) {
    long long H = (kRevTrialLds - rev_trial_fixed(N, P)) / (4LL * N);
    if (H > d_max) H = d_max;
    if (H * P >= d_max && (P == 1 || H >= 16) && P * ((N + 63) / 64 + 1) <= kRevTrialWords) return {(int)H, P};
  }
  return {0, 0};
}

// The line on a run's spikes (see ring_trial_reverse.h): what one weighs, and how much of it a step of all trials may have.
inline double rev_trial_weight(long long S, int N, int P, bool adm) { return (1.5 * P - 0.5 + (double)S / N / 64.0) * (adm ? 2.0 : 1.0); }
inline double rev_trial_load(int N, int B, int P, bool adm) { return 7.0 * (N <= 256 && P == 1 ? 8.0 : (B == 1 && !adm ? 4.0 : 1.0)); }

#endif
