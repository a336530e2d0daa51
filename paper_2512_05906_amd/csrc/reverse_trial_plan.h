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

// The line on a run's spikes (see ring_trial_reverse.h): what one weighs, and how much of it a step of all trials may have.  us per reverse
// step by the kernels over the whole chip / by k_bwd_trial:
//   more than 256 trials are a second round of workgroups, as long as the first: 512 x 128 x 100, 2 spikes 3.16 / 4.08 (FIFO 3.77 / 5.50),
//     512 x 256 x 100 3.10 / 4.08, 512 x 600 x 100, 1 spike 3.39 / 3.73 -- with rows of 10 entries as often the other way (512 x 64 x 10, FIFO 5.32 / 4.26)
//   up to 256 neurons in one piece the line is eight times as high: 128 x 100, 16 trials, 16 spikes 6.99 / 4.88; from 129 on five times: 256 x 100, 8 trials,
//     8 spikes 3.29 / 2.96, 16 4.33 / 4.34
//   bounded kinds, up to 256 neurons, single trials: 128 x 10, 7.3 spikes 2.93 / 2.83, 16 3.70 / 4.14
//   bounded kinds, rows of more than 64 entries, whose rest is a trip more: 128 x 100, one trial, 3.6 spikes 2.66 / 3.01, 2 trials 4 3.12 / 3.04, 8 3.82 / 3.92, 4
//     trials 8 4.22 / 3.94; 256 x 100, 1 to 16 trials, 1 spike 2.35 / 2.17, 4 2.93 / 3.03, 64 trials 4 3.24 / 3.17, 8 3.87 / 4.11
inline double rev_trial_weight(long long S, int N, int P, bool adm) { return (1.5 * P - 0.5 + (double)S / N / 64.0) * (adm ? 2.0 : 1.0); }
inline double rev_trial_load(long long S, int N, int B, int P, bool adm) {
  if (B > 256) return 0.0;
  if (N > 256 || P > 1) return 7.0 * (B == 1 && !adm ? 4.0 : 1.0);
  if (!adm) return 7.0 * (N <= 128 ? 8.0 : 5.0);
  if (S <= 64LL * N) return 7.0 * (B == 1 ? 2.5 : 8.0);
  return 7.0 * (N <= 128 ? (B == 1 ? 1.0 : (B < 4 ? 4.0 : 8.0)) : (B < 64 ? 1.0 : 4.0));
}

#endif
