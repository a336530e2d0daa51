// Which closed-loop runs of FIFO and SORTED give every block of k_queue_run a whole trial (queue_resident.h): sizes.  Host code only.
#ifndef ADSEQ_QUEUE_TRIAL_PLAN_H
#define ADSEQ_QUEUE_TRIAL_PLAN_H

// Up to 4,096 neurons, where there are so many trials, or neurons so few, that a trial's events are not the sooner done by several compute units.
// us per step by blocks over the whole chip / so, at 0.1 / 1 / 5 / 20 spikes per step and trial:
//   FIFO[4]: 100 x 10, one trial 2.3 4.4 6.7 10.4 / 1.7 3.8 6.2 10.1; 300 x 100, 4 trials 3.3 5.9 8.4 23.6 / 2.5 4.9 8.3 21.2, one 2.7 4.7 7.1 19.4 / 2.6 4.7 7.5 20.6;
//   500 x 50, 64 trials 4.9 6.7 8.2 12.8 / 2.4 4.6 6.7 9.9, 16 4.0 6.0 7.2 10.9 / 2.6 4.8 7.3 10.2; 1,000 x 100, 64 trials 5.1 7.3 9.7 13.8 / 3.5 6.1 9.6 19.4
// and at 0.2 / 2 / 10 / 40 / 100:
//   FIFO[4]: 1,000 x 100, 192 trials 7.9 11.6 20.7 83 384 / 4.3 8.0 14.2 42 88, 256 8.5 13.0 24.8 105 500 / 4.5 8.4 14.9 42 95; 2,000 x 100, 192 8.5 12.7 23.0 61 278 / 5.8 10.0 17.1 38 96;
//   4,096 x 256, 256 (0.5, 5, 20, 60) 18.4 41.6 103 338 / 12.9 26.5 62 205;  SORTED[64]: 1,000 x 100, 192 8.9 15.3 63 260 596 / 4.5 10.7 47 199 337; 2,000 x 100, 192 9.4 14.6 44
//   245 529 / 5.8 11.0 37 211 497;  512 x 100, 32 trials 6.6 13.9 84 151 - / 3.6 11.6 59 162 - (the one point on this side of the line that is slower)
// More trials than run at a time (a compute unit holds one, two up to 512 neurons) are rounds as long as the slowest trial's, so that the last one has to
// be nearly full.  At 0.3 / 5 / 40 spikes: 1,000 x 60, FIFO[4], 257 trials 9.1 14.3 44 / 8.0 18.5 47, 300 9.5 15.5 52 / 9.3 18.8 49, 512 10.5 19.8 85 / 9.9 19.5 56, 700 15.0 32.2 113 /
// 14.2 29.1 80; 2,000 x 60, 257 9.8 15.9 52 / 10.8 22.1 54, 500 15.4 31.4 99 / 13.8 25.4 62; with eight neurons per thread not even then: 2,500 x 100, 400 trials (0.5, 5) 16.9 33.5 / 19.5
// 36.9; and where two trials share a compute unit not with a second round: 512 x 60, 300 9.0 14.0 90 / 7.1 15.3 42, 512 9.7 17.3 131 / 7.7 15.4 44, 1,000 11.3 26.3 244 / 13.2 28.6 85.
inline bool queue_trials_pay(int N, int B) {
  const int least = N <= 128 ? 1 : (N <= 320 ? 4 : (N <= 512 ? 32 : 192));   // trials
  if (B < least) return false;
  if (B <= 256) return true;
  const int per = N <= 512 ? 512 : 256, rounds = (B + per - 1) / per;
  return 8LL * B >= 7LL * rounds * per && (N <= 512 ? rounds == 1 : N <= 2048 && rounds <= 3);
}
// Steps of a launch at least: a block takes the states of its whole trial in and out, and the spike list is a launch more.  us per step in calls of 4 / 8 / 16
// steps (whose last one goes by itself), FIFO[8]: 512 x 100, 32 trials, 0.3 spikes 11.6 8.6 7.0 / 11.9 7.8 5.8; 1,000 x 100, 256 trials 15.9 12.3 10.5 / 17.6 11.6 8.1; 2,000 x 100, 192
// trials 17.5 13.2 11.0 / 21.9 14.4 10.2, 5 spikes 27.7 22.0 19.1 / 33.1 23.2 17.9; 4,096 x 100, 192 trials, 5 spikes 37.9 29.9 25.9 / 49.6 34.7 26.7.
inline int queue_trial_steps(int N) { return N <= 1024 ? 7 : 20; }

#endif
