// The state between the stages of a registration (d2d_it_prep_kernel's last
// block, d2d_it_out_kernel) on the CPU, with both orders of the waves: after
// a stage that had already ended, after one whose last step failed, and after
// one whose last step was taken.
#include "d2d_device.hpp"

using namespace d2d_dev;

static void check(bool ok, const char *what, int ended, bool backwards) {
  if (ok) return;
  printf("%s (ended %d, backwards %d)\n", what, ended, (int)backwards);
  exit(1);
}

int main() {
  constexpr int M = 100;
  static State st;
  static double vrows[2 * kTrials * M], hist[8], T[16];
  for (int ended = 0; ended < 4; ++ended) {   // 0 taken, 1 no step, 2 flag set, 3 no trial better
    for (int back = 0; back < 2; ++back) {
      st = State{};
      Cur &c = st.cur[1];
      for (int e = 0; e < kPose; ++e) c.pose[e] = e;
      c.f = ended == 3 ? 1e9 : -1e9;
      c.stopped = ended == 2;
      c.stage = 0;
      c.hist_n = 3;
      c.count[0] = 2;
      st.trial_stop = ended == 1;
      for (int k = 0; k < kTrials; ++k)
        for (int e = 0; e < kPose; ++e) st.trial[k][e] = 100.0 * (k + 1) + e;
      for (int i = 0; i < kTrials * M; ++i) {
        vrows[2 * i] = 0.0;
        vrows[2 * i + 1] = 1.0;
      }
      const bool took = ended == 0;
      const Mix none{nullptr, nullptr, nullptr, M};
      for (int out = 0; out < 2; ++out) {
        gridDim.x = out ? 1 : 2;
        blockIdx.x = out ? 0 : 1;
        const State before = st;
        int counts[2] = {-1, -1};
        emulate::run_block(kThreads, back != 0, [&] {
          if (out)
            d2d_it_out_kernel(&st, 1, 1, vrows, M, hist, 8, T, counts);
          else
            d2d_it_prep_kernel(MixArgs{}, none, MixArgs{}, none, &st, 1, 1, 1, vrows, hist, 8);
        });
        const double first = took ? 100.0 : 0.0;
        if (out) {
          check(T[0] == first && T[11] == first + 11.0, "pose", ended, back != 0);
          check(counts[0] == (took ? 3 : 2) && counts[1] == 0, "counts", ended, back != 0);
        } else {
          const Cur &n = st.cur[0];
          check(n.stopped == 0 && n.stage == 1, "flags", ended, back != 0);
          check(n.pose[0] == first && n.pose[11] == first + 11.0, "pose", ended, back != 0);
          check(n.count[0] == (took ? 3 : 2) && n.hist_n == (took ? 4 : 3), "counts", ended,
                back != 0);
          if (took) check(fabs(hist[3] - log((double)M)) < 1e-12, "f", ended, back != 0);
        }
        st = before;
      }
    }
  }
  printf("stages ok\n");
  return 0;
}
