// The autotuner's range of workgroups per CU: the resident workgroups of the
// kernel that the chosen plan runs, whatever plan was timed last.  Host only;
// prints "ok" or the first case that differs.
#include <cstdio>
#include <cstring>

#include "pmbs_internal.h"

int main() {
  pmbs_sim sim;
  std::memset(&sim.cfg, 0, sizeof sim.cfg);
  std::memset(&sim.plan, 0, sizeof sim.plan);
  // 128, 256, 512 contacts, up to 16 boxes and up to 31
  const int occ[6][2] = {{12, 6}, {7, 4}, {3, 0}, {8, 5}, {9, 2}, {1, 0}};
  std::memcpy(sim.occ, occ, sizeof occ);
  for (int mc : {128, 256, 512})
    for (int last : {-1, 12, 16, 24, 31})
      for (int chosen : {-1, 12, 16, 24, 31})
        for (int nb : {5, 16, 17, 30})
          for (int waves : {1, 2}) {
            sim.cfg.max_contacts = mc;
            sim.plan.small_max_bodies = last;
            sim.plan.small_waves = sim.plan.large_waves = 3 - waves;
            sim.max_nb = nb;
            pmbs_launch_plan win = sim.plan;
            win.small_max_bodies = chosen;
            win.small_waves = win.large_waves = waves;
            const int split = mc == 128 ? 31 : chosen;
            const int small = (split < nb ? split : nb) > 16 ? 3 : 0, large = nb > 16 ? 4 : 1;
            if (pmbs::resident_blocks(&sim, win, 128) != occ[small][waves - 1] ||
                pmbs::resident_blocks(&sim, win, 256) != occ[large][waves - 1]) {
              std::printf("contacts %d, last %d, chosen %d, boxes %d, waves %d\n", mc, last, chosen, nb, waves);
              return 1;
            }
          }
  std::printf("ok\n");
  return 0;
}
