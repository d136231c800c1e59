// ffs_pick.h -- the instantiated kernels (ffs_pick.hip) by machine-count bound
// and processing-time width (1 or 2 bytes); null where there is none.
#pragma once

namespace flowshop {

void* pick_gen(int mmax, int ptb);            // k_generation, mmax 2, 3, 4, 5, 6, 8, 16
void* pick_epoch(int mmax, int ptb);          // k_epoch, the same
void* pick_cand(int mmax, int ptb);           // k_candidates, the same
void* pick_eval(int mmax, int ptb);           // k_evaluate, the same
void* pick_gen_lane(int mmax, int ptb);       // k_generation_lane, up to 8
void* pick_eval_lane(int mmax, int ptb);      // k_evaluate_lane, up to 8
void* pick_cand_features(int sm, int ptb);    // k_cand_features, stage tiers 8, 16, 20, 24, 32

}  // namespace flowshop
