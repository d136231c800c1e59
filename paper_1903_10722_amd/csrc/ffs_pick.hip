// ffs_pick.hip -- instantiations of the kernel templates, one family per
// compilation (FFS_PART), so that the build compiles them side by side.
#include <hip/hip_runtime.h>

#include "ffs_kernels.h"
#include "ffs_lane.h"
#include "ffs_pick.h"

namespace flowshop {

#define FFS_PICK(N, KERNEL)                                                                                  \
    if (m == N)                                                                                             \
        return ptb == 1 ? reinterpret_cast<void*>(&KERNEL<N, uint8_t>) : reinterpret_cast<void*>(&KERNEL<N, uint16_t>);
#define FFS_UP_TO_8(KERNEL) \
    FFS_PICK(2, KERNEL) FFS_PICK(3, KERNEL) FFS_PICK(4, KERNEL) FFS_PICK(5, KERNEL) FFS_PICK(6, KERNEL) FFS_PICK(8, KERNEL)

#if FFS_PART == 0
void* pick_gen(int m, int ptb)
{
    FFS_UP_TO_8(k_generation) FFS_PICK(16, k_generation)
    return nullptr;
}
#elif FFS_PART == 1
void* pick_cand(int m, int ptb)
{
    FFS_UP_TO_8(k_candidates) FFS_PICK(16, k_candidates)
    return nullptr;
}
#elif FFS_PART == 2
void* pick_eval(int m, int ptb)
{
    FFS_UP_TO_8(k_evaluate) FFS_PICK(16, k_evaluate)
    return nullptr;
}
#elif FFS_PART == 3
void* pick_gen_lane(int m, int ptb)
{
    FFS_UP_TO_8(k_generation_lane)
    return nullptr;
}
#elif FFS_PART == 4
void* pick_eval_lane(int m, int ptb)
{
    FFS_UP_TO_8(k_evaluate_lane)
    return nullptr;
}
#elif FFS_PART == 5
void* pick_epoch(int m, int ptb)
{
    FFS_UP_TO_8(k_epoch) FFS_PICK(16, k_epoch)
    return nullptr;
}
#else
void* pick_cand_features(int m, int ptb)
{
    FFS_PICK(8, k_cand_features) FFS_PICK(16, k_cand_features) FFS_PICK(20, k_cand_features)
    FFS_PICK(24, k_cand_features) FFS_PICK(32, k_cand_features)
    return nullptr;
}
#endif

}  // namespace flowshop
