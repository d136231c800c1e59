// ffs_pinned.h -- pinned host blocks that small results pass through.
//
// A copy into pageable memory waits inside the runtime and again at the
// caller's synchronisation; into a pinned block it is one asynchronous copy
// and one wait.  A context takes a block when it is created and gives it back
// when it is destroyed, after its stream has drained; up to kPinKept blocks
// stay allocated between contexts (allocating one takes longer than binding a
// small context), the rest are freed.
#pragma once
#include <stddef.h>

namespace flowshop {

constexpr size_t kPinWords = 256;             // bytes of words that kernels write
constexpr size_t kPinStage = (size_t)64 << 10;   // staging bytes after them
constexpr size_t kPinKept = 16;

char* pin_take();          // null if the allocation fails
void pin_give(char* p);

}  // namespace flowshop
