// Products of few rows on a kernel of their own (gemm_skinny.hip).
#pragma once
#include "gemm_fast.h"

namespace nt {

// whether the kernel takes this (unbatched) product, and is a faster one for it than tiles without a k split
bool skinny_ok(const FastArgs &a, int alay, int blay);
// estimate of its time (us), to be weighed against a k split of tiles
double skinny_cost(const FastArgs &a);
// into how many parts it splits the reduction (inside a program)
int skinny_parts(const FastArgs &a);
nt_status launch_skinny(const FastArgs &a, bool bf16, hipStream_t s);

}  // namespace nt
