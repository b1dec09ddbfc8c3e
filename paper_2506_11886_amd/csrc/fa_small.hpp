// Small calls of fa_decode in one launch: see fa_small.hip.
#pragma once

#include "fa_decode.hpp"

namespace fa {

// LDS bytes of the one-launch form of a small call, 0 where it does not apply
unsigned small_lds(int dtype, int B, int Hkv, int G, int D, int Dkc, int Dvc, int M, int T, int N, int W);
int launch_small(const DecodeParams& p, int dtype, unsigned lds, hipStream_t st, KernelTimers* tm);

}  // namespace fa
