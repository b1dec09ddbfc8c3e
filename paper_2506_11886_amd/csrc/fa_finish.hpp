// Last launch of fa_decode: see fa_finish.hip.
#pragma once

#include "fa_decode.hpp"

namespace fa {

int launch_finish(const DecodeParams& p, hipStream_t st, KernelTimers* tm);

}  // namespace fa
