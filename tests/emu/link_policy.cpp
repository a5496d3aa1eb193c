// The rules for kernels that move a payload over the host link themselves
// (runtime.h: which payloads, and with how many work-groups), for a CPU test.
#include "runtime.h"

extern "C" int emu_by_kernels(uint64_t bytes, uint32_t C) { return mk::by_kernels(bytes, C); }
extern "C" int emu_link_grid(int T, int K, int grid) { return mk::link_grid(T, K, grid); }
