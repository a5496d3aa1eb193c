// The piece plan of delta and codec dumps (runtime.h plan_pieces), for a CPU
// test: the pieces' first chunks to out, their number returned.
#include "runtime.h"

extern "C" uint64_t emu_plan_pieces(uint64_t nc, uint32_t C, uint64_t budget, int ring, int codec, uint64_t round,
                                    uint64_t* out, uint64_t cap) {
    const std::vector<uint64_t> p = mk::plan_pieces(nc, C, budget, ring != 0, codec != 0, round);
    for (uint64_t i = 0; i < p.size() && i < cap; ++i) out[i] = p[i];
    return p.size();
}
