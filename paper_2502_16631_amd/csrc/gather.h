// Gather of DATA chunks to their payload records (gfx950): the last pass of
// the three-pass delta dump and of the codec dump, after the payload offsets
// are known.
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace mk {

struct GatherJob {
    const AllocDesc* allocs;
    const uint32_t* amap;    // allocation of chunk g (required)
    uint32_t C;
    uint32_t pad;
    const uint64_t* off;     // payload offset of chunk g
    uint8_t* slot;           // payload buffer, from offset 0 on
    const uint64_t* list;    // the DATA chunks in order
    const uint64_t* n_list;  // their number
    uint64_t* stamp;         // device clock at the kernel's start, or nullptr
};

// DATA chunks in 16-byte blocks, a last partial block byte by byte and
// zero-padded to 16 bytes. Work-groups take parts of kGatherPart bytes of the
// listed chunks.
constexpr uint32_t kGatherPart = 16384;
hipError_t launch_gather(const GatherJob& j, int grid, hipStream_t s);

}  // namespace mk
