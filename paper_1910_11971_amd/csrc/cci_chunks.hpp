// Division of a reduction into 64-column chunks between the teams of a
// tap-chunk workgroup (host and device).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cci {

// Chunks of each of `teams` teams (all run the same number: the last team's
// last ones may lie past the reduction's nch).
__host__ __device__ inline int32_t team_chunks(int32_t nch, int32_t teams) { return (nch + teams - 1) / teams; }

// Chunk whose packed columns a load for chunk `ch` addresses.  The lanes of a
// chunk past the reduction are out of range by their own offsets; the chunk's
// uniform offset stays inside the packed arrays all the same, because a range
// check may subtract it from the array's size (with one packed row the size is
// less than an empty chunk's offset).
__host__ __device__ inline int32_t load_chunk(int32_t ch, int32_t nch) { return ch < nch ? ch : nch - 1; }

}  // namespace cci
