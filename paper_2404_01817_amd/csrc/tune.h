// tune.h -- the forward autotuner's table (defined in api.hip): the variant
// measured fastest per bucket of (N_max, C_max, B, input mode), for calls
// that ask for NEAT_FWD_TUNED, the batched path and the server.
#pragma once

#include <cstddef>

#include "launch.h"
#include "neat.h"

namespace neat {

// What the autotuner times, in the order of its reported times.
constexpr int TUNE_CANDIDATES[NEAT_TUNE_CANDIDATES] = {FWD_REG, FWD_REG2, FWD_LDS, FWD_LVL,
                                                       FWD_SEG};
// The mapping that FWD_AUTO takes for the job alone, or (throughput) for
// copies of it launched in order; -1 when a candidate launches the same (it is
// timed beside them otherwise, so that tuning never records less than a call
// that is not tuned gets).
int tune_auto(const FwdJob &job, int copies, bool throughput, size_t max_lds);

// The variant recorded for the bucket of (N, C, B, grid): the fastest for a
// call alone, or (throughput) the one with the most genome-inputs per
// second on a full GPU; FWD_AUTO when none is recorded, or when the automatic
// choice itself was fastest.
int tuned_variant(int N, int C, int B, int grid, int throughput);
// Changes whenever a recorded variant changes (plans built from the table
// compare it to know they are stale).
unsigned tune_generation();
// Read the tune cache file at path into the table and keep writing the
// table there after every tuning (nothing happens for a NULL or empty path).
int tune_cache_use(const char *path);

}  // namespace neat
