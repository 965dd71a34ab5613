// Run query kernels of 16-word shards.
#include "query_runs.h"

namespace sbf {

hipError_t launch_query_runs16(const Geometry &g, const uint64_t *words, const SeqArgs &a, const LaunchShape &ls,
                              hipStream_t st) {
  return query_runs_any<16>(g, words, a, ls, st);
}

}  // namespace sbf
