// Run query kernels of 4-word shards.
#include "query_runs.h"

namespace sbf {

hipError_t launch_query_runs4(const Geometry &g, const uint64_t *words, const SeqArgs &a, const LaunchShape &ls,
                              hipStream_t st) {
  return query_runs_any<4>(g, words, a, ls, st);
}

}  // namespace sbf
