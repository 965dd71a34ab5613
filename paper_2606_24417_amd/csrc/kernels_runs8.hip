// Run query kernels of 8-word shards.
#include "query_runs.h"

namespace sbf {

hipError_t launch_query_runs8(const Geometry &g, const uint64_t *words, const SeqArgs &a, const LaunchShape &ls,
                              hipStream_t st) {
  return query_runs_any<8>(g, words, a, ls, st);
}

}  // namespace sbf
