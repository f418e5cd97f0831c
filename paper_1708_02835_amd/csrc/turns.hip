// The one-launch factorisation (flow.hpp) with workgroups that leave, for long launches.
#define FLOW_LEAVE true
#include "flow.hpp"

namespace gl {

int flow_launch_turns(Work &w, hipStream_t s, bool solve) { return flow_launch(w, s, solve); }

void flow_launch_batched_turns(int b, const BatchReq *d, int count, int64_t blocks, int64_t pads, hipStream_t s)
{
    flow_launch_batched(b, d, count, blocks, pads, s);
}

void flow_launch_rhs_turns(const Work &w, double *st, int groups, int *words, double *part, hipStream_t s)
{
    flow_launch_rhs(w, st, groups, words, part, s);
}

}  // namespace gl
