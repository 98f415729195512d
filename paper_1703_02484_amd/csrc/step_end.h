// End of a queued step, run by one workgroup: as a launch of its own or at the end of the step's last kernel.
#pragma once

#include "bd_internal.h"

namespace bd {

// Records the step's control block in the ring, then either advances the step counter and the stamp bases and
// clears the control block for the next step (a list rebuild this step's skin test asked for happens there), or
// stops the batch when the step halted (the host finishes it, from the control block as it stands) or the ring is
// full.  now: the control block as the step left it (ctl itself, or the workgroup's copy of it in LDS).  Every
// thread of the workgroup calls it, after a barrier; the stop flag is written only after the barrier inside.
__device__ __forceinline__ void step_end_body(const int *now, int *ctl, StepBase *base, int *ring, int r_used,
                                              int v_used) {
    if (base->stop) return;
    const int idx = base->batch_idx;
    const int halt = now[K_HALT];
    __syncthreads();   // every thread has read it
    for (int i = threadIdx.x; i < N_CTL; i += blockDim.x) {
        const int c = now[i];
        ring[(size_t)idx * N_CTL + i] = c;
        ctl[i] = halt ? c : 0;
    }
    if (threadIdx.x != 0) return;
    if (halt) {
        base->stop = 1;
        base->nl_now = 0;   // the steps queued after it rebuild no lists
        return;
    }
    base->step += 1;
    base->rbase += r_used;
    base->vbase += v_used;
    base->batch_idx = idx + 1;
    base->nl_now = base->nl_req;
    base->nl_req = 0;
    if (idx + 1 >= kRing) base->stop = 2;
}

}  // namespace bd
