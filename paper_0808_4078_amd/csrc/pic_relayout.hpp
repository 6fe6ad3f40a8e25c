// Who ends the second phase of a re-layout, and who ends the step, among the
// workgroups of one launch, whose order the device does not promise.
#pragma once

namespace pic {

// Workgroup bid of the nb that carry the phase.  Wg gives one workgroup's
//   rebin()    whether the step has a re-layout (read by each wave)
//   copy(bid, nb)  its part of the copies
//   arrive(nb) after all its waves; true in the last of nb workgroups
//   finish()   the new bins take effect
//   advance()  the end of the step, which clears rebin()
// ADV: the end of the step is part of the launch: workgroup 0's in a step
// without a re-layout, else the last one's to arrive.  Workgroup 0 takes a part
// of the copies too: so all of the nb have read rebin() before it is cleared.
template <bool ADV, class Wg>
__device__ __forceinline__ void relayout_end(Wg &wg, int bid, int nb)
{
    if (!wg.rebin()) {
        if (ADV && bid == 0) wg.advance();
        return;
    }
    wg.copy(bid, nb);
    if (!wg.arrive(nb)) return;
    wg.finish();
    if (ADV) wg.advance();
}

}  // namespace pic
