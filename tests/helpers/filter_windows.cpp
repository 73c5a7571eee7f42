// The windows that a batch, server or SIR record gets, for the tests: compiled
// for the host from the library's own header.
#include "mgp_batch_internal.h"

// out: address of position 0 for windows inside the weights, and for those at or
// past their end; 1 if windows run on past n, 0 if they wrap; floats of the region.
extern "C" void filter_windows(uint64_t w, uint64_t aux, uint32_t n, uint32_t B, int in_place, uint64_t* out)
{
    mgp::FilterDev F{};
    F.w = reinterpret_cast<const float*>(w);
    F.n = n;
    F.B_user = B;
    F.set_windows(in_place != 0, reinterpret_cast<float*>(aux));
    out[0] = F.windows.w;
    out[1] = F.windows.seam;
    out[2] = F.tail != nullptr;
    out[3] = mgp::window_floats(in_place != 0, n, B);
}
