// Packed-row annealing kernels specialised to d = 29.  The
// specialised kernels are split over several translation units so that the
// large unrolled ones compile in parallel.
#include "xzzx_device.h"

namespace xzzx {

AnnealKernel static_rows_kernel_g(int d, bool span)
{
    switch (d) {
    case 29: return span ? k_anneal_rows_span_d<29> : k_anneal_rows_d<29>;
    default: return nullptr;
    }
}

}  // namespace xzzx
