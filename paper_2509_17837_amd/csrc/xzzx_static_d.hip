// Packed-row annealing kernels specialised to d = 23.  The
// specialised kernels are split over several translation units so that the
// large unrolled ones compile in parallel.
#include "xzzx_device.h"

namespace xzzx {

AnnealKernel static_rows_kernel_d(int d, bool span)
{
    switch (d) {
    case 23: return span ? k_anneal_rows_span_d<23> : k_anneal_rows_d<23>;
    default: return nullptr;
    }
}

}  // namespace xzzx
