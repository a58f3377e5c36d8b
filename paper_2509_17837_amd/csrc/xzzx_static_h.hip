// Packed-row annealing kernels specialised to d = 31.  The
// specialised kernels are split over several translation units so that the
// large unrolled ones compile in parallel.
#include "xzzx_device.h"

namespace xzzx {

AnnealKernel static_rows_kernel_h(int d, bool span)
{
    switch (d) {
    case 31: return span ? k_anneal_rows_span_d<31> : k_anneal_rows_d<31>;
    default: return nullptr;
    }
}

}  // namespace xzzx
