// Packed-row annealing kernels specialised to d = 15, 17.  The
// specialised kernels are split over several translation units so that the
// large unrolled ones compile in parallel.
#include "xzzx_device.h"

namespace xzzx {

AnnealKernel static_rows_kernel_b(int d, bool span)
{
    switch (d) {
    case 15: return span ? k_anneal_rows_span_d<15> : k_anneal_rows_d<15>;
    case 17: return span ? k_anneal_rows_span_d<17> : k_anneal_rows_d<17>;
    default: return nullptr;
    }
}

}  // namespace xzzx
