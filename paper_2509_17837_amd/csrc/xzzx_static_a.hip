// Packed-row annealing kernels specialised to d = 3, 5, 7, 9, 11, 13.  The
// specialised kernels are split over several translation units so that the
// large unrolled ones compile in parallel.
#include "xzzx_device.h"

namespace xzzx {

AnnealKernel static_rows_kernel_a(int d, bool span)
{
    switch (d) {
    case 3: return span ? k_anneal_rows_span_d<3> : k_anneal_rows_d<3>;
    case 5: return span ? k_anneal_rows_span_d<5> : k_anneal_rows_d<5>;
    case 7: return span ? k_anneal_rows_span_d<7> : k_anneal_rows_d<7>;
    case 9: return span ? k_anneal_rows_span_d<9> : k_anneal_rows_d<9>;
    case 11: return span ? k_anneal_rows_span_d<11> : k_anneal_rows_d<11>;
    case 13: return span ? k_anneal_rows_span_d<13> : k_anneal_rows_d<13>;
    default: return nullptr;
    }
}

}  // namespace xzzx
