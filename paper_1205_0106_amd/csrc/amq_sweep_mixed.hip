// amq_sweep_mixed.hip — batch sweep kernels for options of both storage types
// in one launch, monomial basis, the default tiles.
#include "amq_sweep.h"

namespace amq {

const void *sweep_table_mixed(int degree)
{
    switch (degree) {
    case 0: return (const void *)&sweep_mixed_kernel<64, 32, 0>;
    case 1: return (const void *)&sweep_mixed_kernel<64, 32, 1>;
    case 2: return (const void *)&sweep_mixed_kernel<64, 32, 2>;
    case 3: return (const void *)&sweep_mixed_kernel<64, 32, 3>;
    case 4: return (const void *)&sweep_mixed_kernel<64, 32, 4>;
    case 5: return (const void *)&sweep_mixed_kernel<64, 32, 5>;
    case 6: return (const void *)&sweep_mixed_kernel<64, 32, 6>;
    default: return nullptr;
    }
}

}  // namespace amq
