// Instantiates the batched filter's kernels for one conductance, chosen at
// compile time by IG_COND (0..2).  The build compiles this file once per
// conductance.
#include "batch_kernels.h"

#ifndef IG_COND
#error "IG_COND must be defined"
#endif

namespace igk {

#define IG_CAT2(a, b) a##b
#define IG_CAT(a, b) IG_CAT2(a, b)

const BatchKernels* IG_CAT(batch_kernels_c, IG_COND)() {
    static const BatchKernels table = {
        k_batch_resident<IG_COND>,
        {k_batch_round<IG_COND, 1>, k_batch_round<IG_COND, 2>, k_batch_round<IG_COND, 3>, k_batch_round<IG_COND, 4>},
        {k_batch_persist<IG_COND, 1>, k_batch_persist<IG_COND, 2>, k_batch_persist<IG_COND, 3>,
         k_batch_persist<IG_COND, 4>}};
    return &table;
}

}  // namespace igk
