// Operator sweeps on canonical fields: FP64.
#include "dslash_op.h"

namespace wd {

hipError_t op_launch_f64(const OpArgs &o, int lk, int dag, dim3 grid, int block, hipStream_t s)
{
    WD_OP_CASE(SP_F64, LK_F64_18)
    WD_OP_CASE(SP_F64, LK_F64_18N)
    WD_OP_CASE(SP_F64, LK_F64_12)
    WD_OP_CASE(SP_F64, LK_F64_12N)
    return hipErrorInvalidValue;
}

}  // namespace wd
