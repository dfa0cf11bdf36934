// Operator sweeps on canonical fields: int16 spinors inside.
#include "dslash_op.h"

namespace wd {

hipError_t op_launch_i16(const OpArgs &o, int lk, int dag, dim3 grid, int block, hipStream_t s)
{
    WD_OP_CASE(SP_I16, LK_F32_12)
    WD_OP_CASE(SP_I16, LK_F16_12)
    return hipErrorInvalidValue;
}

}  // namespace wd
