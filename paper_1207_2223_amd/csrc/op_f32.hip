// Operator sweeps on canonical fields: FP32 spinors inside.
#include "dslash_op.h"

namespace wd {

hipError_t op_launch_f32(const OpArgs &o, int lk, int dag, dim3 grid, int block, hipStream_t s)
{
    WD_OP_CASE(SP_F32, LK_F32_12)
    WD_OP_CASE(SP_F32, LK_F32_12N)
    WD_OP_CASE(SP_F32, LK_F32_18)
    WD_OP_CASE(SP_F32, LK_F32_8)
    WD_OP_CASE(SP_F32, LK_F32_8N)
    WD_OP_CASE(SP_F32, LK_F16_12)
    return hipErrorInvalidValue;
}

}  // namespace wd
