// Instantiations of the chained cross-attention kernel on 16x16x32 MFMAs: one joint softmax, and one softmax for each of
// two conditioning sequences (head_dim 128, fp16 operands, 16-bit output rows).
#include "dit_attn_fwd_pipe16.h"

namespace dit {

hipError_t launch_attn_pipe16_chain(const AttnArgs& a, int D, int qk_op, int pv_op, int nw, int qch, hipStream_t s) {
#define DIT_CASE(TWO, DD, QK, PV)                                                                 \
    if ((a.tile_count_a != nullptr) == TWO && D == DD && qk_op == QK && pv_op == PV)               \
        return nw == 8 ? launch_attn_pipe16_chain_inst<DD, QK, PV, 8, TWO>(a, qch, s)              \
                       : launch_attn_pipe16_chain_inst<DD, QK, PV, 4, TWO>(a, qch, s);
    DIT_CASE(false, 128, OP_F16, OP_F16)
    DIT_CASE(false, 128, OP_F16, OP_BF16)
    DIT_CASE(false, 128, OP_BF16, OP_F16)
    DIT_CASE(false, 128, OP_BF16, OP_BF16)
    DIT_CASE(false, 64, OP_F16, OP_F16)
    DIT_CASE(false, 64, OP_F16, OP_BF16)
    DIT_CASE(false, 64, OP_BF16, OP_F16)
    DIT_CASE(false, 64, OP_BF16, OP_BF16)
    DIT_CASE(true, 128, OP_F16, OP_F16)
#undef DIT_CASE
    return hipErrorInvalidValue;
}

}  // namespace dit
