// Instantiations of the chained cross-attention kernel on 16x16x32 MFMAs: one joint softmax, and one softmax for each of
// two conditioning sequences (head_dim 128, fp16 operands, 16-bit output rows).
#include "dit_attn_fwd_pipe16.h"

namespace dit {

namespace {

template <int D, int QK_OP, int PV_OP, bool TWO>
hipError_t launch_form(const AttnArgs& a, const ChainLayout& c, hipStream_t s) {
    if constexpr (!TWO) {
        if (c.rows == 16)
            return c.nw == 8 ? launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, false, 1>(a, c.qch, s)
                             : launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 4, false, 1>(a, c.qch, s);
    }
    if (c.nw != 8) return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 4, TWO>(a, c.qch, s);
    if constexpr (D == 128) {
        if (a.out_once) return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, TWO, 2, true>(a, c.qch, s);
    }
    return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, TWO>(a, c.qch, s);
}

}  // namespace

hipError_t launch_attn_pipe16_chain(const AttnArgs& a, int D, int qk_op, int pv_op, const ChainLayout& c,
                                    hipStream_t s) {
#define DIT_CASE(TWO, DD, QK, PV)                                                                 \
    if ((a.tile_count_a != nullptr) == TWO && D == DD && qk_op == QK && pv_op == PV)               \
        return launch_form<DD, QK, PV, TWO>(a, c, s);
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
