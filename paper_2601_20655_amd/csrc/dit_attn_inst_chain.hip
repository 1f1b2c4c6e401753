// Instantiations of the chained cross-attention kernel on 16x16x32 MFMAs: one joint softmax, and one softmax for each of
// two conditioning sequences (head_dim 128, fp16 operands, 16-bit output rows).
#include "dit_attn_fwd_pipe16.h"

namespace dit {

namespace {

template <int D, int QK_OP, int PV_OP, bool TWO>
hipError_t launch_form(const AttnArgs& a, int nw, int qch, hipStream_t s) {
    if (nw == 8) {
        if constexpr (D == 128) {
            if (a.out_once) return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, TWO, 2, true>(a, qch, s);
        }
        return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, TWO>(a, qch, s);
    }
    if constexpr (!TWO) {
        if (qch == 1) {  // all query tiles in one round: one query block a wavefront (short_tile_rows)
            const int rows = short_tile_rows((int64_t)a.B * a.H, a.Lq);
            AttnArgs b = a;
            b.nQT = (a.Lq + rows - 1) / rows;
            if ((int64_t)b.nQT * a.B * a.H <= kCUs)
                return rows == 64 ? launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 4, false, 1>(b, 1, s)
                                  : launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 8, false, 1>(b, 1, s);
        }
    }
    return launch_attn_pipe16_chain_inst<D, QK_OP, PV_OP, 4, TWO>(a, qch, s);
}

}  // namespace

hipError_t launch_attn_pipe16_chain(const AttnArgs& a, int D, int qk_op, int pv_op, int nw, int qch, hipStream_t s) {
#define DIT_CASE(TWO, DD, QK, PV)                                                                 \
    if ((a.tile_count_a != nullptr) == TWO && D == DD && qk_op == QK && pv_op == PV)               \
        return launch_form<DD, QK, PV, TWO>(a, nw, qch, s);
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
