// Instantiations of the pipelined self-attention kernel on 16x16x32 MFMAs: one sequence per batch entry and
// packed requests.
#include "dit_attn_fwd_pipe16.h"

namespace dit {

#define DIT_PIPE16_CASES(X) \
    X(128, OP_F16, OP_F16)   \
    X(128, OP_F16, OP_BF16)  \
    X(128, OP_BF16, OP_F16)  \
    X(128, OP_BF16, OP_BF16) \
    X(64, OP_F16, OP_F16)    \
    X(64, OP_F16, OP_BF16)   \
    X(64, OP_BF16, OP_F16)   \
    X(64, OP_BF16, OP_BF16)

hipError_t launch_attn_pipe16(const AttnArgs& a, int D, int qk_op, int pv_op, int nw, hipStream_t s) {
    const int rows = nw == 8 ? 256 : short_tile_rows((int64_t)a.B * a.H, a.Lq);
    AttnArgs b = a;
    b.nQT = (a.Lq + rows - 1) / rows;
    const bool one = nw == 4 && (int64_t)b.nQT * a.B * a.H <= kCUs;  // one query block a wavefront
#define DIT_CASE(DD, QK, PV)                                              \
    if (D == DD && qk_op == QK && pv_op == PV)                             \
        return nw == 8     ? launch_attn_pipe16_inst<DD, QK, PV, 8, 2>(b, s) \
               : !one      ? launch_attn_pipe16_inst<DD, QK, PV, 4, 2>(b, s) \
               : rows == 64 ? launch_attn_pipe16_inst<DD, QK, PV, 4, 1>(b, s) \
                           : launch_attn_pipe16_inst<DD, QK, PV, 8, 1>(b, s);
    DIT_PIPE16_CASES(DIT_CASE)
#undef DIT_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_attn_pipe16_split(const AttnArgs& a, int D, int qk_op, int pv_op, hipStream_t s) {
#define DIT_CASE(DD, QK, PV) \
    if (D == DD && qk_op == QK && pv_op == PV) return launch_attn_pipe16_split_inst<DD, QK, PV>(a, s);
    DIT_PIPE16_CASES(DIT_CASE)
#undef DIT_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_attn_pipe16_varlen(const AttnArgs& a, const VarlenTable& vt, int D, int qk_op, int pv_op, int nw,
                                     hipStream_t s) {
    int64_t tiles = 0;
    for (int r = 0; r < vt.n; ++r) tiles += (int64_t)a.H * vt.r[r].nQT;
    const bool one = nw == 4 && tiles <= kCUs;  // as above, in tiles of 128 rows
#define DIT_CASE(DD, QK, PV)                                                            \
    if (D == DD && qk_op == QK && pv_op == PV)                                           \
        return vt.split_tiles > 0 ? launch_attn_pipe16_varlen_inst<DD, QK, PV, 8, true, 2>(a, vt, s)   \
               : nw == 8          ? launch_attn_pipe16_varlen_inst<DD, QK, PV, 8, false, 2>(a, vt, s)  \
               : one              ? launch_attn_pipe16_varlen_inst<DD, QK, PV, 8, false, 1>(a, vt, s)  \
                                  : launch_attn_pipe16_varlen_inst<DD, QK, PV, 4, false, 2>(a, vt, s);
    DIT_PIPE16_CASES(DIT_CASE)
#undef DIT_CASE
    return hipErrorInvalidValue;
}

}  // namespace dit
