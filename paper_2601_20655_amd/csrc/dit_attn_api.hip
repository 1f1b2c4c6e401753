// C ABI of the library: argument validation, workspace carving, kernel sequencing.
// Every argument check happens before the first launch: a call that returns anything but DIT_ERR_HIP has had
// no effect; DIT_ERR_HIP (a launch failed) may leave workspace and output partly written.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include "../../include/dit_attn.h"
#include "dit_attn_internal.h"

namespace dit {
hipError_t launch_attn_d128_qb1(const AttnArgs&, int, int, bool, hipStream_t);
hipError_t launch_attn_d128_qb2(const AttnArgs&, int, int, bool, hipStream_t);
hipError_t launch_attn_d64_qb1(const AttnArgs&, int, int, bool, hipStream_t);
hipError_t launch_attn_d64_qb2(const AttnArgs&, int, int, bool, hipStream_t);

hipError_t launch_attn_pipe_d128_qb1(const AttnArgs&, int, int, int, hipStream_t);
hipError_t launch_attn_pipe_d128_qb2(const AttnArgs&, int, int, int, hipStream_t);
hipError_t launch_attn_pipe_d64_qb1(const AttnArgs&, int, int, int, hipStream_t);
hipError_t launch_attn_pipe_d64_qb2(const AttnArgs&, int, int, int, hipStream_t);
hipError_t launch_attn_pipe_fp8(const AttnArgs&, int D, int pv_op, int nw, hipStream_t);
hipError_t launch_attn_pipe_varlen_fp8(const AttnArgs&, const VarlenTable&, int D, int pv_op, int nw, hipStream_t);

// Software-pipelined kernel: pre-packed tiles, no key mask beyond the ragged tail.
hipError_t launch_attn_pipe(const AttnArgs& a, int D, int qb, int qk_op, int pv_op, int nw, hipStream_t s) {
    if (qk_op == OP_FP8) return qb == 1 ? launch_attn_pipe_fp8(a, D, pv_op, nw, s) : hipErrorInvalidValue;
    if (D == 128 && qb == 1) return launch_attn_pipe_d128_qb1(a, qk_op, pv_op, nw, s);
    if (D == 128 && qb == 2) return launch_attn_pipe_d128_qb2(a, qk_op, pv_op, nw, s);
    if (D == 64 && qb == 1) return launch_attn_pipe_d64_qb1(a, qk_op, pv_op, nw, s);
    if (D == 64 && qb == 2) return launch_attn_pipe_d64_qb2(a, qk_op, pv_op, nw, s);
    return hipErrorInvalidValue;
}

hipError_t launch_attn(const AttnArgs& a, int D, int qb, int qk_op, int pv_op, bool fused, hipStream_t s) {
    if (D == 128 && qb == 1) return launch_attn_d128_qb1(a, qk_op, pv_op, fused, s);
    if (D == 128 && qb == 2) return launch_attn_d128_qb2(a, qk_op, pv_op, fused, s);
    if (D == 64 && qb == 1) return launch_attn_d64_qb1(a, qk_op, pv_op, fused, s);
    if (D == 64 && qb == 2) return launch_attn_d64_qb2(a, qk_op, pv_op, fused, s);
    return hipErrorInvalidValue;
}
}  // namespace dit

namespace {

static_assert(DIT_MAX_REQUESTS == dit::kMaxRequests, "request limit of the ABI and of the kernel table");

thread_local char g_hip_error[256] = "";
thread_local hipEvent_t g_ev_before = nullptr, g_ev_after = nullptr;

dit_status hip_fail(hipError_t e, const char* where) {
    snprintf(g_hip_error, sizeof(g_hip_error), "%s: %s", where, hipGetErrorString(e));
    return DIT_ERR_HIP;
}

}  // namespace

int dit::report_hip_error(hipError_t e, const char* where) { return hip_fail(e, where); }

namespace {

constexpr size_t kAlign = 256;
size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Flags {
    int qk_op, pv_op, qb, nw;
    bool fused, simple, pipelined, resident, mfma32;
};

// Resolve flag bits into operand types and staging mode.
dit_status parse_flags(uint32_t f, Flags* out) {
    const uint32_t known = DIT_FLAG_QK_BF16 | DIT_FLAG_QK_F16 | DIT_FLAG_PV_BF16 | DIT_FLAG_PV_F16 |
                           DIT_FLAG_KV_PREPACK | DIT_FLAG_KV_FUSED | DIT_FLAG_WIDE_QTILE |
                           DIT_FLAG_SIMPLE_SCHEDULE | DIT_FLAG_BIG_WORKGROUP | DIT_FLAG_SMALL_WORKGROUP |
                           DIT_FLAG_PIPELINED_SCHEDULE | DIT_FLAG_KV_RESIDENT | DIT_FLAG_QK_FP8 |
                           DIT_FLAG_MFMA_32X32;
    if (f & ~known) return DIT_ERR_INVALID_ARG;
    if ((f & DIT_FLAG_QK_BF16) && (f & DIT_FLAG_QK_F16)) return DIT_ERR_INVALID_ARG;
    if ((f & DIT_FLAG_PV_BF16) && (f & DIT_FLAG_PV_F16)) return DIT_ERR_INVALID_ARG;
    if ((f & DIT_FLAG_KV_PREPACK) && (f & DIT_FLAG_KV_FUSED)) return DIT_ERR_INVALID_ARG;
    if ((f & DIT_FLAG_QK_FP8) && (f & (DIT_FLAG_QK_BF16 | DIT_FLAG_QK_F16))) return DIT_ERR_INVALID_ARG;
    out->qk_op = (f & DIT_FLAG_QK_FP8) ? dit::OP_FP8 : (f & DIT_FLAG_QK_BF16) ? dit::OP_BF16 : dit::OP_F16;
    out->pv_op = (f & DIT_FLAG_PV_BF16) ? dit::OP_BF16 : dit::OP_F16;
    out->fused = (f & DIT_FLAG_KV_FUSED) != 0;
    out->resident = (f & DIT_FLAG_KV_RESIDENT) != 0;
    out->mfma32 = (f & DIT_FLAG_MFMA_32X32) != 0;
    if (out->resident && out->fused) return DIT_ERR_INVALID_ARG;  // FUSED keeps nothing to reuse
    out->qb = (f & DIT_FLAG_WIDE_QTILE) ? 2 : 1;
    if ((f & DIT_FLAG_SIMPLE_SCHEDULE) && (f & DIT_FLAG_PIPELINED_SCHEDULE)) return DIT_ERR_INVALID_ARG;
    out->simple = (f & DIT_FLAG_SIMPLE_SCHEDULE) != 0;
    out->pipelined = (f & DIT_FLAG_PIPELINED_SCHEDULE) != 0;
    if ((f & DIT_FLAG_BIG_WORKGROUP) && (f & DIT_FLAG_SMALL_WORKGROUP)) return DIT_ERR_INVALID_ARG;
    out->nw = (f & DIT_FLAG_BIG_WORKGROUP) ? 8 : (f & DIT_FLAG_SMALL_WORKGROUP) ? 4 : 0;  // 0 = choose by size
    return DIT_OK;
}

// Self-attention (one sequence per batch entry or packed requests) runs the pipelined kernel on 16x16x32 MFMAs
// unless a flag asks for a form that only exists on 32x32x16 MFMAs (8-bit scores, 64 rows per wavefront, the
// plain and fused schedules) or for the 32x32x16 kernel itself.  The V^T tiles are packed in the matching key order.
bool self_attn_uses_mfma16(const Flags& fl) {
    return !fl.fused && !fl.simple && fl.qb == 1 && fl.qk_op != dit::OP_FP8 && !fl.mfma32;
}

// The one-launch kernel has the default operand types only, and asking for a workgroup size asks for the general
// kernel.
bool takes_short(const Flags& fl, uint32_t flags) {
    return self_attn_uses_mfma16(fl) && fl.qk_op == dit::OP_F16 && fl.pv_op == dit::OP_F16 &&
           !(flags & (DIT_FLAG_BIG_WORKGROUP | DIT_FLAG_SMALL_WORKGROUP));
}

// What the kernel for short sequences takes besides the attention kernel's arguments.
struct ShortCall {
    int qb;
    bool packed;  // table and tiles are in the workspace
    const dit::TableArgs* table;
    const dit::NormArgs* kn;
};

// Attention kernel launch, bracketed by the caller's timing events when the hook is set.  chain: layout of the chained
// cross-attention kernel, null for the other kernels.
dit_status run_attn(const dit::AttnArgs& aa, int D, const Flags& fl, bool fused, bool mfma16, hipStream_t s,
                    const dit::ChainLayout* chain = nullptr, const ShortCall* sc = nullptr) {
    const bool timed = g_ev_before && g_ev_after;
    hipError_t e;
    if (timed && (e = hipEventRecord(g_ev_before, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    if (sc) {
        e = dit::launch_attn_short(aa, *sc->table, *sc->kn, D, sc->qb, sc->packed, s);
    } else if (chain) {
        e = dit::launch_attn_pipe16_chain(aa, D, fl.qk_op, fl.pv_op, *chain, s);
    } else if (aa.tile_count_a) {
        e = dit::launch_attn_split(aa, D, fl.qk_op, fl.pv_op, s);
    } else if (mfma16 && aa.split.n_tail > 0) {
        e = dit::launch_attn_pipe16_split(aa, D, fl.qk_op, fl.pv_op, s);
    } else if (mfma16) {
        e = dit::launch_attn_pipe16(aa, D, fl.qk_op, fl.pv_op, fl.nw, s);
    } else if (!fused && !fl.simple) {
        e = dit::launch_attn_pipe(aa, D, fl.qb, fl.qk_op, fl.pv_op, fl.nw, s);
    } else {
        e = dit::launch_attn(aa, D, fl.qb, fl.qk_op, fl.pv_op, fused, s);
    }
    if (e != hipSuccess) return hip_fail(e, "attention kernel");
    if (timed && (e = hipEventRecord(g_ev_after, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    return DIT_OK;
}

bool dtype_ok(int32_t d) { return d == DIT_BF16 || d == DIT_F32; }

// Rows must start on 16-byte boundaries: base pointer and every stride.
bool aligned16(const void* p, const dit_strides& s, int32_t dtype) {
    const int64_t per16 = dtype == DIT_F32 ? 4 : 8;
    if (reinterpret_cast<uintptr_t>(p) & 15u) return false;
    return s.batch % per16 == 0 && s.token % per16 == 0 && s.head % per16 == 0;
}

// Rows of D contiguous channels may not overlap: a token's and a head's rows are at least D apart, and of the
// two strides the larger one clears all the rows the smaller one steps over ([B,L,H,D]: token >= H*head;
// [B,H,L,D]: head >= L*token).  L = 0 skips the second half (packed requests check their own total).
bool strides_ok(const dit_strides& s, int32_t B, int32_t H, int32_t D, int64_t L) {
    if (s.token < D || s.head < D) return false;
    if (B > 1 && s.batch < D) return false;
    if (s.batch < 0) return false;
    if (H > 1 && L > 1) {
        const bool token_major = s.token >= (int64_t)H * s.head;
        const bool head_major = s.head >= L * s.token;
        if (!token_major && !head_major) return false;
    }
    return true;
}

// Bytes from the first to the last element of a [B, L, H, D] tensor, or of n dense fp32 values.
struct Span {
    uintptr_t begin, end;
    bool meets(const Span& o) const { return begin < o.end && o.begin < end; }
};
Span span_of(const void* p, const dit_strides& s, int32_t dtype, int32_t B, int32_t H, int32_t D, int64_t L) {
    const int64_t n = (int64_t)(B - 1) * s.batch + (L - 1) * s.token + (int64_t)(H - 1) * s.head + D;
    const uintptr_t begin = reinterpret_cast<uintptr_t>(p);
    return {begin, begin + (uintptr_t)n * (dtype == DIT_F32 ? 4 : 2)};
}
Span span_of(const float* p, int64_t n) {
    const uintptr_t begin = reinterpret_cast<uintptr_t>(p);
    return {begin, p ? begin + (uintptr_t)n * 4 : begin};
}

// Whether what a self-attention call writes (out, lse) meets what its key-side passes read (k, v, the weights of the
// key rows): those passes then have to be over before the first row of out is written.
bool writes_over_keys(const dit_self_attn_params* p, int64_t L, const void* k, const void* v, const void* out,
                      const float* lse) {
    const Span rows = span_of(out, p->so, p->out_dtype, p->B, p->H, p->D, L);
    const Span sums = span_of(lse, (int64_t)p->B * p->H * L);
    for (const Span& in : {span_of(k, p->sk, p->in_dtype, p->B, p->H, p->D, L),
                           span_of(v, p->sv, p->in_dtype, p->B, p->H, p->D, L),
                           span_of(p->norm.mode != DIT_NORM_NONE ? p->norm.k_gamma : nullptr, (int64_t)p->H * p->D)})
        if (rows.meets(in) || sums.meets(in)) return true;
    return false;
}

// Whether the 16-bit rows that chained cross-attention writes pass the caches (non-temporal stores): where the
// last-level cache (256 MB) could keep less than half of them for whoever reads them next, and every row starts and
// ends with a 64-byte sector (one that two stores share is put together in the L2; past it each part is a write of its
// own: 4 x 32,760 x 40, 5 key tiles, rows 16 bytes off 1,142 -> 1,190 us).  us through the caches and past them: 4 x
// 32,760 x 40, 5 key tiles (1,342 MB) 1,070 and 1,035, 3 x 32,760 x 40, 2 key tiles 529 and 510; with a pass that reads
// the rows once: 4 x 32,760 x 40, 3 key tiles 1,219 and 1,203, 2 x 32,760 x 40 743 and 738, but 32,760 x 40 (335 MB)
// 375 and 378, 16,000 x 40 192 and 198, 8,000 x 40 100 and 105; with the output projection 2,000 x 40 130 and 133,
// 1,560 x 40 104 and 108, 5,000 x 12 46.8 and 48.3, 7,800 x 12 66.7 and 66.4 -- though the call alone is faster past
// them at every size (7,800 x 12 28.6 and 25.4): what it saves, the reader pays.  Self-attention (alone 3,600 x 40 286
// and 283, with the output projection 471 and 470) and head_dim 64 (630 and 622 to 634): level, through the caches.
bool rows_pass_caches(const void* out, const dit_cross_attn_params* p) {
    const int64_t bytes = 2 * (int64_t)p->B * p->Lq * p->H * p->D;
    if (p->out_dtype != DIT_BF16 || p->D != 128 || bytes <= (int64_t)512 << 20) return false;
    const int64_t strides = p->so.batch | p->so.token | p->so.head;
    return ((reinterpret_cast<uintptr_t>(out) | (uintptr_t)(2 * strides)) & 63u) == 0;
}

// eps >= 0, a known mode; the channel weights are read as float4
dit_status norm_ok(const dit_qk_norm& n) {
    if (n.mode != DIT_NORM_NONE && n.mode != DIT_NORM_HEAD && n.mode != DIT_NORM_TOKEN) return DIT_ERR_INVALID_ARG;
    if (n.mode == DIT_NORM_NONE) return DIT_OK;
    if (!(n.eps >= 0.f) || !isfinite(n.eps)) return DIT_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(n.q_gamma) | reinterpret_cast<uintptr_t>(n.k_gamma)) & 15u)
        return DIT_ERR_ALIGNMENT;
    return DIT_OK;
}

// Workspace tail for the per-token multipliers of q and k rows (TOKEN mode only).
size_t rstd_bytes(const dit_qk_norm& n, int64_t q_rows, int64_t k_rows) {
    if (n.mode != DIT_NORM_TOKEN) return 0;
    return round_up((size_t)q_rows * sizeof(float), kAlign) + round_up((size_t)k_rows * sizeof(float), kAlign);
}

// Fills the normalisation arguments of both kernels, and enqueues what they read: the rotation table (null: there is
// none, or it is in the workspace) and in TOKEN mode the per-token factors.
dit_status setup_rows(const dit::TableArgs* table, const dit_qk_norm& n, const void* q, const void* k, const dit_strides& sq,
                      const dit_strides& sk, int B, int Lq, int Lk, int H, int D, int in_f32, uint8_t* rstd_ws,
                      dit::NormArgs* qn, dit::NormArgs* kn, bool k_resident, hipStream_t s) {
    memset(qn, 0, sizeof(*qn));
    memset(kn, 0, sizeof(*kn));
    dit::RstdArgs rq, rk;
    const bool token = n.mode == DIT_NORM_TOKEN;
    if (n.mode != DIT_NORM_NONE) {
        qn->mode = kn->mode = n.mode;
        qn->eps = kn->eps = n.eps;
        qn->gamma = n.q_gamma;
        kn->gamma = n.k_gamma;
    }
    if (token) {
        rq.x = q; rq.rstd = reinterpret_cast<float*>(rstd_ws); rq.s_b = sq.batch; rq.s_t = sq.token; rq.s_h = sq.head;
        rq.B = B; rq.L = Lq; rq.H = H; rq.D = D; rq.in_f32 = in_f32; rq.eps = n.eps;
        rk = rq;
        rk.x = k; rk.rstd = reinterpret_cast<float*>(rstd_ws + round_up((size_t)B * Lq * sizeof(float), kAlign));
        rk.s_b = sk.batch; rk.s_t = sk.token; rk.s_h = sk.head; rk.L = Lk;
        qn->rstd = rq.rstd;
        kn->rstd = rk.rstd;
    }
    // the key rows' factors only feed the pre-pack pass
    const hipError_t e = dit::launch_row_stats(table, token ? &rq : nullptr, token && !k_resident ? &rk : nullptr, s);
    return e == hipSuccess ? DIT_OK : hip_fail(e, "row_stats_kernel");
}

void set_base(dit::TableArgs* ta, float base) {
    const long double l = log2l((long double)base);
    ta->log2_base = (double)l;
    ta->log2_base_lo = (double)(l - (long double)ta->log2_base);
}

struct SelfPlan {
    Flags fl;
    int64_t L;
    int nKT, nQT;
    int table_entries;
    size_t tab_off, tiles_off, rstd_off;
    size_t base;  // bytes without which the call is refused
    // Query tiles of the last round computed in pieces, where that pays: 8 wavefronts (split_nQT query tiles a head)
    // and this much more workspace, from base on.  A workspace of fewer than `total` bytes gets the whole-tile form.
    dit::SplitPlan split;
    int split_nQT;
    size_t total;
    int short_qb;  // > 0: the kernel for short sequences, in workgroups of 16 short_qb query rows
};

// How the self-attention kernel on 16x16x32 MFMAs is laid over the chip.  Estimates of its time in key-tile steps of an
// 8-wavefront workgroup (one per compute unit, 256 query rows; 1.2 to 1.45 us a step at head_dim 128), from runs over
// 21 shapes of 320 to 75,600 tokens and 2 to 40 heads, both head dimensions:
//   - a workgroup's start and end cost 7.5 steps, the end of a piece one more;
//   - with 4 wavefronts (128 rows) a compute unit holds two workgroups, which together take 1.04 of the 8-wavefront
//     step; one alone takes 0.83 of it; where all of them together are one round, in 16 rows a wavefront
//     (short_tile_rows), 0.58 + 0.001 a workgroup (1,600 x 3: 0.61, 1,600 x 9: 0.68, 6,240 x 4: 0.73, 1,600 x 19:
//     0.84), and in 64-row tiles 0.59;
//   - combining P pieces costs a launch and 2 x 256 rows of fp32 each: 3 + 0.037 P steps.
// The measured order of the forms follows these numbers wherever they are more than a few per cent apart: e.g. (tokens,
// heads) 3,600 x 3: 62.7 us in whole tiles, 40.1 in 5 pieces each; 6,240 x 4: 101.8 and 86.6 (2 pieces); 3,600 x 40:
// 262 and 258 (last 88 of 600 tiles in 2 pieces); 75,600 x 2: 5,294 and 4,395 (last 80 of 592 in 3 pieces); level or
// slower in pieces, and left whole: 1,560 x 12 (33.1 and 37.2), 6,307 x 20 (336 and 357), 20,280 x 3 (497 and 518).
// The figures of 16 rows a wavefront, and the 0.92 below, come from few shapes; at 50 of 640 to 10,125 tokens x 2 to 40
// heads, 39 to 247 tiles, both head dimensions, the choice was never more than 2 % slower than the better of whole
// tiles and pieces (3,600 x 6 65.3 whole, 67.9 in pieces, x 4 57.8 and 52.8; 4,800 x 6 88.4 and 86.9; 2,400 x 12 55.8,
// 62.4).
using dit::kCUs;
constexpr double kEnds = 7.5;
constexpr int kMaxPieces = 1024;  // 136.3 MB of workspace at head_dim 128

// tiles of 32 nw query rows; tiles64: of 64
double whole_tile_steps(int64_t tiles, int64_t tiles64, int nKT, int nw) {
    if (nw == 8) return (double)((tiles + kCUs - 1) / kCUs) * (nKT + kEnds);
    if (tiles <= kCUs) return (nKT + kEnds) * (tiles64 <= kCUs ? 0.59 : 0.58 + 0.001 * tiles);
    const int64_t pairs = tiles / (2 * kCUs), rest = tiles - pairs * 2 * kCUs;
    return (nKT + kEnds) * (1.04 * pairs + (rest == 0 ? 0.0 : rest <= kCUs ? 0.83 : 1.04));
}

// nw: the form that runs the tiles whole; tiles, tiles_nw, tiles64: query tiles of 256, of 32 nw and of 64 rows
dit::SplitPlan choose_split(int64_t tiles, int64_t tiles_nw, int64_t tiles64, int nKT, int nw) {
    dit::SplitPlan best{0, 0, 1};
    // (tiles of 16 rows a wavefront do a little better than their estimate: 3,600 x 8 whole 72.9, in pieces 80.1 at
    // 0.93 of it; 3,600 x 4 59.8 and 55.5 at 0.91)
    double best_steps = (nw == 4 && tiles_nw <= kCUs ? 0.92 : 0.97) * whole_tile_steps(tiles_nw, tiles64, nKT, nw);
    const int64_t rounds = tiles / kCUs;
    if (tiles % kCUs == 0 || tiles > (1 << 20)) return best;
    for (int64_t r = rounds; r >= 0 && r >= rounds - 1; --r) {  // rounds of whole tiles
        const int64_t tail = tiles - r * kCUs;
        for (int np = 2; np <= 16 && tail * np <= kMaxPieces && nKT / np >= 6; ++np) {
            const double steps = r * (nKT + kEnds) + (double)((tail * np + kCUs - 1) / kCUs) * ((double)nKT / np + kEnds + 1) +
                                 3.0 + 0.037 * (double)(tail * np);
            if (steps < best_steps) {
                best_steps = steps;
                best = dit::SplitPlan{(int)(r * kCUs), (int)tail, np};
            }
        }
    }
    return best;
}

}  // namespace

// Every workgroup works on all keys of its head, so this pays while one round of workgroups takes the call.  us a call,
// one after the other, general path and this (tokens x heads, 16-bit rows): head_dim 64, 16 rows: 256 x 4 16.0 and 9.3,
// 413 x 8 16.1 and 11.4, 512 x 2 16.8 and 10.7, 1,024 x 4 19.3 and 15.7; 32 rows: 512 x 15 16.8 and 13.0, 1,024 x 8
// 18.2 and 16.0.  head_dim 128, 16 rows: 64 x 4 13.7 and 12.0, 256 x 8 16.5 and 15.1, 384 x 10 19.4 and 17.7; 413 x 8
// 19.0 and 20.3, 640 x 2 21.1 and 24.0 (not taken); 32 rows spill there: 413 x 12 25.7.  In more than one round, on
// packed tiles: head_dim 64, 1,024 x 12 19.2 and 24.4, 256 x 40 12.6 and 16.5; 128, 256 x 24 17.2 and 21.5, 256 x 160
// 31.5 and 76.1.
int dit::choose_short(int64_t L, int64_t BH, int D, int table_entries) {
    if (table_entries > kShortTable || L > (D == 64 ? 1024 : 384)) return 0;
    if (BH * ((L + 15) / 16) <= kCUs) return 1;
    return D == 64 && BH * ((L + 31) / 32) <= kCUs ? 2 : 0;
}

// One launch saves two, about 2 us on the device and 3 more where the host is what a call waits for, and pays with
// every workgroup's own table and packing.  What makes that longer adds up, each about a microsecond: fp32 rows,
// per-token factors (a launch of their own ahead of it, which makes the table on the way otherwise), both together past
// 256 tokens (fp32 512 x 8 15.8 and 13.2 / 17.4 and 16.5), a table of more than two entries a thread,
// at head_dim 128 twice the work a key and more than three key tiles, at head_dim 64 more tiles than wavefronts (from
// 769 tokens on for most of them) and 32 query rows.  us in one launch and in three, replayed from a graph / called one
// after the other, at 0 to 2 of these: head_dim 64, 256 x 4 7.8 and 9.9 / 9.3 and 15.0; 512 x 15 12.3 and 13.7 / 13.0
// and 15.5; fp32 576 x 4 13.6 and 12.2 / 14.0 and 16.3; head_dim 128, 64 x 40 11.8 and 12.9 / 12.4 and 14.0; 256 x 8
// 14.6 and 13.8 / 15.1 and 15.0; fp32 192 x 20 15.9 and 15.3 / 16.3 and 17.0; at 3 and more: head_dim 64, 1,024 x 4
// 16.3 and 14.2 / 17.0 and 15.7, fp32 x 8 23.3 and 15.5 / 23.7 and 16.7, fp32, per token, 512 x 15 18.3 and 16.2 / 19.5
// and 18.0; head_dim 128, 1 x 6 x 64 tokens x 10 18.7 and 16.6 / 19.1 and 18.0, fp32, per token 23.6 and 19.2 / 24.2
// and 20.6 (the general path: 20.2 / 21.6).
bool dit::short_packs_itself(int64_t L, int D, int qb, int table_entries, bool f32_rows, bool token_norm) {
    const int own = D == 64 ? (L > 512) + 2 * (L > 768) + (qb == 2) : 1 + (L > 192);
    const int rows = f32_rows + token_norm + (f32_rows && token_norm && L > 256);
    return own + rows + (table_entries > 1024) < 3;
}

namespace {

dit_status plan_self(const dit_self_attn_params* p, SelfPlan* pl) {
    if (!p) return DIT_ERR_INVALID_ARG;
    if (p->B < 1 || p->H < 1 || p->D < 1 || p->T < 1 || p->Hg < 1 || p->Wg < 1) return DIT_ERR_INVALID_ARG;
    if (p->D != 64 && p->D != 128) return DIT_ERR_UNSUPPORTED;
    if (p->d_t < 0 || p->d_h < 0 || p->d_w < 0 || ((p->d_t | p->d_h | p->d_w) & 1) ||
        p->d_t + p->d_h + p->d_w != p->D)
        return DIT_ERR_INVALID_ARG;
    if (!(p->rope_base > 0.f) || !isfinite(p->rope_base) || !isfinite(p->scale)) return DIT_ERR_INVALID_ARG;
    if (!dtype_ok(p->in_dtype) || !dtype_ok(p->out_dtype)) return DIT_ERR_INVALID_ARG;
    dit_status st = parse_flags(p->flags, &pl->fl);
    if (st != DIT_OK) return st;
    if ((st = norm_ok(p->norm)) != DIT_OK) return st;
    if (pl->fl.fused && p->norm.mode != DIT_NORM_NONE) return DIT_ERR_UNSUPPORTED;
    const int64_t L = (int64_t)p->T * p->Hg * p->Wg;
    if (L > (1 << 24)) return DIT_ERR_UNSUPPORTED;  // token indices are 32-bit with room for tile padding
    if ((int64_t)p->B * p->H > (1 << 20)) return DIT_ERR_UNSUPPORTED;
    if (pl->fl.fused) {
        // fused staging keeps V in bf16 and is built for head_dim 128 with bf16 inputs only
        if (p->in_dtype != DIT_BF16 || p->D != 128 || pl->fl.pv_op != dit::OP_BF16 ||
            !(p->flags & DIT_FLAG_PV_BF16))
            return DIT_ERR_UNSUPPORTED;
    }
    if (!strides_ok(p->sq, p->B, p->H, p->D, L) || !strides_ok(p->sk, p->B, p->H, p->D, L) ||
        !strides_ok(p->sv, p->B, p->H, p->D, L) || !strides_ok(p->so, p->B, p->H, p->D, L))
        return DIT_ERR_INVALID_ARG;
    pl->L = L;
    pl->nKT = (int)((L + dit::kBK - 1) / dit::kBK);
    if (pl->fl.nw == 8 && pl->fl.qb == 2) return DIT_ERR_UNSUPPORTED;  // would need 512 registers x 512 lanes
    // 8-bit score operands exist in the pipelined 32-rows-per-wavefront kernel only
    if (pl->fl.qk_op == dit::OP_FP8 && (pl->fl.fused || pl->fl.simple || pl->fl.qb == 2)) return DIT_ERR_UNSUPPORTED;
    if (pl->fl.fused || pl->fl.simple || pl->fl.qb == 2) {
        pl->fl.nw = 4;  // only the pipelined 32-rows-per-wavefront kernel has the 8-wavefront form
    } else if (pl->fl.nw == 0) {
        const int64_t t8 = ((L + 255) / 256) * p->B * p->H, t4 = ((L + 127) / 128) * p->B * p->H;
        const int64_t t64 = ((L + 63) / 64) * p->B * p->H;
        if (self_attn_uses_mfma16(pl->fl))
            pl->fl.nw = whole_tile_steps(t8, t64, pl->nKT, 8) <= whole_tile_steps(t4, t64, pl->nKT, 4) ? 8 : 4;
        else  // 8 wavefronts when 256-row workgroups still cover the 256 CUs at least twice over
            pl->fl.nw = t8 >= 512 ? 8 : 4;
    }
    const int bq = 32 * pl->fl.nw * pl->fl.qb;
    pl->nQT = (int)((L + bq - 1) / bq);
    if ((int64_t)pl->nQT * p->B * p->H > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;
    if ((int64_t)pl->nKT * p->B * p->H > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;  // one pre-pack workgroup each
    pl->table_entries = p->T * (p->d_t / 2) + p->Hg * (p->d_h / 2) + p->Wg * (p->d_w / 2);
    pl->tab_off = 0;
    pl->tiles_off = round_up((size_t)pl->table_entries * sizeof(float2), kAlign);
    size_t tiles = pl->fl.fused ? 0 : (size_t)p->B * p->H * pl->nKT * dit::tile_bytes(p->D);
    pl->rstd_off = pl->tiles_off + round_up(tiles, kAlign);
    pl->base = pl->rstd_off + rstd_bytes(p->norm, (int64_t)p->B * L, (int64_t)p->B * L);
    if (pl->base == 0) pl->base = kAlign;
    pl->total = pl->base;
    pl->split = dit::SplitPlan{0, 0, 1};
    pl->short_qb = 0;
    if (takes_short(pl->fl, p->flags))
        pl->short_qb = dit::choose_short(L, (int64_t)p->B * p->H, p->D, pl->table_entries);
    if (self_attn_uses_mfma16(pl->fl) && !(p->flags & DIT_FLAG_SMALL_WORKGROUP)) {
        pl->split_nQT = (int)((L + 255) / 256);
        pl->split = choose_split((int64_t)pl->split_nQT * p->B * p->H, (int64_t)pl->nQT * p->B * p->H,
                                 ((L + 63) / 64) * p->B * p->H, pl->nKT, pl->fl.nw);
        if (pl->split.n_tail > 0)
            pl->total = pl->base + round_up(dit::part_o_bytes((int64_t)pl->split.n_tail * pl->split.n_piece, p->D), kAlign) +
                        round_up(dit::part_ml_bytes((int64_t)pl->split.n_tail * pl->split.n_piece), kAlign);
    }
    return DIT_OK;
}

// The split of a plan, if the workspace holds its pieces: fills the kernel's arguments and switches the plan to it.
void apply_split(SelfPlan* pl, int D, uint8_t* ws, size_t workspace_bytes, dit::AttnArgs* aa) {
    if (pl->split.n_tail == 0 || workspace_bytes < pl->total) return;
    pl->fl.nw = 8;
    pl->nQT = pl->split_nQT;
    aa->nQT = pl->nQT;
    aa->split = pl->split;
    aa->part_o = reinterpret_cast<float*>(ws + pl->base);
    aa->part_ml = reinterpret_cast<float2*>(
        ws + pl->base + round_up(dit::part_o_bytes((int64_t)pl->split.n_tail * pl->split.n_piece, D), kAlign));
}

struct VarlenPlan {
    Flags fl;
    dit::VarlenTable vt;
    int maxT, maxHg, maxWg;
    int table_entries;
    size_t tab_off, tiles_off, rstd_off;
    size_t base, total;     // as in SelfPlan
    size_t part_ml_off;     // with pieces: their row statistics (their outputs start at base)
    dit::SplitPlan single;  // one request: its split as dit_attn_forward would have it
};

// Time, in the steps of whole_tile_steps, until `slots` workgroups at a time have worked off the classes of equal
// workgroups in the order given (longest first); *half: until half of the slots have nothing left to do.
struct PackedClass {
    int64_t count;
    double steps;
};
double work_off(const PackedClass* c, int n, int64_t slots, double* half = nullptr) {
    struct Group {
        double at;
        int64_t slots;
    } g[2 * DIT_MAX_REQUESTS + 8];
    int ng = 1;
    g[0] = Group{0.0, slots};  // ascending in time
    for (int i = 0; i < n; ++i) {
        int64_t left = c[i].count;
        while (left > 0) {
            const int64_t k = left < g[0].slots ? left : g[0].slots;
            const double end = g[0].at + c[i].steps;
            left -= k;
            g[0].slots -= k;
            if (g[0].slots == 0) {
                --ng;
                for (int j = 0; j < ng; ++j) g[j] = g[j + 1];
            }
            int j = ng;
            while (j > 0 && g[j - 1].at > end) --j;
            if (j > 0 && g[j - 1].at == end) {
                g[j - 1].slots += k;
            } else if (ng < (int)(sizeof(g) / sizeof(g[0]))) {
                for (int m = ng; m > j; --m) g[m] = g[m - 1];
                g[j] = Group{end, k};
                ++ng;
            } else {
                g[j < ng ? j : ng - 1].slots += k;
            }
        }
    }
    if (half) {
        int64_t done = 0;
        int i = 0;
        for (; i < ng - 1 && done + g[i].slots < slots / 2; ++i) done += g[i].slots;
        *half = g[i].at;
    }
    return g[ng - 1].at;
}

// Several packed requests: wavefronts per workgroup, and pieces per query tile of each request, by the numbers that
// choose_split goes by.  A request is cut into pieces of at most one length common to all; batches of more than six
// rounds of workgroups are left whole (their last round is a small part of them).  *nw is for whole tiles; pieces, where
// a request gets more than one, are computed by 8 wavefronts.
void choose_packed(const dit::VarlenTable& vt, int H, uint32_t flags, int* nw, int* pieces) {
    PackedClass c8[DIT_MAX_REQUESTS], c4[DIT_MAX_REQUESTS];
    int64_t n8 = 0, n4 = 0;
    for (int r = 0; r < vt.n; ++r) {
        const dit::ReqDesc& d = vt.r[r];
        c8[r] = PackedClass{(int64_t)H * ((d.L + 255) / 256), d.nKT + kEnds};
        c4[r] = PackedClass{(int64_t)H * ((d.L + 127) / 128), d.nKT + kEnds};
        n8 += c8[r].count;
        n4 += c4[r].count;
    }
    if (n8 > 6 * kCUs) {
        if (*nw == 0) *nw = 8;
        return;
    }
    const double t8 = work_off(c8, vt.n, kCUs);
    double half4 = 0.0;  // from here on at most one workgroup per compute unit is left
    const double all4 = work_off(c4, vt.n, 2 * kCUs, &half4);
    // (packed requests are not cut into 64-row tiles)
    const double t4 = n4 <= kCUs ? (0.58 + 0.001 * n4) * all4 : 1.04 * half4 + 0.83 * (all4 - half4);
    if (*nw == 0) *nw = t8 <= t4 ? 8 : 4;
    if (flags & DIT_FLAG_SMALL_WORKGROUP) return;
    double best = 0.97 * (*nw == 8 ? t8 : t4);
    int best_len = 0;
    const int longest = vt.r[0].nKT;
    auto pieces_of = [](int nKT, int len) {
        int np = (nKT + len - 1) / len;
        if (np > nKT / 6) np = nKT / 6;
        return np > 16 ? 16 : np < 1 ? 1 : np;
    };
    for (int cut : {2, 3, 4, 5, 6, 8, 12, 16}) {
        const int len = (longest + cut - 1) / cut;
        if (len < 6) break;
        PackedClass c[DIT_MAX_REQUESTS];
        int64_t total = 0;
        for (int r = 0; r < vt.n; ++r) {
            const int np = pieces_of(vt.r[r].nKT, len);
            PackedClass k{c8[r].count * np, (double)vt.r[r].nKT / np + kEnds + (np > 1 ? 1 : 0)};
            if (np > 1) total += k.count;
            int j = r;
            for (; j > 0 && c[j - 1].steps < k.steps; --j) c[j] = c[j - 1];
            c[j] = k;
        }
        if (total > kMaxPieces) break;
        const double t = work_off(c, vt.n, kCUs) + 3.0 + 0.037 * (double)total;
        if (t < best) {
            best = t;
            best_len = len;
        }
    }
    if (best_len == 0) return;
    for (int r = 0; r < vt.n; ++r) pieces[r] = pieces_of(vt.r[r].nKT, best_len);
}

// workspace_bytes: what the call has (the plan of a workspace query assumes that everything fits)
dit_status plan_varlen(const dit_varlen_attn_params* p, size_t workspace_bytes, VarlenPlan* pl) {
    if (!p || !p->grids) return DIT_ERR_INVALID_ARG;
    if (p->n_requests < 1 || p->H < 1 || p->D < 1) return DIT_ERR_INVALID_ARG;
    if (p->n_requests > DIT_MAX_REQUESTS) return DIT_ERR_UNSUPPORTED;
    if (p->D != 64 && p->D != 128) return DIT_ERR_UNSUPPORTED;
    if (p->d_t < 0 || p->d_h < 0 || p->d_w < 0 || ((p->d_t | p->d_h | p->d_w) & 1) ||
        p->d_t + p->d_h + p->d_w != p->D)
        return DIT_ERR_INVALID_ARG;
    if (!(p->rope_base > 0.f) || !isfinite(p->rope_base) || !isfinite(p->scale)) return DIT_ERR_INVALID_ARG;
    if (!dtype_ok(p->in_dtype) || !dtype_ok(p->out_dtype)) return DIT_ERR_INVALID_ARG;
    dit_status st = parse_flags(p->flags, &pl->fl);
    if (st != DIT_OK) return st;
    if ((st = norm_ok(p->norm)) != DIT_OK) return st;
    // only the pipelined kernel with pre-packed tiles and 32 rows per wavefront has this form
    if (pl->fl.fused || pl->fl.simple || pl->fl.qb == 2) return DIT_ERR_UNSUPPORTED;
    if (p->H > (1 << 16)) return DIT_ERR_UNSUPPORTED;
    if (!strides_ok(p->sq, 1, p->H, p->D, 0) || !strides_ok(p->sk, 1, p->H, p->D, 0) ||
        !strides_ok(p->sv, 1, p->H, p->D, 0) || !strides_ok(p->so, 1, p->H, p->D, 0))
        return DIT_ERR_INVALID_ARG;

    const int n = p->n_requests;
    int64_t Ls[DIT_MAX_REQUESTS], tok0[DIT_MAX_REQUESTS];
    int order[DIT_MAX_REQUESTS];
    int64_t total = 0, big_blocks = 0;
    pl->maxT = pl->maxHg = pl->maxWg = 0;
    for (int i = 0; i < n; ++i) {
        const dit_grid& g = p->grids[i];
        if (g.T < 1 || g.Hg < 1 || g.Wg < 1) return DIT_ERR_INVALID_ARG;
        Ls[i] = (int64_t)g.T * g.Hg * g.Wg;
        if (Ls[i] > (1 << 24)) return DIT_ERR_UNSUPPORTED;
        tok0[i] = total;
        total += Ls[i];
        big_blocks += (Ls[i] + 255) / 256 * p->H;
        if (g.T > pl->maxT) pl->maxT = g.T;
        if (g.Hg > pl->maxHg) pl->maxHg = g.Hg;
        if (g.Wg > pl->maxWg) pl->maxWg = g.Wg;
        order[i] = i;
    }
    if (total > (1 << 24)) return DIT_ERR_UNSUPPORTED;  // token indices are 32-bit with room for tile padding
    // longest request first (stable, so equal lengths keep the caller's order)
    for (int i = 1; i < n; ++i) {
        const int o = order[i];
        int j = i;
        for (; j > 0 && Ls[order[j - 1]] < Ls[o]; --j) order[j] = order[j - 1];
        order[j] = o;
    }
    dit::VarlenTable& vt = pl->vt;
    memset(&vt, 0, sizeof(vt));
    vt.n = n;
    vt.total_tokens = (int)total;
    int tile0 = 0;
    for (int r = 0; r < n; ++r) {
        const int i = order[r];
        dit::ReqDesc& d = vt.r[r];
        d.tok0 = (int)tok0[i];
        d.L = (int)Ls[i];
        d.Hg = p->grids[i].Hg;
        d.Wg = p->grids[i].Wg;
        d.nKT = (int)((Ls[i] + dit::kBK - 1) / dit::kBK);
        d.tile0 = tile0;
        tile0 += d.nKT;
    }
    vt.total_tiles = tile0;
    if ((int64_t)tile0 * p->H > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;

    pl->table_entries = pl->maxT * (p->d_t / 2) + pl->maxHg * (p->d_h / 2) + pl->maxWg * (p->d_w / 2);
    pl->tab_off = 0;
    pl->tiles_off = round_up((size_t)pl->table_entries * sizeof(float2), kAlign);
    pl->rstd_off = pl->tiles_off + round_up((size_t)tile0 * p->H * dit::tile_bytes(p->D), kAlign);
    pl->base = pl->rstd_off + rstd_bytes(p->norm, total, total);
    pl->total = pl->base;
    pl->single = dit::SplitPlan{0, 0, 1};
    int pieces[DIT_MAX_REQUESTS];
    for (int r = 0; r < n; ++r) pieces[r] = 1;
    if (!self_attn_uses_mfma16(pl->fl)) {
        if (pl->fl.nw == 0) pl->fl.nw = big_blocks >= 512 ? 8 : 4;
    } else if (n == 1) {
        // one request is laid out as dit_attn_forward does it, so that its result is the same bit for bit
        const int64_t t8 = ((total + 255) / 256) * p->H, t4 = ((total + 127) / 128) * p->H;
        const int64_t t64 = ((total + 63) / 64) * p->H;
        const int nKT = vt.r[0].nKT;
        if (pl->fl.nw == 0) pl->fl.nw = whole_tile_steps(t8, t64, nKT, 8) <= whole_tile_steps(t4, t64, nKT, 4) ? 8 : 4;
        if (!(p->flags & DIT_FLAG_SMALL_WORKGROUP))
            pl->single = choose_split(t8, pl->fl.nw == 8 ? t8 : t4, t64, nKT, pl->fl.nw);
    } else {
        choose_packed(vt, p->H, p->flags, &pl->fl.nw, pieces);
    }
    int64_t n_pieces = (int64_t)pl->single.n_tail * pl->single.n_piece;
    for (int r = 0; r < n; ++r)
        if (pieces[r] > 1) n_pieces += (int64_t)pieces[r] * p->H * ((vt.r[r].L + 255) / 256);
    if (n_pieces > 0)
        pl->total = pl->base + round_up(dit::part_o_bytes(n_pieces, p->D), kAlign) +
                    round_up(dit::part_ml_bytes(n_pieces), kAlign);
    pl->part_ml_off = pl->base + round_up(dit::part_o_bytes(n_pieces, p->D), kAlign);
    if (n_pieces > 0 && workspace_bytes < pl->total) {  // no room for the pieces: whole tiles
        for (int r = 0; r < n; ++r) pieces[r] = 1;
        pl->single = dit::SplitPlan{0, 0, 1};
        n_pieces = 0;
    }
    if (n_pieces > 0) pl->fl.nw = 8;

    // query tiles, pieces, and the order the workgroups are handed out in: longest first
    const int bq = 32 * pl->fl.nw;
    int64_t queue[8] = {0, 0, 0, 0, 0, 0, 0, 0}, piece0 = 0;
    vt.split_tiles = 0;
    for (int r = 0; r < n; ++r) {
        dit::ReqDesc& d = vt.r[r];
        d.nQT = (d.L + bq - 1) / bq;
        d.n_piece = pieces[r];
        d.piece0 = (int)piece0;
        if (d.n_piece > 1) {
            piece0 += (int64_t)p->H * d.nQT * d.n_piece;
            vt.split_tiles += p->H * d.nQT;
        }
        int j = r;
        for (; j > 0; --j) {
            const dit::ReqDesc& o = vt.r[vt.order[j - 1]];
            if ((int64_t)o.nKT * d.n_piece >= (int64_t)d.nKT * o.n_piece) break;
            vt.order[j] = vt.order[j - 1];
        }
        vt.order[j] = r;
    }
    for (int i = 0; i < n; ++i) {
        const dit::ReqDesc& d = vt.r[vt.order[i]];
        const int64_t blocks = (int64_t)p->H * d.n_piece * d.nQT;
        if (blocks > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;
        // the kernel's rule: XCD x takes range (x + i) % 8 of the eight the request's workgroups are cut into
        for (int x = 0; x < 8; ++x) queue[x] += (blocks >> 3) + (((x + i) & 7) < (blocks & 7) ? 1 : 0);
    }
    int64_t qmax = 0;
    for (int x = 0; x < 8; ++x) qmax = queue[x] > qmax ? queue[x] : qmax;
    if (8 * qmax > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;
    vt.queue_len = (int)qmax;
    return DIT_OK;
}

}  // namespace

// Wavefronts per workgroup and query tiles per workgroup (1 .. 32, from one head on into the next, of one request) of the
// chained cross-attention kernel.  Estimate in microseconds: rounds of workgroups x (start + query tiles x (what a query
// tile costs once + its key tiles)), fitted to chain lengths of 1 to 32 in both workgroup sizes at 11 shapes of 800 to
// 32,760 queries and 1 to 9 key tiles.  A compute unit (the device has `cus`) holds one workgroup (head_dim 64 with 4
// wavefronts: two, each half as slow again per key tile as alone).  How many key tiles attend is on the device; three
// fifths of the capacity are taken for it.
// Measured, us, lengths that fill the rounds and their neighbours: 32,760 queries x 12 heads, 5 key tiles: 4 query tiles a
// workgroup 98, 6 (one round) 77, 8 92; 32,760 x 40, 9 key tiles: 1 459, 4 416, 10 408, 16 549, 20 (one round) 416; 7,800 x
// 12, 3 key tiles: 1 25.0, 2 21.9; with 4 wavefronts 3 24.5; 1,105 x 7 x 3 requests, 7 key tiles: 18.1, with 4 14.1.
// head_dim 64 (13 shapes of 300 to 30,000 queries, 1 to 10 key tiles): 9,000 x 30, 10 key tiles: 8 wavefronts 1 72.9, 4 94.6, 5 (one
// round) 60.5, 6 70.5, 4 wavefronts 3 67.7, 4 85.2, 5 68.9; 3 key tiles: 5 32.2, with 4 33.5; 1,500 x 12, 10 key tiles:
// 14.6, with 4 12.9.  (With figures that held 8 wavefronts dear it was 4 wavefronts everywhere: 9,000 x 30 82, 39.6 with 3.)
void dit::choose_chain(int Lq, int B, int64_t H, int nKT, int D, int cus, int* nw, int* qch) {
    const double n = 0.6 * nKT + 0.5;
    double best = 0.0;
    int best_nw = 0;
    for (int w : {8, 4}) {
        if (*nw != 0 && *nw != w) continue;
        const int64_t tiles = (Lq + 32 * w - 1) / (32 * w) * H;  // of one request
        const int slots = D == 64 && w == 4 ? 2 * cus : cus;
        const double start = 2.5;
        const double tile = D == 64 ? (w == 8 ? 1.35 + 0.88 * n : 1.6 + n) : w == 8 ? 4.0 + 1.85 * n : 5.0 + 0.8 * n;
        const double alone = slots > cus ? 1.6 + 0.68 * n : tile;
        for (int ch = 1; ch <= 32 && ch <= tiles; ++ch) {
            const int64_t wgs = (tiles + ch - 1) / ch * B;
            const int64_t full = wgs / slots, left = wgs % slots;
            const double last = left == 0 ? 0.0 : start + ch * (2 * left <= slots ? alone : tile);
            const double t = full * (start + ch * tile) + last;
            if (best_nw == 0 || t < best) {
                best = t;
                best_nw = w;
                *qch = ch;
            }
        }
    }
    *nw = best_nw;
}

// One softmax whose 128-row query tiles are one round of workgroups takes those, or 64-row ones where they are too, in
// 16 rows a wavefront (see attn_pipe16_body); everything else goes by the estimate.
dit::ChainLayout dit::layout_chain(int Lq, int B, int64_t H, int nKT, int D, bool two, int cus, int nw) {
    ChainLayout c{nw, 32, 1};
    if (nw != 8 && !two && (int64_t)(Lq + 127) / 128 * B * H <= cus) {
        c.nw = short_tile_rows(B * H, Lq, cus) / 16;
        c.rows = 16;
    } else {
        choose_chain(Lq, B, H, nKT, D, cus, &c.nw, &c.qch);
    }
    return c;
}

namespace {

struct CrossPlan {
    Flags fl;
    bool layout16;  // tile images in the layout of the 16x16x32 kernels
    bool chain16;  // the chained 16x16x32 kernel (default)
    dit::ChainLayout chain;  // with it
    int nKT, nQT;
    int split, nTA;  // decoupled form: first key of the second sequence, tiles of the first (0, 0: joint)
    size_t mask_off, list_off, count_off, count_a_off, keysrc_off, tiles_off, rstd_off, total;
};

dit_status plan_cross(const dit_cross_attn_params* p, CrossPlan* pl) {
    if (!p) return DIT_ERR_INVALID_ARG;
    if (p->B < 1 || p->H < 1 || p->D < 1 || p->Lq < 1 || p->Lk < 1) return DIT_ERR_INVALID_ARG;
    if (p->D != 64 && p->D != 128) return DIT_ERR_UNSUPPORTED;
    if (!isfinite(p->scale)) return DIT_ERR_INVALID_ARG;
    if (!dtype_ok(p->in_dtype) || !dtype_ok(p->out_dtype)) return DIT_ERR_INVALID_ARG;
    dit_status st = parse_flags(p->flags, &pl->fl);
    if (st != DIT_OK) return st;
    if (pl->fl.fused) return DIT_ERR_UNSUPPORTED;
    if ((st = norm_ok(p->norm)) != DIT_OK) return st;
    if (p->Lq > (1 << 24) || p->Lk > (1 << 24) || (int64_t)p->B * p->H > (1 << 20)) return DIT_ERR_UNSUPPORTED;
    if (!strides_ok(p->sq, p->B, p->H, p->D, p->Lq) || !strides_ok(p->sk, p->B, p->H, p->D, p->Lk) ||
        !strides_ok(p->sv, p->B, p->H, p->D, p->Lk) || !strides_ok(p->so, p->B, p->H, p->D, p->Lq))
        return DIT_ERR_INVALID_ARG;
    if (p->Lk_split < 0 || p->Lk_split > p->Lk) return DIT_ERR_INVALID_ARG;
    pl->split = (p->Lk_split == p->Lk) ? 0 : p->Lk_split;  // a split at either end is the joint softmax
    pl->nTA = (pl->split + dit::kBK - 1) / dit::kBK;
    pl->nKT = pl->nTA + (p->Lk - pl->split + dit::kBK - 1) / dit::kBK;
    if (pl->fl.qk_op == dit::OP_FP8) return DIT_ERR_UNSUPPORTED;  // self-attention only
    if (pl->split > 0 && (pl->fl.pipelined || pl->fl.qb == 2)) return DIT_ERR_UNSUPPORTED;
    if (pl->fl.nw == 8 && pl->fl.qb == 2) return DIT_ERR_UNSUPPORTED;
    // the pipelined kernel keeps the list of non-empty tiles in the 64 lanes of a wavefront
    if (pl->fl.pipelined && pl->nKT > 64) return DIT_ERR_UNSUPPORTED;
    // Default: the pipelined 16x16x32 kernel, each workgroup chaining several query tiles.
    // The plain kernel serves DIT_FLAG_SIMPLE_SCHEDULE (also with DIT_FLAG_MFMA_32X32
    // or 64 rows per wavefront); DIT_FLAG_PIPELINED_SCHEDULE asks for the listed 32x32x16 pipelined kernel.
    // (the chained kernel takes 16-bit query rows, normalised or not: fp32 rows go to the plain kernel)
    const bool bf16 = p->in_dtype == DIT_BF16;
    // Two softmaxes are chained where the form as a whole gains by it, and by nothing that depends on the rest of the call: a
    // row has the bits of its own kernel in a batch as alone.  Not with bf16 score operands, whose scores can be -inf (a
    // row's second pass would start from them), nor with bf16 probabilities, which the plain kernel sums as rounded.  At 45
    // shapes of 75 to 32,760 queries x 2 to 40 heads, 1 to 8 + 5 key tiles, resident keys, time of the plain kernel over
    // that of the chained one: head_dim 128 with bf16 output 1.07 (0.96 to 1.20; 32,760 x 40, 5 + 5 tiles 585 -> 489 us, 9,000
    // x 30, 1 + 5 tiles 86 -> 82), with fp32 output 1.02 (0.93 to 1.15: a pass over one or two tiles does not pay for parking
    // and wider rows), head_dim 64 0.95 (0.80 to 1.13).
    const bool two = p->D == 128 && pl->fl.qk_op == dit::OP_F16 && pl->fl.pv_op == dit::OP_F16;
    // Wherever one of the calls that may share resident tiles can be chained, all of them lay the tiles out for it: not
    // the number or the type of the query rows or the type of the output decides.  The plain kernel reads either layout.
    pl->layout16 = !pl->fl.simple && !pl->fl.pipelined && !pl->fl.mfma32 && pl->fl.qb == 1 && (pl->split == 0 ? bf16 : two);
    pl->chain16 = pl->layout16 && bf16 && (pl->split == 0 || p->out_dtype == DIT_BF16);
    if (!pl->fl.pipelined && !pl->chain16) pl->fl.simple = true;
    if (pl->chain16) {
        pl->chain = dit::layout_chain(p->Lq, p->B, p->H, pl->nKT, p->D, pl->split > 0, kCUs, pl->fl.nw);
    } else if (pl->fl.simple || pl->fl.qb == 2) {
        pl->fl.nw = 4;
    } else if (pl->fl.nw == 0) {
        // few key tiles per query tile: two small workgroups per CU overlap each other's
        // prologue and epilogue better than one large workgroup saves on tile traffic (measured)
        pl->fl.nw = 4;
    }
    const int bq = pl->chain16 ? pl->chain.nw * pl->chain.rows : 32 * pl->fl.nw * pl->fl.qb;
    pl->nQT = (p->Lq + bq - 1) / bq;
    if ((int64_t)pl->nQT * p->B * p->H > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;
    if ((int64_t)pl->nKT * p->B * p->H > 0x7fffffffLL) return DIT_ERR_UNSUPPORTED;
    // workspace: per-tile key masks, compacted list of non-empty tiles, their count, the source key of
    // every tile slot, tile images
    pl->mask_off = 0;
    pl->list_off = round_up((size_t)p->B * pl->nKT * sizeof(uint64_t), kAlign);
    pl->count_off = pl->list_off + round_up((size_t)p->B * pl->nKT * sizeof(int), kAlign);
    pl->count_a_off = pl->count_off + round_up((size_t)p->B * sizeof(int), kAlign);
    pl->keysrc_off = pl->count_a_off + round_up((size_t)p->B * sizeof(int), kAlign);
    pl->tiles_off = pl->keysrc_off + round_up((size_t)p->B * pl->nKT * dit::kBK * sizeof(int), kAlign);
    pl->rstd_off = pl->tiles_off + round_up((size_t)p->B * p->H * pl->nKT * dit::tile_bytes(p->D), kAlign);
    pl->total = pl->rstd_off + rstd_bytes(p->norm, (int64_t)p->B * p->Lq, (int64_t)p->B * p->Lk);
    return DIT_OK;
}

}  // namespace

int dit::packed_layout(const void* params, size_t workspace_bytes, int* split_tiles) {
    VarlenPlan pl;
    if (plan_varlen(static_cast<const dit_varlen_attn_params*>(params), workspace_bytes, &pl) != DIT_OK) return 0;
    *split_tiles = pl.vt.split_tiles + pl.single.n_tail;
    return pl.fl.nw;
}

extern "C" {

size_t dit_attn_workspace_bytes(const dit_self_attn_params* p) {
    SelfPlan pl;
    return plan_self(p, &pl) == DIT_OK ? pl.total : 0;
}

size_t dit_cross_attn_workspace_bytes(const dit_cross_attn_params* p) {
    CrossPlan pl;
    return plan_cross(p, &pl) == DIT_OK ? pl.total : 0;
}

dit_status dit_attn_forward(const void* q, const void* k, const void* v, void* out, float* lse,
                            const dit_self_attn_params* p, void* workspace, size_t workspace_bytes,
                            void* stream) {
    SelfPlan pl;
    dit_status st = plan_self(p, &pl);
    if (st != DIT_OK) return st;
    if (!q || !out) return DIT_ERR_INVALID_ARG;
    if (!pl.fl.resident && (!k || !v)) return DIT_ERR_INVALID_ARG;
    if (!aligned16(q, p->sq, p->in_dtype) || !aligned16(out, p->so, p->out_dtype)) return DIT_ERR_ALIGNMENT;
    if (!pl.fl.resident && (!aligned16(k, p->sk, p->in_dtype) || !aligned16(v, p->sv, p->in_dtype)))
        return DIT_ERR_ALIGNMENT;
    if (lse && (reinterpret_cast<uintptr_t>(lse) & 3u)) return DIT_ERR_ALIGNMENT;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) || workspace_bytes < pl.base)
        return DIT_ERR_WORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);

    dit::RopeGeom rg;
    rg.hd[0] = p->d_t / 2; rg.hd[1] = p->d_h / 2; rg.hd[2] = p->d_w / 2;
    rg.off[0] = 0; rg.off[1] = p->T * rg.hd[0]; rg.off[2] = rg.off[1] + p->Hg * rg.hd[1];
    rg.Hg = p->Hg; rg.Wg = p->Wg;

    dit::TableArgs ta;
    ta.tab = reinterpret_cast<float2*>(ws + pl.tab_off);
    ta.n[0] = p->T; ta.n[1] = p->Hg; ta.n[2] = p->Wg;
    ta.origin[0] = p->t0; ta.origin[1] = p->h0; ta.origin[2] = p->w0;
    ta.rg = rg;
    set_base(&ta, p->rope_base);
    ta.total = pl.table_entries;
    hipError_t e = hipSuccess;
    const float scale = p->scale > 0.f ? p->scale : 1.0f / sqrtf((float)p->D);

    dit::NormArgs qn, kn;
    // a short sequence in one launch, or, the same bit for bit, in one on tiles that are in the workspace before it
    const bool one = pl.short_qb > 0 && !pl.fl.resident && !writes_over_keys(p, pl.L, k, v, out, lse) &&
                     dit::short_packs_itself(pl.L, p->D, pl.short_qb, pl.table_entries, p->in_dtype == DIT_F32,
                                             p->norm.mode == DIT_NORM_TOKEN);
    st = setup_rows(pl.fl.resident || one ? nullptr : &ta, p->norm, q, k, p->sq, p->sk, p->B, (int)pl.L, (int)pl.L,
                    p->H, p->D, p->in_dtype == DIT_F32, ws + pl.rstd_off, &qn, &kn, pl.fl.resident, s);
    if (st != DIT_OK) return st;

    if (!pl.fl.fused && !pl.fl.resident && !one) {
        dit::PackArgs pa;
        memset(&pa, 0, sizeof(pa));
        pa.kn = kn;
        pa.k = k; pa.v = v; pa.valid = nullptr;
        pa.tiles = ws + pl.tiles_off;
        pa.tile_mask = nullptr;
        pa.tab = ta.tab;
        pa.B = p->B; pa.H = p->H; pa.Lk = (int)pl.L; pa.nKT = pl.nKT;
        pa.in_f32 = p->in_dtype == DIT_F32;
        pa.v_layout = self_attn_uses_mfma16(pl.fl) ? 1 : 0;
        pa.sk_b = p->sk.batch; pa.sk_t = p->sk.token; pa.sk_h = p->sk.head;
        pa.sv_b = p->sv.batch; pa.sv_t = p->sv.token; pa.sv_h = p->sv.head;
        pa.rg = rg;
        e = dit::launch_prepack(pa, p->D, pl.fl.qk_op, pl.fl.pv_op, s);
        if (e != hipSuccess) return hip_fail(e, "kv_prepack_kernel");
    }

    dit::AttnArgs aa;
    memset(&aa, 0, sizeof(aa));
    aa.q = q; aa.out = out; aa.lse = lse;
    aa.tiles = pl.fl.fused ? nullptr : ws + pl.tiles_off;
    aa.tile_mask = nullptr;
    aa.tab = ta.tab;
    aa.k = k; aa.v = v;
    aa.sk_b = p->sk.batch; aa.sk_t = p->sk.token; aa.sk_h = p->sk.head;
    aa.sv_b = p->sv.batch; aa.sv_t = p->sv.token; aa.sv_h = p->sv.head;
    aa.B = p->B; aa.H = p->H; aa.Lq = (int)pl.L; aa.Lk = (int)pl.L; aa.nKT = pl.nKT; aa.nQT = pl.nQT;
    aa.in_f32 = p->in_dtype == DIT_F32; aa.out_f32 = p->out_dtype == DIT_F32;
    aa.sq_b = p->sq.batch; aa.sq_t = p->sq.token; aa.sq_h = p->sq.head;
    aa.so_b = p->so.batch; aa.so_t = p->so.token; aa.so_h = p->so.head;
    aa.rg = rg;
    aa.qscale = scale * dit::kLog2e;
    aa.qn = qn;
    if (pl.short_qb > 0) {
        aa.nQT = (int)((pl.L + 16 * pl.short_qb - 1) / (16 * pl.short_qb));
        const ShortCall sc{pl.short_qb, !one, &ta, &kn};
        return run_attn(aa, p->D, pl.fl, false, true, s, nullptr, &sc);
    }
    apply_split(&pl, p->D, ws, workspace_bytes, &aa);
    return run_attn(aa, p->D, pl.fl, pl.fl.fused, self_attn_uses_mfma16(pl.fl), s);
}

}  // extern "C"

namespace {

// Both cross-attention entry points: which keys attend comes as a byte mask (kv_valid, nullable) or as two counts
// per request (kv_len with second_start; use_len).
dit_status cross_forward(const void* q, const void* k, const void* v, const uint8_t* kv_valid, bool use_len,
                         const int32_t* kv_len, int32_t second_start, void* out, float* lse,
                         const dit_cross_attn_params* p, void* workspace, size_t workspace_bytes, void* stream) {
    CrossPlan pl;
    dit_status st = plan_cross(p, &pl);
    if (st != DIT_OK) return st;
    if (use_len) {
        if (second_start < 0 || second_start > p->Lk) return DIT_ERR_INVALID_ARG;
        if (pl.split > 0 && second_start != pl.split) return DIT_ERR_INVALID_ARG;
        if (!pl.fl.resident && !kv_len) return DIT_ERR_INVALID_ARG;
        if (kv_len && (reinterpret_cast<uintptr_t>(kv_len) & 3u)) return DIT_ERR_ALIGNMENT;
    }
    if (!q || !out) return DIT_ERR_INVALID_ARG;
    if (!pl.fl.resident && (!k || !v)) return DIT_ERR_INVALID_ARG;
    if (!aligned16(q, p->sq, p->in_dtype) || !aligned16(out, p->so, p->out_dtype)) return DIT_ERR_ALIGNMENT;
    if (!pl.fl.resident && (!aligned16(k, p->sk, p->in_dtype) || !aligned16(v, p->sv, p->in_dtype)))
        return DIT_ERR_ALIGNMENT;
    if (lse && (reinterpret_cast<uintptr_t>(lse) & 3u)) return DIT_ERR_ALIGNMENT;
    if (lse && pl.split > 0) return DIT_ERR_UNSUPPORTED;  // two softmaxes have no single log-sum-exp
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) || workspace_bytes < pl.total)
        return DIT_ERR_WORKSPACE;

    if (pl.chain16) {  // a partition of the chip has fewer compute units
        int cus = 0;
        const hipError_t e = dit::compute_units(&cus);
        if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
        if (cus != kCUs) {
            pl.chain = dit::layout_chain(p->Lq, p->B, p->H, pl.nKT, p->D, pl.split > 0, cus, pl.fl.nw);
            pl.nQT = (p->Lq + pl.chain.nw * pl.chain.rows - 1) / (pl.chain.nw * pl.chain.rows);
        }
    }

    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    const float scale = p->scale > 0.f ? p->scale : 1.0f / sqrtf((float)p->D);

    dit::NormArgs qn, kn;
    st = setup_rows(nullptr, p->norm, q, k, p->sq, p->sk, p->B, p->Lq, p->Lk, p->H, p->D, p->in_dtype == DIT_F32,
                    ws + pl.rstd_off, &qn, &kn, pl.fl.resident, s);
    if (st != DIT_OK) return st;

    dit::PackArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.kn = kn;
    pa.k = k; pa.v = v; pa.valid = kv_valid;
    pa.tiles = ws + pl.tiles_off;
    pa.tile_mask = reinterpret_cast<uint64_t*>(ws + pl.mask_off);
    pa.tile_list = reinterpret_cast<int*>(ws + pl.list_off);
    pa.tile_count = reinterpret_cast<int*>(ws + pl.count_off);
    pa.tile_count_a = pl.split > 0 ? reinterpret_cast<int*>(ws + pl.count_a_off) : nullptr;
    const bool listed = kv_valid && dit::mask_needs_key_list(p->B, p->H, p->Lk, pl.split);
    pa.key_src = listed ? reinterpret_cast<int*>(ws + pl.keysrc_off) : nullptr;
    pa.kv_len = use_len ? kv_len : nullptr;
    pa.second_start = second_start;
    pa.split = pl.split;
    pa.nTA = pl.nTA;
    pa.tab = nullptr;
    pa.v_layout = pl.layout16 ? 1 : 0;
    pa.B = p->B; pa.H = p->H; pa.Lk = p->Lk; pa.nKT = pl.nKT;
    pa.in_f32 = p->in_dtype == DIT_F32;
    pa.sk_b = p->sk.batch; pa.sk_t = p->sk.token; pa.sk_h = p->sk.head;
    pa.sv_b = p->sv.batch; pa.sv_t = p->sv.token; pa.sv_h = p->sv.head;
    if (!pl.fl.resident) {
        hipError_t e = hipSuccess;
        if (pa.key_src && (e = dit::launch_key_compact(pa, s)) != hipSuccess) return hip_fail(e, "key_compact_kernel");
        e = dit::launch_prepack(pa, p->D, pl.fl.qk_op, pl.fl.pv_op, s);
        if (e != hipSuccess) return hip_fail(e, "kv_prepack_kernel");
        if (pa.key_src) {  // (otherwise the pre-pack writes the tile list itself)
            e = dit::launch_tile_compact(pa, s);
            if (e != hipSuccess) return hip_fail(e, "tile_compact_kernel");
        }
    }

    dit::AttnArgs aa;
    memset(&aa, 0, sizeof(aa));
    aa.q = q; aa.out = out; aa.lse = lse;
    aa.tiles = pa.tiles;
    aa.tile_mask = pa.tile_mask;
    aa.tile_list = pa.tile_list;
    aa.tile_count = pa.tile_count;
    aa.tile_count_a = pa.tile_count_a;
    aa.nTA = pl.nTA;
    aa.layout16 = pl.layout16;
    aa.tab = nullptr;
    aa.B = p->B; aa.H = p->H; aa.Lq = p->Lq; aa.Lk = p->Lk; aa.nKT = pl.nKT; aa.nQT = pl.nQT;
    aa.in_f32 = p->in_dtype == DIT_F32; aa.out_f32 = p->out_dtype == DIT_F32;
    aa.sq_b = p->sq.batch; aa.sq_t = p->sq.token; aa.sq_h = p->sq.head;
    aa.so_b = p->so.batch; aa.so_t = p->so.token; aa.so_h = p->so.head;
    aa.out_once = rows_pass_caches(out, p);
    aa.qscale = scale * dit::kLog2e;
    aa.qn = qn;
    return run_attn(aa, p->D, pl.fl, false, false, s, pl.chain16 ? &pl.chain : nullptr);
}

}  // namespace

extern "C" {

dit_status dit_cross_attn_forward(const void* q, const void* k, const void* v, const uint8_t* kv_valid,
                                  void* out, float* lse, const dit_cross_attn_params* p, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    return cross_forward(q, k, v, kv_valid, false, nullptr, 0, out, lse, p, workspace, workspace_bytes, stream);
}

dit_status dit_cross_attn_forward_lengths(const void* q, const void* k, const void* v, const int32_t* kv_len,
                                          int32_t second_start, void* out, float* lse,
                                          const dit_cross_attn_params* p, void* workspace, size_t workspace_bytes,
                                          void* stream) {
    return cross_forward(q, k, v, nullptr, true, kv_len, second_start, out, lse, p, workspace, workspace_bytes,
                         stream);
}

size_t dit_attn_varlen_workspace_bytes(const dit_varlen_attn_params* p) {
    VarlenPlan pl;
    return plan_varlen(p, SIZE_MAX, &pl) == DIT_OK ? pl.total : 0;
}

dit_status dit_attn_varlen_forward(const void* q, const void* k, const void* v, void* out, float* lse,
                                   const dit_varlen_attn_params* p, void* workspace, size_t workspace_bytes,
                                   void* stream) {
    VarlenPlan pl;
    dit_status st = plan_varlen(p, workspace_bytes, &pl);
    if (st != DIT_OK) return st;
    if (!q || !out) return DIT_ERR_INVALID_ARG;
    if (!pl.fl.resident && (!k || !v)) return DIT_ERR_INVALID_ARG;
    if (!aligned16(q, p->sq, p->in_dtype) || !aligned16(out, p->so, p->out_dtype)) return DIT_ERR_ALIGNMENT;
    if (!pl.fl.resident && (!aligned16(k, p->sk, p->in_dtype) || !aligned16(v, p->sv, p->in_dtype)))
        return DIT_ERR_ALIGNMENT;
    if (lse && (reinterpret_cast<uintptr_t>(lse) & 3u)) return DIT_ERR_ALIGNMENT;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) || workspace_bytes < pl.base)
        return DIT_ERR_WORKSPACE;

    // one request is laid out as dit_attn_forward does it, so that its result is the same bit for bit; a short one goes
    // there
    if (pl.vt.n == 1 && takes_short(pl.fl, p->flags) &&
        dit::choose_short(pl.vt.total_tokens, p->H, p->D, pl.table_entries) > 0) {
        dit_self_attn_params one;
        memset(&one, 0, sizeof(one));
        one.B = 1; one.H = p->H; one.D = p->D;
        one.T = p->grids[0].T; one.Hg = p->grids[0].Hg; one.Wg = p->grids[0].Wg;
        one.t0 = p->t0; one.h0 = p->h0; one.w0 = p->w0;
        one.d_t = p->d_t; one.d_h = p->d_h; one.d_w = p->d_w;
        one.rope_base = p->rope_base; one.scale = p->scale;
        one.in_dtype = p->in_dtype; one.out_dtype = p->out_dtype; one.flags = p->flags;
        one.sq = p->sq; one.sk = p->sk; one.sv = p->sv; one.so = p->so;
        one.sq.batch = one.sk.batch = one.sv.batch = one.so.batch = 0;
        one.norm = p->norm;
        SelfPlan sp;
        // (rows that overlap are refused there, not here)
        if (plan_self(&one, &sp) == DIT_OK && workspace_bytes >= sp.base)
            return dit_attn_forward(q, k, v, out, lse, &one, workspace, workspace_bytes, stream);
    }

    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);

    // one table for all requests, long enough for the largest extent on each axis
    dit::RopeGeom rg;
    rg.hd[0] = p->d_t / 2; rg.hd[1] = p->d_h / 2; rg.hd[2] = p->d_w / 2;
    rg.off[0] = 0; rg.off[1] = pl.maxT * rg.hd[0]; rg.off[2] = rg.off[1] + pl.maxHg * rg.hd[1];
    rg.Hg = pl.maxHg; rg.Wg = pl.maxWg;  // replaced per request inside the kernels

    dit::TableArgs ta;
    ta.tab = reinterpret_cast<float2*>(ws + pl.tab_off);
    ta.n[0] = pl.maxT; ta.n[1] = pl.maxHg; ta.n[2] = pl.maxWg;
    ta.origin[0] = p->t0; ta.origin[1] = p->h0; ta.origin[2] = p->w0;
    ta.rg = rg;
    set_base(&ta, p->rope_base);
    ta.total = pl.table_entries;
    hipError_t e = hipSuccess;
    const float scale = p->scale > 0.f ? p->scale : 1.0f / sqrtf((float)p->D);

    dit::NormArgs qn, kn;
    dit_strides sq1 = p->sq, sk1 = p->sk;
    sq1.batch = sk1.batch = 0;
    st = setup_rows(pl.fl.resident ? nullptr : &ta, p->norm, q, k, sq1, sk1, 1, pl.vt.total_tokens, pl.vt.total_tokens,
                    p->H, p->D, p->in_dtype == DIT_F32, ws + pl.rstd_off, &qn, &kn, pl.fl.resident, s);
    if (st != DIT_OK) return st;

    dit::PackArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.kn = kn;
    pa.k = k; pa.v = v;
    pa.tiles = ws + pl.tiles_off;
    pa.tab = ta.tab;
    pa.B = 1; pa.H = p->H; pa.Lk = pl.vt.total_tokens; pa.nKT = pl.vt.total_tiles;
    pa.in_f32 = p->in_dtype == DIT_F32;
    pa.v_layout = self_attn_uses_mfma16(pl.fl) ? 1 : 0;
    pa.sk_t = p->sk.token; pa.sk_h = p->sk.head;
    pa.sv_t = p->sv.token; pa.sv_h = p->sv.head;
    pa.rg = rg;
    if (!pl.fl.resident) {
        e = dit::launch_prepack_varlen(pa, pl.vt, p->D, pl.fl.qk_op, pl.fl.pv_op, s);
        if (e != hipSuccess) return hip_fail(e, "kv_prepack_varlen_kernel");
    }

    dit::AttnArgs aa;
    memset(&aa, 0, sizeof(aa));
    aa.q = q; aa.out = out; aa.lse = lse;
    aa.tiles = pa.tiles;
    aa.tab = ta.tab;
    aa.B = 1; aa.H = p->H; aa.Lq = pl.vt.total_tokens; aa.Lk = pl.vt.total_tokens;
    aa.nKT = pl.vt.total_tiles; aa.nQT = pl.vt.r[0].nQT;  // (one request: as in dit_attn_forward)
    aa.split = pl.single;
    aa.part_o = reinterpret_cast<float*>(ws + pl.base);
    aa.part_ml = reinterpret_cast<float2*>(ws + pl.part_ml_off);
    aa.in_f32 = p->in_dtype == DIT_F32; aa.out_f32 = p->out_dtype == DIT_F32;
    aa.sq_t = p->sq.token; aa.sq_h = p->sq.head;
    aa.so_t = p->so.token; aa.so_h = p->so.head;
    aa.rg = rg;
    aa.qscale = scale * dit::kLog2e;
    aa.qn = qn;

    const bool timed = g_ev_before && g_ev_after;
    if (timed && (e = hipEventRecord(g_ev_before, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    e = pl.fl.qk_op == dit::OP_FP8
            ? dit::launch_attn_pipe_varlen_fp8(aa, pl.vt, p->D, pl.fl.pv_op, pl.fl.nw, s)
            : pl.single.n_tail > 0 ? dit::launch_attn_pipe16_split(aa, p->D, pl.fl.qk_op, pl.fl.pv_op, s)
            : self_attn_uses_mfma16(pl.fl)
                  ? dit::launch_attn_pipe16_varlen(aa, pl.vt, p->D, pl.fl.qk_op, pl.fl.pv_op, pl.fl.nw, s)
                  : dit::launch_attn_pipe_varlen(aa, pl.vt, p->D, pl.fl.qk_op, pl.fl.pv_op, pl.fl.nw, s);
    if (e != hipSuccess) return hip_fail(e, "attention kernel");
    if (timed && (e = hipEventRecord(g_ev_after, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    return DIT_OK;
}

dit_status dit_linear_forward(const void* x, const void* w, const void* bias, void* y, const dit_linear_params* p,
                              void* stream) {
    if (!x || !w || !y || !p) return DIT_ERR_INVALID_ARG;
    if (p->M < 1 || p->N < 1 || p->K < 1 || p->flags != 0) return DIT_ERR_INVALID_ARG;
    if (p->ldx < p->K || p->ldw < p->K || p->ldy < p->N) return DIT_ERR_INVALID_ARG;
    if (p->out_dtype != DIT_BF16 && p->out_dtype != DIT_F32) return DIT_ERR_INVALID_ARG;
    if (p->K % dit::kLinBK != 0 || p->N % 8 != 0) return DIT_ERR_UNSUPPORTED;
    // the kernel addresses the rows of one 256-row tile with 32-bit byte offsets
    if (p->ldx > (int64_t)1 << 22 || p->ldw > (int64_t)1 << 22) return DIT_ERR_UNSUPPORTED;
    const size_t ye = p->out_dtype == DIT_F32 ? 4 : 2;
    if ((uintptr_t)x % 16 || (uintptr_t)w % 16 || (uintptr_t)y % 16 || (p->ldx * 2) % 16 || (p->ldw * 2) % 16 ||
        (p->ldy * ye) % 16 || (uintptr_t)bias % 8)
        return DIT_ERR_ALIGNMENT;
    dit::LinearArgs a{};
    a.x = static_cast<const uint16_t*>(x);
    a.w = static_cast<const uint16_t*>(w);
    a.bias = static_cast<const uint16_t*>(bias);
    a.y = y;
    a.M = p->M;
    a.N = p->N;
    a.K = p->K;
    a.ldx = p->ldx;
    a.ldw = p->ldw;
    a.ldy = p->ldy;
    a.nTM = (p->M + dit::kLinBM - 1) / dit::kLinBM;
    a.nTN = (p->N + dit::kLinBN - 1) / dit::kLinBN;
    a.out_f32 = p->out_dtype == DIT_F32;
    if ((int64_t)a.nTM * a.nTN > 0x7fffffff) return DIT_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool timed = g_ev_before && g_ev_after;
    hipError_t e;
    if (timed && (e = hipEventRecord(g_ev_before, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    e = dit::launch_linear(a, s);
    if (e != hipSuccess) return hip_fail(e, "linear_kernel");
    if (timed && (e = hipEventRecord(g_ev_after, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    return DIT_OK;
}

dit_status dit_qkv_proj_forward(const void* x, const void* w, const void* bias, void* q_out,
                                const dit_linear_params* lp, const dit_self_attn_params* ap, void* workspace,
                                size_t workspace_bytes, void* stream) {
    if (!x || !w || !q_out || !lp || !ap) return DIT_ERR_INVALID_ARG;
    SelfPlan pl;
    dit_status st = plan_self(ap, &pl);
    if (st != DIT_OK) return st;
    // what the fused form covers: one sequence, head_dim 128, an even number of heads (a 256-feature tile is two
    // heads of one of q, k, v), 16-bit rows, the default attention kernel's tile images.  Of the q/k normalisations
    // the per-head one is done in the epilogue (a head's channels are inside a tile); the per-token one takes a second
    // pass over the K' images, because a token-wide mean spans every tile of the k part.
    if (ap->B != 1 || ap->D != 128 || (ap->H & 1) || ap->in_dtype != DIT_BF16 || !self_attn_uses_mfma16(pl.fl) ||
        pl.fl.resident)
        return DIT_ERR_UNSUPPORTED;
    if (lp->flags != 0 || lp->out_dtype != DIT_BF16) return DIT_ERR_INVALID_ARG;
    if (lp->M != pl.L || lp->N != 3 * (int64_t)ap->H * ap->D || lp->K < 1) return DIT_ERR_INVALID_ARG;
    if (lp->ldx < lp->K || lp->ldw < lp->K) return DIT_ERR_INVALID_ARG;
    if (lp->K % dit::kLinBK != 0) return DIT_ERR_UNSUPPORTED;
    if (lp->ldx > (int64_t)1 << 22 || lp->ldw > (int64_t)1 << 22) return DIT_ERR_UNSUPPORTED;
    if ((uintptr_t)x % 16 || (uintptr_t)w % 16 || (lp->ldx * 2) % 16 || (lp->ldw * 2) % 16 || (uintptr_t)bias % 8)
        return DIT_ERR_ALIGNMENT;
    if (!aligned16(q_out, ap->sq, DIT_BF16)) return DIT_ERR_ALIGNMENT;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) || workspace_bytes < pl.base)
        return DIT_ERR_WORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    dit::RopeGeom rg;
    rg.hd[0] = ap->d_t / 2; rg.hd[1] = ap->d_h / 2; rg.hd[2] = ap->d_w / 2;
    rg.off[0] = 0; rg.off[1] = ap->T * rg.hd[0]; rg.off[2] = rg.off[1] + ap->Hg * rg.hd[1];
    rg.Hg = ap->Hg; rg.Wg = ap->Wg;
    dit::TableArgs ta;
    ta.tab = reinterpret_cast<float2*>(ws + pl.tab_off);
    ta.n[0] = ap->T; ta.n[1] = ap->Hg; ta.n[2] = ap->Wg;
    ta.origin[0] = ap->t0; ta.origin[1] = ap->h0; ta.origin[2] = ap->w0;
    ta.rg = rg;
    set_base(&ta, ap->rope_base);
    ta.total = pl.table_entries;
    hipError_t e = dit::launch_row_stats(&ta, nullptr, nullptr, s);
    if (e != hipSuccess) return hip_fail(e, "row_stats_kernel");

    dit::LinearArgs a{};
    a.x = static_cast<const uint16_t*>(x);
    a.w = static_cast<const uint16_t*>(w);
    a.bias = static_cast<const uint16_t*>(bias);
    a.y = q_out;
    a.M = lp->M;
    a.N = lp->N;
    a.K = lp->K;
    a.ldx = lp->ldx;
    a.ldw = lp->ldw;
    a.ldy = 0;
    a.nTM = (lp->M + dit::kLinBM - 1) / dit::kLinBM;
    a.nTN = lp->N / dit::kLinBN;
    a.out_f32 = 0;
    a.qkv = 1;
    a.qkv_H = ap->H;
    a.qkv_nKT = pl.nKT;
    a.qkv_tiles = ws + pl.tiles_off;
    a.qkv_tab = ta.tab;
    a.qkv_rg = rg;
    a.qkv_sq_t = ap->sq.token;
    a.qkv_sq_h = ap->sq.head;
    a.qkv_qk_f16 = pl.fl.qk_op == dit::OP_F16;
    a.qkv_pv_f16 = pl.fl.pv_op == dit::OP_F16;
    a.qkv_norm = ap->norm.mode == DIT_NORM_HEAD ? 1 : ap->norm.mode == DIT_NORM_TOKEN ? 2 : 0;
    a.qkv_eps = ap->norm.eps;
    a.qkv_kgamma = ap->norm.k_gamma;
    if ((int64_t)a.nTM * a.nTN > 0x7fffffff) return DIT_ERR_UNSUPPORTED;
    const bool timed = g_ev_before && g_ev_after;
    if (timed && (e = hipEventRecord(g_ev_before, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    e = dit::launch_linear(a, s);
    if (e != hipSuccess) return hip_fail(e, "linear_kernel");
    if (timed && (e = hipEventRecord(g_ev_after, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
    if (ap->norm.mode == DIT_NORM_TOKEN) {
        dit::KRescaleArgs ra;
        ra.tiles = a.qkv_tiles;
        ra.H = ap->H;
        ra.nKT = pl.nKT;
        ra.L = (int)pl.L;
        ra.eps = ap->norm.eps;
        ra.qk_f16 = a.qkv_qk_f16;
        e = dit::launch_k_rescale(ra, s);
        if (e != hipSuccess) return hip_fail(e, "k_rescale_kernel");
    }
    return DIT_OK;
}

void dit_attn_set_timing_events(void* before, void* after) {
    g_ev_before = static_cast<hipEvent_t>(before);
    g_ev_after = static_cast<hipEvent_t>(after);
}

const char* dit_strerror(dit_status s) {
    switch (s) {
        case DIT_OK: return "ok";
        case DIT_ERR_INVALID_ARG: return "invalid argument";
        case DIT_ERR_UNSUPPORTED: return "unsupported shape or flag combination";
        case DIT_ERR_ALIGNMENT: return "pointer or stride breaks 16-byte row alignment";
        case DIT_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case DIT_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

const char* dit_last_hip_error(void) { return g_hip_error; }

int dit_attn_version(void) { return 10800; }  // 1.8.0

}  // extern "C"
