// Self-attention of short sequences in one launch (gfx950): rotation table, key and value packing, attention and the
// combination of key ranges by one workgroup per 16 or 32 query rows of a head.
//
// Sequences of a few hundred tokens are all latency on the general path: three launches one behind the other (rotation
// table, pre-pack, attention), each of which fills a small part of the chip, and in the last one a wavefront walks the
// key tiles one by one.  Here the wavefronts of a workgroup take one 64-key tile each (further ones in turn), all at
// the same time: K rows come from memory straight into the layout of the score MFMA's A operand, where a lane holds
// eight consecutive channels of a key, that is four whole rotation pairs; V rows go through LDS in rows and come back
// transposed (ds_read_b64_tr_b16); each wavefront keeps its own running maximum, and the results are put together
// through LDS as those of pieces along the keys are.  Every workgroup works out the rotation table and rotates all keys
// of its head again, which is the price, and why the sequence has to be short (choose_short).
//
// The workspace is left as the general path leaves it, byte for byte: rotation table, and tile images in the layout of
// the 16x16x32 kernels, written from the operand registers by the workgroups of the first query rows.  With RESIDENT
// the operands are read from such images instead of being made -- after the table and pre-pack kernels of the same
// call, where it writes over its keys or that is faster (short_packs_itself), or in a call on resident tiles -- with
// the same bits.
//
// What bounds it: one wavefront's chain of table entry (fp64), rows from memory, rotation, scores, maximum, products
// and combination, two wavefronts per SIMD; at head_dim 64 with up to four key tiles all of it (9 to 10 us) is what the
// host needs for a launch (per-token factors are a launch of their own ahead of it).  Whole calls, us, the general
// path and this: 256 tokens (4 x 8 x 8) x 4 heads x 64 16.0 and 9.3, 256 (16 x 16) x 8 x 128 16.5 and 15.1, on resident
// tiles 7.6 and 4.2, 11.3 and 6.5 (more at choose_short and short_packs_itself).  All eight wavefronts work on the
// table, whatever the number of key tiles: with as many wavefronts as tiles 60 tokens x 128 took 16.5 instead of 12.3.
// Tried: the first rows requested ahead of the table (registers: 18.3 -> 20.0 at 512 x 2 x 128).
#include "dit_attn_fwd_pipe16.h"

namespace dit {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

template <int D>
struct ShortGeom {
    static constexpr int VPITCH = D * 2 + 16;              // bytes of a V row in LDS
    static constexpr int OPITCH = D * 4 + 16;              // bytes of a row of a wavefront's partial output
    static constexpr int AREA = kBK * VPITCH;              // per wavefront: V rows, later its partial output
    static_assert(32 * OPITCH <= AREA, "the partial output takes the place of the V rows");
};

// IN: 0 bf16 rows, 1 fp32 rows, 2 resident tiles (query rows of either type)
template <int D, int QB, int IN>
__global__ void __launch_bounds__(64 * kShortWaves)
    attn_short_kernel(const AttnArgs a, const TableArgs ta, const NormArgs kn) {
    using G = TileGeom<D>;
    using S = ShortGeom<D>;
    constexpr int NKS = D / 32, NCB = D / 16;
    constexpr bool RESIDENT = IN == 2, F32 = IN == 1;
    const bool q_f32 = RESIDENT ? a.in_f32 != 0 : F32;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = a.nKT < kShortWaves ? a.nKT : kShortWaves;  // wavefronts that have key tiles
    const int i16 = lane & 15, g4 = lane >> 4;
    uint8_t* const area = smem + wave * S::AREA;
    float2* const stats = reinterpret_cast<float2*>(smem + nt * S::AREA);  // [wavefront][16 QB]: maximum, row sum
    // channel weights of the q and the k rows, this head (ones without), and, not RESIDENT, the rotation table
    float* const gamma = reinterpret_cast<float*>(stats + nt * 16 * QB);
    float2* const tab = reinterpret_cast<float2*>(gamma + 2 * D);

    const int logical = xcd_contiguous_block();
    const int bh = logical / a.nQT, rb = logical - bh * a.nQT;
    const int b = bh / a.H, h = bh - b * a.H;
    const int L = a.Lq;
    uint8_t* const tiles = const_cast<uint8_t*>(a.tiles) + (size_t)bh * a.nKT * G::TILE_BYTES;

    // ---- query rows are requested first ----
    u32x4 qraw[QB][NKS][2];
    int qrow[QB];
    auto request_q = [&](auto f32_tag) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int row = (rb * QB + qb) * 16 + i16;
            qrow[qb] = row < L ? row : L - 1;
            const int64_t off = (int64_t)b * a.sq_b + (int64_t)h * a.sq_h + (int64_t)qrow[qb] * a.sq_t + 8 * g4;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                if constexpr (decltype(f32_tag)::value) {
                    const float* const row = static_cast<const float*>(a.q) + off + 32 * ks;
                    const u32x4* const src = reinterpret_cast<const u32x4*>(row);
                    qraw[qb][ks][0] = src[0];
                    qraw[qb][ks][1] = src[1];
                } else {
                    const uint16_t* const src = static_cast<const uint16_t*>(a.q) + off + 32 * ks;
                    qraw[qb][ks][0] = *reinterpret_cast<const u32x4*>(src);
                }
            }
        }
    };
    if (q_f32) request_q(std::true_type{});
    else request_q(std::false_type{});

    // ---- key and value rows of a tile.  Rows past the end: the last one, and zeros in its place as operands. ----
    u32x4 kraw[4][NKS][2];
    int key[4];
    auto request_k = [&](int j, int kb) __attribute__((always_inline)) {
        const int n = j * kBK + 16 * kb + i16;
        key[kb] = n < L ? n : L - 1;
        const int64_t off = (int64_t)b * a.sk_b + (int64_t)h * a.sk_h + (int64_t)key[kb] * a.sk_t + 8 * g4;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            if constexpr (F32) {
                const u32x4* const src = reinterpret_cast<const u32x4*>(static_cast<const float*>(a.k) + off + 32 * ks);
                kraw[kb][ks][0] = src[0];
                kraw[kb][ks][1] = src[1];
            } else {
                kraw[kb][ks][0] = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.k) + off + 32 * ks);
            }
        }
    };
    // V rows, CPR lanes a row, 64 / CPR rows a pass, NVB passes at a time: into LDS as operands
    constexpr int CPR = D / 8, NVP = kBK * CPR / 64, NVB = F32 ? 4 : 8, NB = NVP / NVB;
    u32x4 vraw[NVB][2];
    auto request_v = [&](int j, int batch) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NVB; ++p) {
            const int n = j * kBK + (batch * NVB + p) * (64 / CPR) + lane / CPR;
            const int64_t off = (int64_t)b * a.sv_b + (int64_t)h * a.sv_h + (int64_t)(n < L ? n : L - 1) * a.sv_t +
                                8 * (lane % CPR);
            if constexpr (F32) {
                const u32x4* const src = reinterpret_cast<const u32x4*>(static_cast<const float*>(a.v) + off);
                vraw[p][0] = src[0];
                vraw[p][1] = src[1];
            } else {
                vraw[p][0] = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.v) + off);
            }
        }
    };
    // as much in flight as the registers hold (fp32 rows at head_dim 128: half of the keys)
    constexpr int KAHEAD = F32 && D == 128 ? 2 : 4;
    auto request_tile = [&](int j) __attribute__((always_inline)) {
        request_v(j, 0);
#pragma unroll
        for (int kb = 0; kb < KAHEAD; ++kb) request_k(j, kb);
    };

    // ---- rotation table and channel weights, in LDS; the first workgroup leaves the table in the workspace too ----
    // (RESIDENT: the weights of the k rows are in the tiles; their array is not read, it may be gone)
    for (int i = tid; i < (RESIDENT ? D : 2 * D); i += 64 * kShortWaves) {
        const float* const src = i < D ? a.qn.gamma : kn.gamma;
        gamma[i] = src ? src[(int64_t)h * D + (i & (D - 1))] : 1.f;
    }
    if constexpr (!RESIDENT) {
        for (int i = tid; i < ta.total; i += 64 * kShortWaves) {
            const float2 e = rope_entry(ta, i);
            tab[i] = e;
            if (logical == 0) ta.tab[i] = e;
        }
    }
    __syncthreads();

    const int h0 = a.rg.hd[0], h01 = a.rg.hd[0] + a.rg.hd[1];
    auto entry = [&](const RopeRow& rr, int ip) __attribute__((always_inline)) {
        const int idx = (ip < h0 ? rr.b[0] : ip < h01 ? rr.b[1] : rr.b[2]) + ip;
        if constexpr (RESIDENT) return a.tab[(uint32_t)idx];
        else return tab[idx];
    };
    // eight channels 32 ks + 8 g of a row at table rows rr: x -> rotated
    auto rotate8 = [&](float (&x)[8], const RopeRow& rr, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) {
            const float2 r = rotate_pair(x[2 * pp], x[2 * pp + 1], entry(rr, 16 * ks + 4 * g4 + pp));
            x[2 * pp] = r.x;
            x[2 * pp + 1] = r.y;
        }
    };
    auto values8 = [&](const u32x4 (&raw)[2], bool f32, float (&x)[8]) __attribute__((always_inline)) {
        if (f32) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(raw[e >> 2][e & 3]);
        } else {
            widen8(raw[0], x);
        }
    };
    // Multiplier of a row whose channels the four lanes (i, 0..3) hold.
    // (The empty statement makes the row a new value behind the branch: the compiler otherwise keeps what it widened
    // for the sum, of all rows at once.)
    // The order of a per-head sum is that of the kernel that reads the rows on the general path: of q rows the
    // attention kernel's (a lane's channels one after the other), of k rows the pre-pack's (eight channels, then chunks
    // pairwise), so that the tile images are the same whoever writes them.
    auto row_factor = [&](const NormArgs& n, u32x4 (&raw)[NKS][2], bool f32, int64_t stat,
                          auto k_row) __attribute__((always_inline)) {
        constexpr bool K_ROW = decltype(k_row)::value;
        float rs = 1.f;
        if (n.mode == 2) rs = n.rstd[stat];
        if (n.mode == 1) {
            float ss[NKS];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                float x[8];
                values8(raw[ks], f32, x);
                ss[ks] = K_ROW || ks == 0 ? 0.f : ss[ks - 1];
#pragma unroll
                for (int e = 0; e < 8; ++e) ss[ks] = fmaf(x[e], x[e], ss[ks]);
            }
            if constexpr (K_ROW) {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) ss[ks] = sum_across_rows16(ss[ks]);
#pragma unroll
                for (int m = 1; m < NKS; m <<= 1)
#pragma unroll
                    for (int ks = 0; ks < NKS; ks += 2 * m) ss[ks] += ss[ks + m];
            } else {
                ss[0] = sum_across_rows16(ss[NKS - 1]);
            }
            rs = 1.0f / sqrtf(ss[0] * (1.0f / D) + n.eps);
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            asm volatile("" : "+v"(raw[ks][0]));
            if (f32) asm volatile("" : "+v"(raw[ks][1]));
        }
        return rs;
    };
    // eight channels 32 ks + 8 g: times the row's factor and the channel weights (both 1 without a normalisation)
    auto scale8 = [&](float (&x)[8], float rs, const float* g, int ks) __attribute__((always_inline)) {
        const f32x4* const w = reinterpret_cast<const f32x4*>(g + 32 * ks + 8 * g4);
        const f32x4 w0 = w[0], w1 = w[1];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] *= rs * (e < 4 ? w0[e & 3] : w1[e & 3]);
    };

    // ---- query rows -> operand registers ----
    u32x4 Qf[QB][NKS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        int pt, ph, pw;
        token_pos(qrow[qb], a.rg, pt, ph, pw);
        const RopeRow rr = rope_row(a.rg, pt, ph, pw);
        const float rs = row_factor(a.qn, qraw[qb], q_f32, (int64_t)b * L + qrow[qb], std::false_type{});
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            float x[8];
            values8(qraw[qb][ks], q_f32, x);
            scale8(x, rs, gamma, ks);
            rotate8(x, rr, ks);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] *= a.qscale;
            Qf[qb][ks] = pack8<OP_F16>(x);
            asm volatile("" : "+v"(Qf[qb][ks]));
        }
    }

    // ---- this wavefront's key tiles ----
    f32x4 O[NCB][QB];
    float m_run[QB], l_run[QB];  // l_run: this lane's part of the row sum
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = -INFINITY;
        l_run[qb] = 0.f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) O[cb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int gsw = g4 ^ (((i16 >> 2) ^ (i16 >> 3)) & 1);  // layout 1: where chunk g of row i of 16 lies (pack_tile)
    for (int j = wave; j < a.nKT; j += kShortWaves) {
        uint8_t* const image = tiles + (size_t)j * G::TILE_BYTES;
        u32x4 Kf[4][NKS], Vf[RESIDENT ? NCB : 1];  // (RESIDENT: one 32-key group ahead)
        if constexpr (RESIDENT) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    Kf[kb][ks] =
                        *reinterpret_cast<const u32x4*>(image + (16 * kb + i16) * G::KROW + ks * 64 + gsw * 16);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
                Vf[cb] = *reinterpret_cast<const u32x4*>(image + G::K_BYTES + (16 * cb + i16) * G::VROW + gsw * 16);
        } else {
            auto stage_v = [&](int batch) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < NVB; ++p) {
                    const int r = (batch * NVB + p) * (64 / CPR) + lane / CPR;
                    float x[8];
                    values8(vraw[p], F32, x);
                    const u32x4 v = pack8<OP_F16>(x);
                    *reinterpret_cast<u32x4*>(area + r * S::VPITCH + (lane % CPR) * 16) =
                        j * kBK + r < L ? v : mk4(0u, 0u, 0u, 0u);
                }
            };
            request_tile(j);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                if (kb < NB) {
                    stage_v(kb);
                    __builtin_amdgcn_sched_barrier(0);
                    if (kb + 1 < NB) request_v(j, kb + 1);
                }
                if (kb > 0 && kb + KAHEAD - 1 < 4) request_k(j, kb + KAHEAD - 1);
                __builtin_amdgcn_sched_barrier(0);
                const bool inside = j * kBK + 16 * kb + i16 < L;
                int pt, ph, pw;
                token_pos(key[kb], a.rg, pt, ph, pw);
                const RopeRow rr = rope_row(a.rg, pt, ph, pw);
                const float rs = row_factor(kn, kraw[kb], F32, (int64_t)b * L + key[kb], std::true_type{});
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    float x[8];
                    values8(kraw[kb][ks], F32, x);
                    scale8(x, rs, gamma + D, ks);
                    rotate8(x, rr, ks);
                    u32x4 p = pack8<OP_F16>(x);
                    // (here, not where it is used: the values ahead of it take twice the registers)
                    asm volatile("" : "+v"(p));
                    Kf[kb][ks] = inside ? p : mk4(0u, 0u, 0u, 0u);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (rb == 0) {  // uniform over the workgroup: the K' image, pads (zeros) and all
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks)
                        *reinterpret_cast<u32x4*>(image + (16 * kb + i16) * G::KROW + ks * 64 + gsw * 16) = Kf[kb][ks];
                *reinterpret_cast<u32x4*>(image + lane * G::KROW + D * 2) = mk4(0u, 0u, 0u, 0u);
            }
        }

        // scores: sc[kb][r] = query 16 qb + i, key 16 kb + 4 g + r
        u32x4 P[QB][2];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            f32x4 sc[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) sc[kb] = mfma16<OP_F16>(Kf[kb][ks], Qf[qb][ks], sc[kb]);
            }
            if ((j + 1) * kBK > L) {
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        sc[kb][r] = j * kBK + 16 * kb + 4 * g4 + r < L ? sc[kb][r] : -INFINITY;
            }
            float mx = sc[0][0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e >> 2][e & 3]);
            // (finite: a tile has a key, and scores of fp16 operands are finite)
            const float m_new = fmaxf(m_run[qb], max_across_rows16(mx));
            const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
            m_run[qb] = m_new;
            float sum = 0.f;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                float p[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(sc[2 * m + (e >> 2)][e & 3] - m_new);
                    sum += p[e];
                }
                P[qb][m] = mk4(pack2<OP_F16>(p[0], p[1]), pack2<OP_F16>(p[2], p[3]), pack2<OP_F16>(p[4], p[5]),
                               pack2<OP_F16>(p[6], p[7]));
            }
            l_run[qb] = l_run[qb] * alpha + sum;
            if (j != wave) {
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) O[cb][qb][r] *= alpha;
            }
        }
        // O^T += V^T P^T.  The transposing read: of 16 lanes, lane s names 8 bytes of row s / 4, columns 4 (s % 4) .. +
        // 3, and lane i gets column i of the four rows.  Group g takes keys 32 m + 16 g' + 4 g .. + 3 of channels 16 cb
        // .. + 15.
        asm volatile("" ::: "memory");  // (one wavefront's LDS accesses complete in order)
        const uint8_t* const tr = area + (4 * g4 + (i16 >> 2)) * S::VPITCH + (i16 & 3) * 8;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                u32x4 vf;
                uint8_t* const chunk = image + G::K_BYTES + (16 * cb + i16) * G::VROW + gsw * 16;
                if constexpr (RESIDENT) {
                    vf = Vf[cb];
                    if (m == 0) Vf[cb] = *reinterpret_cast<const u32x4*>(chunk + 64);
                } else {
                    const uint8_t* const src = tr + 32 * m * S::VPITCH + cb * 32;
                    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)src));
                    const uint2 hi = __builtin_bit_cast(
                        uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(src + 16 * S::VPITCH)));
                    vf = mk4(lo.x, lo.y, hi.x, hi.y);
                    if (rb == 0) *reinterpret_cast<u32x4*>(chunk + m * 64) = vf;
                }
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) O[cb][qb] = mfma16<OP_F16>(vf, P[qb][m], O[cb][qb]);
            }
        if constexpr (!RESIDENT) {
            if (rb == 0) {
#pragma unroll
                for (int d = 0; d < D; d += 64)
                    *reinterpret_cast<u32x4*>(image + G::K_BYTES + (d + lane) * G::VROW + kBK * 2) =
                        mk4(0u, 0u, 0u, 0u);
            }
        }
        asm volatile("" ::: "memory");
    }

    // ---- the wavefronts' results, put together: sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w ----
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        if (wave >= nt) break;
        const float l = sum_across_rows16(l_run[qb]);
        if (g4 == 0) stats[wave * 16 * QB + 16 * qb + i16] = make_float2(m_run[qb], l);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            *reinterpret_cast<f32x4*>(area + (16 * qb + i16) * S::OPITCH + (16 * cb + 4 * g4) * 4) = O[cb][qb];
    }
    __syncthreads();
    for (int t = tid; t < 16 * QB * (D / 4); t += 64 * kShortWaves) {
        const int r = t / (D / 4), c = t % (D / 4), row = rb * 16 * QB + r;
        float m = -INFINITY;
        for (int w = 0; w < nt; ++w) m = fmaxf(m, stats[w * 16 * QB + r].x);
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < nt; ++w) {
            const float2 ml = stats[w * 16 * QB + r];
            const f32x4 x = *reinterpret_cast<const f32x4*>(smem + w * S::AREA + r * S::OPITCH + c * 16);
            const float f = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - m);
            l = fmaf(f, ml.y, l);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, x[e], o[e]);
        }
        if (row >= L) continue;
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        const int64_t off = (int64_t)b * a.so_b + (int64_t)h * a.so_h + (int64_t)row * a.so_t + 4 * c;
        if (a.out_f32)
            *reinterpret_cast<float4*>(static_cast<float*>(a.out) + off) =
                make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
        else
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + off) =
                make_uint2(pack2<OP_BF16>(o[0] * inv, o[1] * inv), pack2<OP_BF16>(o[2] * inv, o[3] * inv));
        if (a.lse && c == 0)
            a.lse[(int64_t)bh * L + row] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
    }
}

template <int D, int QB, int IN>
hipError_t launch_inst(const AttnArgs& a, const TableArgs& ta, const NormArgs& kn, hipStream_t s) {
    auto kern = attn_short_kernel<D, QB, IN>;
    const int nt = a.nKT < kShortWaves ? a.nKT : kShortWaves;
    constexpr int most = kShortWaves * (ShortGeom<D>::AREA + 16 * QB * 8) + 2 * D * 4 + kShortTable * 8;
    static_assert(most <= 160 * 1024, "LDS of a compute unit");
    const int smem = nt * (ShortGeom<D>::AREA + 16 * QB * 8) + 2 * D * 4 + (IN == 2 ? 0 : ta.total * 8);
    static std::atomic<uint64_t> attr_set{0};
    const hipError_t e = allow_dynamic_lds(kern, most, attr_set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * a.H * a.nQT)), dim3(64 * kShortWaves), smem, s, a, ta, kn);
    return hipGetLastError();
}

template <int D, int QB>
hipError_t launch_rows(const AttnArgs& a, const TableArgs& ta, const NormArgs& kn, bool resident, hipStream_t s) {
    if (resident) return launch_inst<D, QB, 2>(a, ta, kn, s);
    return a.in_f32 ? launch_inst<D, QB, 1>(a, ta, kn, s) : launch_inst<D, QB, 0>(a, ta, kn, s);
}

}  // namespace

hipError_t launch_attn_short(const AttnArgs& a, const TableArgs& ta, const NormArgs& kn, int D, int qb, bool resident,
                             hipStream_t s) {
    if (D == 128 && qb == 1) return launch_rows<128, 1>(a, ta, kn, resident, s);
    if (D == 64)
        return qb == 1 ? launch_rows<64, 1>(a, ta, kn, resident, s) : launch_rows<64, 2>(a, ta, kn, resident, s);
    return hipErrorInvalidValue;
}

}  // namespace dit
