// Memory-bound helper kernels that run before the attention kernel on the same stream:
//  * row_stats_kernel: (cos, sin) of every (axis, position, pair) angle, evaluated in fp64
//    and stored as fp32, so that the rotation itself never calls a transcendental; per-token factors of
//    the q and k rows.
//  * kv_prepack_kernel: rotates K, rounds K' and V once to the MFMA operand types (16-bit, or for
//    K' 8-bit E4M3 with one power-of-two factor per row) and writes each 64-key tile as the exact
//    byte image the attention kernel keeps in LDS (K' rows, then V^T rows with keys permuted into
//    the order the PV product consumes).
#include <type_traits>

#include "dit_attn_device.h"

namespace dit {

// 1/sqrt(mean of x^2 over all H*D channels + eps) of one token row, by one wavefront.  The order of the sum is fixed:
// chunk i (16 bytes of 16-bit rows) belongs to column i % 256, the columns 64 u .. 64 u + 63 are added up pairwise by
// the distances 1, 2, 4 .. 32, then the four sums (0 + 1) + (2 + 3); a lane holds one column of each u.
__device__ __forceinline__ void token_rstd(const RstdArgs& a, int64_t row) {
    if (row >= (int64_t)a.B * a.L) return;
    const int lane = threadIdx.x & 63;
    const int b = (int)(row / a.L), n = (int)(row - (int64_t)b * a.L);
    const int shift = a.D == 128 ? 4 : 3;  // 16-byte chunks per head
    const int chunks = a.H << shift;
    const int64_t base = (int64_t)b * a.s_b + (int64_t)n * a.s_t;
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = lane; i0 < chunks; i0 += 256) {
        float x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 64 * u;
#pragma unroll
            for (int e = 0; e < 8; ++e) x[u][e] = 0.f;
            if (i < chunks) load8(a.x, base + (int64_t)(i >> shift) * a.s_h + 8 * (i & ((1 << shift) - 1)), a.in_f32, x[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) ss[u] = fmaf(x[u][e], x[u][e], ss[u]);
    }
    // lane l ends up with the sum of u = l % 4: two exchanges, then one, where every lane keeps half of what it has
    const bool odd = lane & 1, high = lane & 2;
    float lo = odd ? ss[1] : ss[0], hi = odd ? ss[3] : ss[2];
    lo += __shfl_xor(odd ? ss[0] : ss[1], 1);
    hi += __shfl_xor(odd ? ss[2] : ss[3], 1);
    float tot = high ? hi : lo;
    tot += __shfl_xor(high ? lo : hi, 2);
#pragma unroll
    for (int m = 4; m < 64; m <<= 1) tot += __shfl_xor(tot, m);
    tot += __shfl_xor(tot, 1);
    tot += __shfl_xor(tot, 2);
    if (lane == 0) a.rstd[row] = 1.0f / sqrtf(tot / (float)(a.H * a.D) + a.eps);
}

// What the pre-pack and the attention kernel need before they can start, in one launch: the rotation table (the first
// table_blocks workgroups, one entry a thread) and the per-token factors of the q rows and the k rows (four rows a
// workgroup, one wavefront each).  Memory-bound where there are factors: 32,760 tokens x 12 heads of q and k
// 41 us, 4.9 TB/s (one workgroup of 256 threads per row and three launches: 65).
__global__ void __launch_bounds__(256) row_stats_kernel(const TableArgs t, const RstdArgs q, const RstdArgs k,
                                                        int table_blocks, int q_blocks) {
    const int blk = blockIdx.x;
    const int wave = threadIdx.x >> 6;
    if (blk < table_blocks) {
        const int i = blk * 256 + threadIdx.x;
        if (i < t.total) t.tab[i] = rope_entry(t, i);
    }
    else if (blk < table_blocks + q_blocks) token_rstd(q, (int64_t)(blk - table_blocks) * 4 + wave);
    else token_rstd(k, (int64_t)(blk - table_blocks - q_blocks) * 4 + wave);
}

// any of the three may be null
hipError_t launch_row_stats(const TableArgs* t, const RstdArgs* q, const RstdArgs* k, hipStream_t s) {
    TableArgs ta{};
    RstdArgs qa{}, ka{};
    if (t) ta = *t;
    if (q) qa = *q;
    if (k) ka = *k;
    const int64_t tb = ((int64_t)ta.total + 255) / 256;
    const int64_t qb = ((int64_t)qa.B * qa.L + 3) / 4, kb = ((int64_t)ka.B * ka.L + 3) / 4;
    if (tb + qb + kb == 0) return hipSuccess;
    hipLaunchKernelGGL(row_stats_kernel, dim3((unsigned)(tb + qb + kb)), dim3(256), 0, s, ta, qa, ka, (int)tb, (int)qb);
    return hipGetLastError();
}

// One workgroup per (tile, group of up to kRescaleHeads heads): four lanes a key row.  The lanes of a row first add
// up the heads' shares of the row's sum of squares, each lane every fourth head and then the four partial sums in a
// fixed order, so that every workgroup -- whichever heads it then scales -- arrives at the same factor for a token.
constexpr int kRescaleHeads = 8;
__global__ void __launch_bounds__(256) k_rescale_kernel(const KRescaleArgs a) {
    using G = TileGeom<128>;
    const int groups = (a.H + kRescaleHeads - 1) / kRescaleHeads;
    const int hg = blockIdx.x % groups, j = blockIdx.x / groups;
    const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
    const int tok = j * kBK + r;
    const bool live = tok < a.L;  // slots past the sequence hold zeros and stay as they are
    float ssq = 0.f;
    for (int hh = part; hh < a.H; hh += 4)
        ssq += reinterpret_cast<const float*>(a.tiles + ((size_t)hh * a.nKT + j) * G::TILE_BYTES + kBK * G::KROW)[r];
    ssq += __shfl_xor(ssq, 1);
    ssq += __shfl_xor(ssq, 2);
    const float rs = 1.0f / sqrtf(ssq / (float)(a.H * 128) + a.eps);
    if (!live) return;
    const int h_end = (hg + 1) * kRescaleHeads < a.H ? (hg + 1) * kRescaleHeads : a.H;
    for (int h = hg * kRescaleHeads; h < h_end; ++h) {
        // chunk 4 c + part: the four lanes of a row move 64 contiguous bytes per instruction
        uint8_t* const row = a.tiles + ((size_t)h * a.nKT + j) * G::TILE_BYTES + r * G::KROW + part * 16;
        u32x4 v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = *reinterpret_cast<const u32x4*>(row + c * 64);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float x[8];
            if (a.qk_f16) {
                const uint32_t w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f16x2 p = __builtin_bit_cast(f16x2, w[e]);
                    x[2 * e] = (float)p.x;
                    x[2 * e + 1] = (float)p.y;
                }
            } else {
                widen8(v[c], x);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] *= rs;
            *reinterpret_cast<u32x4*>(row + c * 64) = a.qk_f16 ? pack8<OP_F16>(x) : pack8<OP_BF16>(x);
        }
        // the pad behind the row too, so that the pass leaves no sector partly written (see pack_tile)
        if (part == 3) *reinterpret_cast<u32x4*>(row + 256 - 48) = mk4(0u, 0u, 0u, 0u);
    }
}

hipError_t launch_k_rescale(const KRescaleArgs& a, hipStream_t s) {
    const int groups = (a.H + kRescaleHeads - 1) / kRescaleHeads;
    hipLaunchKernelGGL(k_rescale_kernel, dim3((unsigned)(groups * a.nKT)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// What one workgroup packs: 64 keys of one (batch or request, head).
struct PackTile {
    uint8_t* dst;        // tile image
    int64_t k_off, v_off;  // element offset of key 0 of this sequence for this head
    int key0, key_end;   // keys [key0, key0 + 64) clipped to key_end
    const int* key_src;  // if set: slot r holds key key_src[r] (-1: empty) instead of key0 + r
    // ranges (key counts instead of a mask): slot i = slot0 + r of the tile sequence holds key sa + i if i < la,
    // key sb + (i - la) if i - la < lb, else nothing
    bool ranges;
    int slot0, la, sa, lb, sb;
    RopeGeom rg;         // with this sequence's grid
    int h;               // head (channel weights of the normalisation)
    int64_t stat_off;    // index of key 0 in the per-token normalisation table
};

template <int D, int QK_OP, int PV_OP>
__device__ __forceinline__ void pack_tile(const PackArgs& a, const PackTile& t, uint16_t* vs) {
    using G = TileGeom<D>;
    constexpr int CPR = D / 8;
    constexpr int ROWS_PER_PASS = kThreads / CPR;
    constexpr int NI = kBK / ROWS_PER_PASS;
    constexpr int VS = D + 2;  // padded row of the transposition buffer, in 16-bit elements
    const int tid = threadIdx.x;
    const int c = tid % CPR;

    // All rows of the tile are requested before the first is used: at sizes that leave the chip to a few workgroups
    // each, row by row, was four trips to memory one after the other (4 heads of 6,240 tokens 10.4 -> 9.1 us; 12 heads
    // of 32,760 99 -> 90, 40 heads 284 -> 270).  So are their rotation entries and factors (92 -> 122 registers; 6,240 x
    // 4 9.2 -> 8.5, 3,600 x 40 34.9 -> 32.8, level at 32,760 tokens).
    auto rows = [&](auto f32_tag) __attribute__((always_inline)) {
        constexpr bool F32 = decltype(f32_tag)::value;
        u32x4 rk[NI][F32 ? 2 : 1], rv[NI][F32 ? 2 : 1];
        int keys[NI];
        float2 cs[NI][4];  // rotation entries of the lane's four pairs
        float rstd[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = tid / CPR + i * ROWS_PER_PASS;
            int key;
            if (t.ranges) {
                const int i_ = t.slot0 + r;
                key = i_ < t.la ? t.sa + i_ : (i_ - t.la < t.lb ? t.sb + (i_ - t.la) : -1);
            } else {
                key = t.key_src ? t.key_src[r] : t.key0 + r < t.key_end ? t.key0 + r : -1;
            }
            keys[i] = key;
#pragma unroll
            for (int w = 0; w < (F32 ? 2 : 1); ++w) rk[i][w] = rv[i][w] = mk4(0u, 0u, 0u, 0u);
            if (key >= 0) {
                const int64_t ko = t.k_off + (int64_t)key * a.sk_t + 8 * c, vo = t.v_off + (int64_t)key * a.sv_t + 8 * c;
                const u32x4* const ks = reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(a.k) + ko * (F32 ? 4 : 2));
                const u32x4* const vsrc = reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(a.v) + vo * (F32 ? 4 : 2));
#pragma unroll
                for (int w = 0; w < (F32 ? 2 : 1); ++w) {
                    rk[i][w] = ks[w];
                    rv[i][w] = vsrc[w];
                }
            }
            const int kc = key >= 0 ? key : 0;
            if (a.tab) {
                int pt, ph, pw;
                token_pos(kc, t.rg, pt, ph, pw);
                const RopeRow rr = rope_row(t.rg, pt, ph, pw);
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) cs[i][pp] = rope_one(a.tab, t.rg, rr, 4 * c + pp);
            }
            if (a.kn.mode == 2) rstd[i] = a.kn.rstd[t.stat_off + kc];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = tid / CPR + i * ROWS_PER_PASS;
            const int key = keys[i];
            const bool ok = key >= 0;
            float xk[8], xv[8];
            if constexpr (F32) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    xk[e] = __uint_as_float(rk[i][e >> 2][e & 3]);
                    xv[e] = __uint_as_float(rv[i][e >> 2][e & 3]);
                }
            } else {
                widen8(rk[i][0], xk);
                widen8(rv[i][0], xv);
            }
            if (a.kn.mode) {  // the CPR neighbouring lanes that share a row add up its squares
                float rs;
                if (a.kn.mode == 2) {
                    rs = rstd[i];
                } else {
                    float ss = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) ss = fmaf(xk[e], xk[e], ss);
#pragma unroll
                    for (int m = 1; m < CPR; m <<= 1) ss += __shfl_xor(ss, m);
                    rs = 1.0f / sqrtf(ss * (1.0f / D) + a.kn.eps);
                }
                if (ok) norm8(xk, a.kn, rs, t.h, D, c);
            }
            if (ok) {
                if (a.tab) {
#pragma unroll
                    for (int pp = 0; pp < 4; ++pp) {
                        const float2 y = rotate_pair(xk[2 * pp], xk[2 * pp + 1], cs[i][pp]);
                        xk[2 * pp] = y.x;
                        xk[2 * pp + 1] = y.y;
                    }
                }
            }
            if constexpr (QK_OP == OP_FP8) {
                // one power-of-two factor per key row brings its largest magnitude into [128, 256)
                float am = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) am = fmaxf(am, fabsf(xk[e]));
#pragma unroll
                for (int m = 1; m < CPR; m <<= 1) am = fmaxf(am, __shfl_xor(am, m));
                const int ex = fp8_row_exponent(am);
                const float sc = pow2i(ex);
#pragma unroll
                for (int e = 0; e < 8; ++e) xk[e] *= sc;
                // chunk c = channels [8c, 8c+8) goes where the lane that multiplies it against the same
                // channels of q' finds it: contraction step c / 8, lane half c % 2, slot (c / 2) % 4
                const int off = (c >> 3) * 64 + (c & 1) * 32 + ((c >> 1) & 3) * 8;
                *reinterpret_cast<uint2*>(t.dst + r * G::KROW8 + off) = pack8_fp8(xk);
                if (c == CPR - 1) *reinterpret_cast<u32x4*>(t.dst + r * G::KROW8 + D) = mk4(0u, 0u, 0u, 0u);  // the pad, see below
                if (c == 0) t.dst[G::KSCALE_OFF + r] = (uint8_t)(127 - ex);
            } else {
                // (layout 1: rows 4..11 of every 16 keep their 16-byte chunks in swapped pairs, see below)
                const int cs = a.v_layout ? c ^ (((r >> 2) ^ (r >> 3)) & 1) : c;
                *reinterpret_cast<u32x4*>(t.dst + r * G::KROW + cs * 16) = pack8<QK_OP>(xk);
                // the 16 pad bytes behind the row are written too (zeros): a part is then a run of fully written
                // 32-byte sectors, and none of them has to be read back from memory to be completed
                if (c == CPR - 1) *reinterpret_cast<u32x4*>(t.dst + r * G::KROW + D * 2) = mk4(0u, 0u, 0u, 0u);
            }
            const u32x4 pv = pack8<PV_OP>(xv);
            uint32_t* row = reinterpret_cast<uint32_t*>(vs + r * VS + 8 * c);
            row[0] = pv.x; row[1] = pv.y; row[2] = pv.z; row[3] = pv.w;
        }
    };
    if (a.in_f32) rows(std::true_type{});
    else rows(std::false_type{});
    __syncthreads();

    // V^T chunk (d, kc) = eight key slots, in the order the attention kernel's PV operand wants its keys:
    //  32x32x16 MFMAs (v_layout 0): slot 4g+e holds key 16*(kc/2) + 8g + 4*(kc%2) + e of the tile;
    //  16x16x32 MFMAs (v_layout 1): slot 4g+e holds key 32*(kc/4) + 16g + 4*(kc%4) + e.
#pragma unroll
    for (int i = 0; i < D / 32; ++i) {
        const int d = (tid >> 3) + 32 * i;
        const int kc = tid & 7;
        const int k0 = a.v_layout ? 32 * (kc >> 2) + 4 * (kc & 3) : 16 * (kc >> 1) + 4 * (kc & 1);
        const int kstep = a.v_layout ? 16 : 8;
        uint32_t w[4];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e2 = 0; e2 < 2; ++e2) {
                const int ka = k0 + kstep * g + 2 * e2;
                w[2 * g + e2] = (uint32_t)vs[ka * VS + d] | ((uint32_t)vs[(ka + 1) * VS + d] << 16);
            }
        // Layout 1, both parts: in rows 4..11 of every 16, neighbouring chunks 2n and 2n+1 change places.  A
        // 16x16x32 operand read has lane 16 g + i fetch chunk g of row i, and the LDS serves the 64 lanes of a
        // 128-bit read in four cycles of four lane quads each: quads {0,3,5,6}, {1,2,4,7}, {8,11,13,14},
        // {9,10,12,15} (found by letting two lanes at a time read one bank and watching the conflict counter).
        // With plain rows two lanes of every cycle meet in one bank (every operand read then takes 8 LDS cycles
        // instead of 4); with the swap each cycle's 16 lanes cover the 16 bank groups once.
        const int kcs = a.v_layout ? kc ^ (((d >> 2) ^ (d >> 3)) & 1) : kc;
        *reinterpret_cast<u32x4*>(t.dst + G::K_BYTES + d * G::VROW + kcs * 16) = mk4(w[0], w[1], w[2], w[3]);
        if (kc == 7) *reinterpret_cast<u32x4*>(t.dst + G::K_BYTES + d * G::VROW + kBK * 2) = mk4(0u, 0u, 0u, 0u);
    }
}

// Key padding masks.  Attention does not depend on the order of its keys, so the keys that attend, in ascending order,
// are packed densely into the tiles of their group: padded keys cost no tile, wherever they sit.  Every workgroup finds
// the keys of its own tile: slot r holds the valid key of rank rank0 + r among mask bytes [k0, k1) (src[r], -1: none).
// Returns the number of valid keys.  cnt: one count per 64 keys of the range.  Two small passes ahead of this one, one
// that lists the keys and one that lists the tiles, take 4 to 9 us a call longer where the masks are short or the
// workgroups few; see mask_needs_key_list for where they are the better way.
constexpr int kMaskKeys = 4096;  // the counts are summed up by one wavefront
__device__ __forceinline__ int find_keys(const uint8_t* valid, int k0, int k1, int rank0, int* src, int* cnt) {
    const int tid = threadIdx.x, lane = tid & 63;
    for (int r = tid; r < kBK; r += kThreads) src[r] = -1;
    for (int key0 = k0 + (tid & ~63); key0 < k1; key0 += kThreads) {
        const uint64_t m = __ballot(key0 + lane < k1 && valid[key0 + lane] != 0);
        if (lane == 0) cnt[(key0 - k0) >> 6] = __popcll(m);
    }
    __syncthreads();
    const int groups = (k1 - k0 + 63) >> 6;
    int c = lane < groups ? cnt[lane] : 0, upto = c;  // every wavefront sums up all counts for itself
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const int o = __shfl_up(upto, m);
        if (lane >= m) upto += o;
    }
    const int total = __shfl(upto, 63);
    if (rank0 < total) {
        for (int key0 = k0 + (tid & ~63); key0 < k1; key0 += kThreads) {
            const int g = (key0 - k0) >> 6;
            const int first = __shfl(upto - c, g) - rank0, n = __shfl(c, g);
            if (first >= kBK || first + n <= 0) continue;  // uniform over the wavefront
            const bool ok = key0 + lane < k1 && valid[key0 + lane] != 0;
            const uint64_t m = __ballot(ok);
            const int slot = first + __popcll(m & ((1ull << lane) - 1ull));
            if (ok && slot >= 0 && slot < kBK) src[slot] = key0 + lane;
        }
    }
    __syncthreads();
    return total;
}

// One workgroup per (tile, head, batch).
template <int D, int QK_OP, int PV_OP>
__global__ void __launch_bounds__(kThreads) kv_prepack_kernel(const PackArgs a) {
    using G = TileGeom<D>;
    __shared__ __attribute__((aligned(16))) uint16_t vs[kBK * (D + 2)];
    __shared__ int src[kBK], cnt[kMaskKeys / 64];
    const int tid = threadIdx.x;
    // heads vary fastest: neighbouring workgroups read neighbouring 256-byte pieces of the same 64 tokens
    const int h = blockIdx.x % a.H, jb = blockIdx.x / a.H, j = jb % a.nKT, b = jb / a.nKT;
    PackTile t;
    t.dst = a.tiles + ((size_t)(b * a.H + h) * a.nKT + j) * G::TILE_BYTES;
    t.k_off = (int64_t)b * a.sk_b + (int64_t)h * a.sk_h;
    t.v_off = (int64_t)b * a.sv_b + (int64_t)h * a.sv_h;
    // keys of this tile: [key0, key0 + 64) clipped to key_end (two key groups when split > 0)
    const bool second = a.split > 0 && j >= a.nTA;
    t.key0 = second ? a.split + (j - a.nTA) * kBK : j * kBK;
    t.key_end = (a.split > 0 && !second) ? a.split : a.Lk;
    t.key_src = a.key_src ? a.key_src + ((size_t)b * a.nKT + j) * kBK : nullptr;
    t.ranges = a.kv_len != nullptr;
    t.slot0 = t.la = t.sa = t.lb = t.sb = 0;
    int ca = 0, cb = 0;  // tiles that hold a key, first and second key group (decoupled) or all (joint: ca)
    const bool find = a.valid && !a.key_src;
    if (find) {
        const uint8_t* const valid = a.valid + (size_t)b * a.Lk;
        // whoever writes list entries and counts below needs the other group's number of keys too
        if (h == 0 && a.split > 0) {
            const int other = second ? find_keys(valid, 0, a.split, 0x3fffffff, src, cnt)
                                     : find_keys(valid, a.split, a.Lk, 0x3fffffff, src, cnt);
            (second ? ca : cb) = (other + kBK - 1) / kBK;
        }
        const int mine = find_keys(valid, second ? a.split : 0, t.key_end, (second ? j - a.nTA : j) * kBK, src, cnt);
        (second ? cb : ca) = (mine + kBK - 1) / kBK;
        t.key_src = src;
    } else if (a.tile_mask && !a.key_src && !t.ranges) {  // no mask: all keys
        ca = a.split > 0 ? a.nTA : a.nKT;
        cb = a.nKT - ca;
    }
    if (t.ranges) {
        // counts are clamped to the ranges they count in: whatever the caller wrote, every key index stays inside k, v
        const int end0 = a.split > 0 ? a.split : a.second_start;
        int len0 = a.kv_len[2 * b], len1 = a.kv_len[2 * b + 1];
        len0 = len0 < 0 ? 0 : (len0 > end0 ? end0 : len0);
        len1 = len1 < 0 ? 0 : (len1 > a.Lk - a.second_start ? a.Lk - a.second_start : len1);
        if (a.split > 0) {  // two key groups, each in tiles of its own
            t.slot0 = (second ? j - a.nTA : j) * kBK;
            t.la = second ? len1 : len0;
            t.sa = second ? a.split : 0;
            ca = (len0 + kBK - 1) / kBK;
            cb = (len1 + kBK - 1) / kBK;
        } else {  // one softmax: the second range follows the first densely
            t.slot0 = j * kBK;
            t.la = len0; t.sa = 0; t.lb = len1; t.sb = a.second_start;
            ca = (len0 + len1 + kBK - 1) / kBK;
        }
    }
    t.rg = a.rg;
    t.h = h;
    t.stat_off = (int64_t)b * a.Lk;
    pack_tile<D, QK_OP, PV_OP>(a, t, vs);

    if (a.tile_mask && h == 0 && tid < 64) {
        bool ok;
        if (t.ranges) ok = t.slot0 + tid < t.la + t.lb;
        else ok = t.key_src ? t.key_src[tid] >= 0 : t.key0 + tid < t.key_end;
        const uint64_t m = __ballot(ok);
        if (tid == 0) {
            a.tile_mask[(size_t)b * a.nKT + j] = m;
            if (!a.key_src) {
                // the list of tiles that hold a key and its counts (listed masks: tile_compact_kernel derives them)
                const int jj = second ? j - a.nTA : j;
                if (m != 0ull) a.tile_list[(size_t)b * a.nKT + (second ? ca + jj : jj)] = j;
                if (j == 0) {
                    a.tile_count[b] = ca + cb;
                    if (a.tile_count_a) a.tile_count_a[b] = ca;
                }
            }
        }
    }
}

// Packed requests: one workgroup per (tile of any request, head).
template <int D, int QK_OP, int PV_OP>
__global__ void __launch_bounds__(kThreads) kv_prepack_varlen_kernel(const PackArgs a, const VarlenTable vt) {
    using G = TileGeom<D>;
    __shared__ __attribute__((aligned(16))) uint16_t vs[kBK * (D + 2)];
    const int h = blockIdx.x % a.H, gj = blockIdx.x / a.H;
    int r = 0;
    while (r + 1 < vt.n && gj >= vt.r[r + 1].tile0) ++r;
    const ReqDesc& q = vt.r[r];
    const int j = gj - q.tile0;
    PackTile t;
    t.dst = a.tiles + ((size_t)q.tile0 * a.H + (size_t)h * q.nKT + j) * G::TILE_BYTES;
    t.k_off = (int64_t)q.tok0 * a.sk_t + (int64_t)h * a.sk_h;
    t.v_off = (int64_t)q.tok0 * a.sv_t + (int64_t)h * a.sv_h;
    t.key0 = j * kBK;
    t.key_end = q.L;
    t.key_src = nullptr;
    t.ranges = false;
    t.rg = a.rg;
    t.rg.Hg = q.Hg;
    t.rg.Wg = q.Wg;
    t.h = h;
    t.stat_off = q.tok0;
    pack_tile<D, QK_OP, PV_OP>(a, t, vs);
}

// Where mask_needs_key_list says so: one wavefront per (batch entry, key group) writes the group's valid keys, in
// ascending order, densely into the slots of the group's tiles; the slots left over get -1.
__global__ void __launch_bounds__(64) key_compact_kernel(const uint8_t* valid, int* key_src, int Lk, int nKT,
                                                         int split, int nTA) {
    const int b = blockIdx.x, g = blockIdx.y, lane = threadIdx.x;
    const int k0 = g == 0 ? 0 : split, k1 = (g == 0 && split > 0) ? split : Lk;
    const int t0 = g == 0 ? 0 : nTA, t1 = (g == 0 && split > 0) ? nTA : nKT;
    int* out = key_src + ((size_t)b * nKT + t0) * kBK;
    int count = 0;
    for (int base = k0; base < k1; base += 64) {
        const int key = base + lane;
        const bool ok = key < k1 && valid[(size_t)b * Lk + key] != 0;
        const uint64_t m = __ballot(ok);
        if (ok) out[count + __popcll(m & ((1ull << lane) - 1ull))] = key;
        count += __popcll(m);
    }
    for (int i = count + lane; i < (t1 - t0) * kBK; i += 64) out[i] = -1;
}

// Every workgroup (one per request, head and tile) reads the mask of its key group; past 20 MiB in all that takes
// longer than listing the keys once does.  Whole calls with 64 queries, us, each tile by itself and from the list
// (requests x heads x keys): 1 x 12 x 512 18 and 23, 4 x 12 x 4,096 (12.6 MB read) 85 and 93, 4 x 40 x 2,048 (10.5 MB)
// 96 and 99; at the line 2 x 40 x 4,096 124 and 127, 8 x 40 x 2,048 201 and 199; 16 x 12 x 3,072 (28 MB) 175 and 172,
// 4 x 40 x 4,096 (42 MB) 225 and 210, head_dim 64 16 x 12 x 4,096 (50 MB) 150 and 134.
bool mask_needs_key_list(int B, int H, int Lk, int split) {
    const auto read = [](int64_t keys) { return (keys + kBK - 1) / kBK * keys; };
    return Lk > kMaskKeys || (int64_t)B * H * (read(split) + read(Lk - split)) > (20 << 20);
}

hipError_t launch_key_compact(const PackArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(key_compact_kernel, dim3(a.B, a.split > 0 ? 2 : 1), dim3(64), 0, s, a.valid, a.key_src, a.Lk,
                       a.nKT, a.split, a.nTA);
    return hipGetLastError();
}

// One wavefront per batch entry: tile_list[b] = ascending indices of tiles whose key mask is not empty.
__global__ void __launch_bounds__(64) tile_compact_kernel(const uint64_t* tile_mask, int* tile_list,
                                                          int* tile_count, int* tile_count_a, int nKT, int nTA) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const uint64_t* m = tile_mask + (size_t)b * nKT;
    int* out = tile_list + (size_t)b * nKT;
    int count = 0, count_a = 0;
    for (int base = 0; base < nKT; base += 64) {
        const int t = base + lane;
        const bool keep = t < nKT && m[t] != 0ull;
        const uint64_t votes = __ballot(keep);
        if (keep) out[count + __popcll(votes & ((1ull << lane) - 1ull))] = t;
        count += __popcll(votes);
        count_a += __popcll(__ballot(keep && t < nTA));
    }
    if (lane == 0) {
        tile_count[b] = count;
        if (tile_count_a) tile_count_a[b] = count_a;
    }
}

hipError_t launch_tile_compact(const PackArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(tile_compact_kernel, dim3(a.B), dim3(64), 0, s, a.tile_mask, a.tile_list, a.tile_count,
                       a.tile_count_a, a.nKT, a.nTA);
    return hipGetLastError();
}

template <int D, int QK_OP, int PV_OP>
static hipError_t launch_prepack_inst(const PackArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((kv_prepack_kernel<D, QK_OP, PV_OP>), dim3((unsigned)((int64_t)a.H * a.nKT * a.B)), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prepack_varlen(const PackArgs& a, const VarlenTable& vt, int D, int qk_op, int pv_op, hipStream_t s) {
#define DIT_PACKV_CASE(DD, QK, PV)                                                                        \
    if (D == DD && qk_op == QK && pv_op == PV) {                                                           \
        hipLaunchKernelGGL((kv_prepack_varlen_kernel<DD, QK, PV>), dim3((unsigned)((int64_t)a.H * vt.total_tiles)), dim3(kThreads), 0, \
                           s, a, vt);                                                                      \
        return hipGetLastError();                                                                          \
    }
    DIT_PACKV_CASE(128, OP_F16, OP_F16)
    DIT_PACKV_CASE(128, OP_F16, OP_BF16)
    DIT_PACKV_CASE(128, OP_BF16, OP_F16)
    DIT_PACKV_CASE(128, OP_BF16, OP_BF16)
    DIT_PACKV_CASE(64, OP_F16, OP_F16)
    DIT_PACKV_CASE(64, OP_F16, OP_BF16)
    DIT_PACKV_CASE(64, OP_BF16, OP_F16)
    DIT_PACKV_CASE(64, OP_BF16, OP_BF16)
    DIT_PACKV_CASE(128, OP_FP8, OP_F16)
    DIT_PACKV_CASE(128, OP_FP8, OP_BF16)
    DIT_PACKV_CASE(64, OP_FP8, OP_F16)
    DIT_PACKV_CASE(64, OP_FP8, OP_BF16)
#undef DIT_PACKV_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_prepack(const PackArgs& a, int D, int qk_op, int pv_op, hipStream_t s) {
#define DIT_PACK_CASE(DD, QK, PV) \
    if (D == DD && qk_op == QK && pv_op == PV) return launch_prepack_inst<DD, QK, PV>(a, s);
    DIT_PACK_CASE(128, OP_F16, OP_F16)
    DIT_PACK_CASE(128, OP_F16, OP_BF16)
    DIT_PACK_CASE(128, OP_BF16, OP_F16)
    DIT_PACK_CASE(128, OP_BF16, OP_BF16)
    DIT_PACK_CASE(64, OP_F16, OP_F16)
    DIT_PACK_CASE(64, OP_F16, OP_BF16)
    DIT_PACK_CASE(64, OP_BF16, OP_F16)
    DIT_PACK_CASE(64, OP_BF16, OP_BF16)
    DIT_PACK_CASE(128, OP_FP8, OP_F16)
    DIT_PACK_CASE(128, OP_FP8, OP_BF16)
    DIT_PACK_CASE(64, OP_FP8, OP_F16)
    DIT_PACK_CASE(64, OP_FP8, OP_BF16)
#undef DIT_PACK_CASE
    return hipErrorInvalidValue;
}

}  // namespace dit
