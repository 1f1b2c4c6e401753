// Software-pipelined self-attention forward on 16x16x32 MFMAs (gfx950), the default self-attention kernel.
//
// Same pipeline as attn_pipe_body (dit_attn_fwd_pipe.h): scores of tile j+1 on the matrix cores while tile
// j's softmax runs on the vector ALU, PV of tile j while the maxima of tile j+1 are taken, K'/V^T tile images
// streamed global -> LDS directly, 8 wavefronts in two staggered halves.  What differs is the shape of the
// matrix instruction.  On this chip the board's power limit, not instruction issue, bounds a kernel that keeps
// the matrix cores busy with real data, and v_mfma_f32_16x16x32 delivers 14 % more flops per joule than
// v_mfma_f32_32x32x16 (an MFMA-only loop on random fp16 operands sustains 1,790 against 1,560 TFLOP/s on the
// same board): its dot products are 32 long, so each accumulator element is read and written half as often per
// flop.  The price is twice as many instructions and two query blocks per wavefront that share every K'/V^T
// fragment read from LDS (so the LDS traffic is unchanged).
//
// Layout of v_mfma_f32_16x16x32 (D(16x16) += A(16x32) B(32x16)), lane l = 16 g + i:
//   A: row i, contraction indices 8g .. 8g+7;  B: column i, contraction indices 8g .. 8g+7;
//   C/D: column i, rows 4g .. 4g+3.
// Scores: S^T(key, query) = K' Q'^T with keys on the rows: a lane holds, for each of its two queries
// (16 qb + i), the scores of keys 16 kb + 4g + r (kb = 0..3, r = 0..3) of a 64-key tile: 16 per query.
// The rounded probabilities of key blocks 2m and 2m+1 (8 values) are, in that order, the lane's B operand for the
// 32-key group m of O^T += V^T P^T, and the V^T tile image stores its keys in exactly that order
// (kv_prepack_kernel, V16 layout), so P never moves between lanes.
#pragma once
#include "dit_attn_fwd_pipe.h"

namespace dit {

// The 16x16 results are kept four to a 16-register block (the scores of a query block: quarter kb = key block;
// the output: quarter = channel block within a group of four) and the MFMA works on one quarter of the block.
// Element-wise changes on the rare paths are then sub-register writes of one wide value, which the register
// allocator keeps in place (as separate 4-register values it copied all of them around every branch).
template <int OP>
__device__ __forceinline__ f32x16 mfma16_q(u32x4 a, u32x4 b, f32x16 c, int q) {
    f32x4 x = {c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
    x = mfma16<OP>(a, b, x);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[4 * q + i] = x[i];
    return c;
}
// the same with the accumulator quarter starting from `init`
template <int OP>
__device__ __forceinline__ f32x16 mfma16_q_init(u32x4 a, u32x4 b, f32x4 init, f32x16 c, int q) {
    const f32x4 x = mfma16<OP>(a, b, init);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[4 * q + i] = x[i];
    return c;
}

// Lane (i, g) keeps max over the four lanes (i, 0..3): one swap of neighbouring 16-lane rows, one of the halves.
__device__ __forceinline__ float max_across_rows16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max_across_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}

// The same for a sum (x of (i, g) + x of (i, g ^ 1), then the two halves): no trip through the LDS crossbar.
__device__ __forceinline__ float sum_across_rows16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// NW = wavefronts per workgroup (4 or 8); a wavefront owns QBN (2 or 1) blocks of 16 query rows, the workgroup's
// NW * 16 QBN rows share every K/V tile in LDS.
// QBN = 1: 16 rows a wavefront, for calls whose tiles all fit one round (short_tile_rows).  A fragment read from LDS
// then feeds one MFMA instead of two, which a full chip pays for (14,040 x 12 1,040 -> 1,340 us); but where compute
// units have one workgroup each, what counts is how long its steps take: 128 rows by 8 wavefronts, two a SIMD under
// each other's latencies, instead of 4; 64 rows by 4 where even those fill at most half of the chip.  Whole calls, us,
// 4 x 32 rows, 8 x 16, 4 x 16, (tokens, heads) head_dim 128: 1,600 x 9 44.1, 38.0, 35.5; 640 x 20 29.3, 26.4, 24.2;
// 1,020 x 12 34.3, 30.0, 28.2; 640 x 40 33.9, 29.9, (two rounds) 33.0; 3,600 x 8 75.5, 69.7, (79.3); head_dim 64: 1,600
// x 9 29.5, 25.9, 25.1; 3,600 x 8 51.1, 44.0.  The same bits in all three.  Chained (cross-attention, tiles in one
// round), whole calls: 1,000 queries x 20 heads, 757 keys 27.8 -> 24.0, on resident keys 18.8 -> 15.5; 200 x 40, 769
// keys 31.5 -> 27.0; head_dim 64 19.0 -> 16.8, 21.1 -> 18.9.
// The chained form keeps, behind the tile buffers, one area per wavefront the size of its 32 query rows in 16
// bits.  The rows of the NEXT query tile are copied into it (global -> LDS) while the current one is in its loop;
// at the boundary they are converted into operand registers, and the area then serves as the staging area of the
// output rows (below) before the rows after next are requested.  Held in registers across the store instead, the
// raw rows pushed the operand registers into scratch memory, eight reloads waited for one by one per query tile.
template <int D>
constexpr int chain_stage_bytes() { return 32 * D * 2; }
template <int D, int NW>
constexpr int chain_lds_bytes() { return pipe_lds_bytes<D, NW>() + NW * chain_stage_bytes<D>(); }

// Cache policy (non-temporal) of bytes that are read once: query rows of the chained form at head_dim 128, 32 rows a
// wavefront.  us, cross-attention and the output projection behind it, through the caches and past them: 8,000 x 40, 5
// key tiles 402 and 397, 16,000 x 40 728 and 721, 4 x 32,760 x 40 level; not at head_dim 64 (4 x 128 x 25 22.5, with it
// 22.7) or in calls of one round (4 x 144 x 18 25.0, 25.4).  Key and value rows in the pre-pack, and its tile images:
// level, left as they were.  Output rows: rows_pass_caches.
constexpr int kOnce = 2;

// CHAIN: the workgroup takes pv.qt_count consecutive query tiles of one sequence, one after the other and on into the
// next heads, as ONE stream of key-tile steps: the last step of a query tile multiplies the NEXT one's rows, converted
// just ahead of it, with its first key tile where the other steps multiply the key tile to come, so that between two
// query tiles there is only the store of the output and the first maxima, no first-score stage and no barrier of its
// own, and the two staggered halves stay half a step apart through it (one stores while the other is in its last
// product).  For sequences of a few key tiles (cross-attention: 3 to 13) all this is otherwise as long as the loop.
// Each half has the whole chain as code of its own: where only the key loop was doubled, the registers' roles did not
// agree behind it (660 bytes of spills a lane).  In-kernel stamps, 8 wavefronts, 7.75 key tiles on average: 38,600 ->
// 32,300 clocks a query tile (lock step, first scores and their barrier 3,400 of it -> none).  Whole calls of 4 x
// 32,760 queries x 40 heads 1,622 -> 1,488 us, kernel alone at 1 x 32,760 x 40, 9 key tiles 440 -> 386, 7,800 x 12, 3 key
// tiles 24 -> 22.  What bounds it now, by counters at 4 to 12 key tiles (32,760 x 40): 15,200 clocks a query tile, of
// start and end of the pass, conversion, maxima and store, and 2,480 a key tile, where the matrix cores take 2,048; at
// 8 key tiles they are busy 44 % of the time, the vector ALU 49 %, and wavefronts wait a quarter of theirs.
//
// PIECES: the sequence of keys that pv describes may be a range of the real one (pv.piece >= 0); the workgroup then
// leaves its unnormalised output, running maxima and row sums in piece pv.piece of a.part_o / a.part_ml.
// bf16 score operands can make a score -inf, which a row passes over wherever it has a maximum already; a piece may
// START with a tile of nothing else.  Such a row is `empty` until a tile has a score for it: its scores are taken as
// they are (relative to 0: probabilities, sums and output stay 0) and its first finite maximum, above or below 0,
// moves them whatever the threshold (empty_thr).
//
// TWO (chained): decoupled cross-attention, one softmax over the tiles of each conditioning sequence, their results added.
// A query tile goes through the stream twice: the last step of its first pass multiplies the SAME rows with the first key
// tile of the second sequence, and the first result, normalised, waits as fp16 pairs in the output rows themselves (each
// lane in the row it will write; 16-bit rows, which are as wide) until the last step of the second pass brings
// it into the wavefront's LDS area, free by then.  In registers (the plain kernel's way) there is no room for it here, in
// LDS beside the next rows neither with 8 wavefronts (154 KiB are taken; with 4 there would be).  Row sums in fp32 over the unrounded probabilities, as in the plain kernel.  What the
// form costs beside its steps: a tenth of the call for parking (2 x 32,760 x 12, 11 key tiles: 376 us, without its stores
// and loads 337) and the second pass's first maxima: 23,500 clocks a query tile and 2,670 a key tile.  585 -> 489 us at
// 32,760 queries x 40 heads, 5 + 5 key tiles, resident keys (plain kernel before).  With all of O rewritten before the rows are staged 42 registers spilled: 532.
template <int D, int QK_OP, int PV_OP, int NW, bool CHAIN = false, bool PIECES = false, bool TWO = false, int QBN = 2,
          bool ONCE = false>
__device__ __forceinline__ void attn_pipe16_body(const AttnArgs& a, const PipeView& pv) {
    using G = TileGeom<D>;
    constexpr int NKS = D / 32;        // MFMAs of one score chain
    constexpr int NCB = D / 16;        // 16-channel blocks of the output
    constexpr int NKF = 4 * NKS;       // K' fragments of a tile: (ks, kb), each feeds the QBN query blocks
    constexpr int NVF = 2 * NCB;       // V^T fragments of a tile: (m, cb)
    constexpr int WR = 16 * QBN;  // query rows of a wavefront
    constexpr int BQ = NW * WR;
    constexpr int NI = G::PART_KIB / NW;  // full rounds of wavefront-wide 1 KiB loads per tile part
    static_assert(G::PART_KIB - NW * NI == 2, "two odd pieces per tile part");
    static_assert(QK_OP != OP_FP8, "16-bit score operands only");
    static_assert(QBN == 2 || (!TWO && !PIECES), "one query block a wavefront: whole tiles, one softmax");
    static_assert(!TWO || (CHAIN && D == 128 && QK_OP == OP_F16 && PV_OP == OP_F16),
                  "a pass takes its first maxima as they are: finite scores only; its row sums are those of unrounded probabilities");

    constexpr bool STAG = pipe_staggered<NW>();
    constexpr int VST = STAG ? 3 : 2;  // V^T buffers
    // whole output rows through an LDS area of the wavefront's own (store_rows); 4 wavefronts without a chain keep the room
    // for a second workgroup on the compute unit instead.  8 wavefronts of self-attention stored from the accumulators before;
    // the gain is in the figures of start_q.
    constexpr bool STAGED = CHAIN || NW == 8;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t* const kbuf = smem;  // K buffers 0/1, then the V buffers
    uint8_t* const vbuf = smem + 2 * G::K_BYTES;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g4 = lane >> 4;
    int qt = pv.qt, h = pv.h;
    RopeGeom rg = a.rg;
    rg.Hg = pv.Hg;
    rg.Wg = pv.Wg;

    u32x4 Qf[QBN][NKS];
    uint8_t* const qarea = smem + (2 + VST) * G::K_BYTES + wave * chain_stage_bytes<D>();  // STAGED only
    constexpr int QPR = D / 8;  // 16-byte pieces per 16-bit query row
    // chained form: this wavefront's 32 rows of query tile `qtile` -> its area, piece p of row r in slot
    // p ^ (r % QPR) (the copy fills LDS in lane order, so the swizzle is in which piece a lane fetches)
    // (In the three pieces of code that run once per query tile of a chain -- this copy, the conversion and the
    // store -- every per-lane offset is worked out from a lane number the compiler cannot see through: left to
    // itself it works them all out ahead of the chain, cannot keep them in registers through the key loop, and
    // reloads some seventy of them from scratch memory at every query tile.)
    auto opaque_lane = [&]() {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    auto request_q_lds = [&](int head, int qtile) {
        const int ln = opaque_lane();
        const uint16_t* const q = static_cast<const uint16_t*>(a.q) + (int64_t)pv.b * a.sq_b + (int64_t)head * a.sq_h;
#pragma unroll
        for (int k = 0; k < WR * QPR / 64; ++k) {
            const int r = k * (64 / QPR) + ln / QPR, slot = ln % QPR;
            const int row = qtile * BQ + wave * WR + r;
            const int qr = row < pv.Lq ? row : pv.Lq - 1;
            const uint16_t* src = q + (int64_t)qr * a.sq_t + 8 * (slot ^ (r & (QPR - 1)));
            __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(qarea + k * 1024), 16, 0,
                                             D == 128 && QBN == 2 ? kOnce : 0);
        }
    };
    if constexpr (CHAIN) request_q_lds(h, qt);

    // ---- tile streaming (as in attn_pipe_body): a tile part is PART_KIB pieces of 1 KiB; wavefront w moves
    // pieces w, w+NW, ... of both parts; the two odd pieces of the K part go to wavefronts 0 and 1, those of
    // the V part to wavefronts 2 and 3.
    const uint8_t* const tiles = pv.tiles;  // wavefront-uniform
    int n_steps = TWO ? pv.n_first : pv.nKT;  // of this pass
    int last = n_steps - 1;
    const int tail = pv.Lk - (pv.nKT - 1) * kBK;  // valid keys of the last tile (1..64)
    // past the end: the last tile again
    auto tile_of = [&](int j) -> int { return j < last ? j : last; };
    uint64_t last_mask = 0;  // chained: of the last tile (of the pass)
    auto mask_of = [&](int j) -> uint64_t {
        if constexpr (CHAIN) return j == last ? last_mask : ~0ull;
        else return (j == last && tail < kBK) ? ((1ull << tail) - 1ull) : ~0ull;
    };
    constexpr int NDMA = 2 * NI + 1;
    auto dma_piece = [&](int i, int tk, int kb_, int tv, int vb_, uint32_t lane_off) {
        const uint8_t* ksrc = tiles + (size_t)tk * G::TILE_BYTES;
        const uint8_t* vsrc = tiles + (size_t)tv * G::TILE_BYTES + G::K_BYTES;
        uint8_t* kdst = kbuf + kb_ * G::K_BYTES;
        uint8_t* vdst = vbuf + vb_ * G::V_BYTES;
        if (i < 2 * NI) {
            const int c = (wave + NW * (i >> 1)) * 1024;
            if ((i & 1) == 0) {
                __builtin_amdgcn_global_load_lds((gptr_t)(ksrc + c + lane_off), (lptr_t)(kdst + c), 16, 0, 0);
            } else {
                __builtin_amdgcn_global_load_lds((gptr_t)(vsrc + c + lane_off), (lptr_t)(vdst + c), 16, 0, 0);
            }
        } else if (NW == 4 || wave < 4) {
            const int c = (NW * NI + (wave & 1)) * 1024;
            const uint8_t* osrc = wave < 2 ? ksrc : vsrc;
            uint8_t* odst = wave < 2 ? kdst : vdst;
            __builtin_amdgcn_global_load_lds((gptr_t)(osrc + c + lane_off), (lptr_t)(odst + c), 16, 0, 0);
        }
    };
    auto dma_tiles = [&](int tk, int kb_, int tv, int vb_) {
        // (the empty statement keeps the lane's offset a 32-bit value of this block: known ahead of the loop it is
        // widened there, and every load then adds it to its uniform base on the vector ALU, two registers each)
        uint32_t lane_off = lane * 16;
        asm volatile("" : "+v"(lane_off));
#pragma unroll
        for (int i = 0; i < NDMA; ++i) dma_piece(i, tk, kb_, tv, vb_, lane_off);
    };
    // chained: the stream of key tiles.  Behind the last tile of a query tile comes the first of the next one, which may
    // be of the next head (past the last head of the sequence: the last one again, for loads that nobody uses).  stream_k
    // is the tile whose K' part the next interval requests, stream_v the one before it, whose V^T part it requests.
    int stream_head = 0, stream_k = TWO ? pv.skip_first : 0, stream_v = stream_k;  // tile images, from the chain's first one
    int stream_idx = 0, stream_qt = pv.qt, stream_h = pv.h;
    // (selections, no branches: it runs among the MFMAs)
    auto stream_advance = [&]() {
        stream_v = stream_k;
        ++stream_k;
        ++stream_idx;
        const int wrap = stream_idx >= pv.nKT;  // (a sequence without a key: its first tile again)
        stream_idx = wrap ? 0 : stream_idx;
        stream_qt += wrap;
        const int turn = stream_qt == a.nQT;
        stream_qt = turn ? 0 : stream_qt;
        stream_h += turn;
        stream_head += (turn & (stream_h < a.H)) ? a.nKT : 0;
        if constexpr (TWO) stream_k = stream_head + stream_idx + (stream_idx < pv.n_first ? pv.skip_first : pv.skip_second);
        else stream_k = wrap ? stream_head : stream_k;
    };
    auto dma_wait_and_sync = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    // ---- running state ----
    constexpr int NOG = NCB / 4;  // output blocks of 64 channels: quarter cb % 4 of O[cb / 4]
    f32x16 O[NOG][QBN];
    f32x4 negm[QBN];  // every element = -m_run: the accumulator a score MFMA chain starts from
    float m_run[QBN], l_run[QBN];
    constexpr bool EMPTY_ROWS = PIECES && QK_OP == OP_BF16;
    float empty_thr[2] = {kRescaleThr, kRescaleThr};  // EMPTY_ROWS: -inf while the row is empty
    auto reset_state = [&]() {
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            m_run[qb] = 0.f;
            l_run[qb] = 0.f;
#pragma unroll
            for (int og = 0; og < NOG; ++og)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[og][qb][r] = 0.f;
        }
    };
    reset_state();

    // Rows 4..11 of every 16 hold neighbouring 16-byte chunks in swapped pairs (pack_tile, layout 1): with that,
    // the lanes the LDS serves in one cycle of a 128-bit read fall into distinct banks (plain rows gave two-way
    // conflicts on every operand read).
    const int gsw = g4 ^ (((i16 >> 2) ^ (i16 >> 3)) & 1);
    const int kread_off = i16 * G::KROW + gsw * 16;
    const int vread_off = i16 * G::VROW + gsw * 16;
    // K' fragment f = 4 ks + kb: keys 16 kb .. +15, channels 32 ks .. +31 (the lane: key i, channels 8g .. +7)
    auto k_operand = [&](const uint8_t* kt, int f) {
        return *reinterpret_cast<const u32x4*>(kt + (f & 3) * 16 * G::KROW + (f >> 2) * 64);
    };
    // V^T fragment v = NCB m + cb: channels 16 cb .. +15, key slots 32 m .. +31 (the lane: channel i, slots 8g .. +7)
    auto v_operand = [&](const uint8_t* vt, int v) {
        return *reinterpret_cast<const u32x4*>(vt + (v % NCB) * 16 * G::VROW + (v / NCB) * 64);
    };

    // S^T of one tile from zero (first tile only): S[qb][4 kb + r] = score of key 16 kb + 4 g + r
    auto qk_tile = [&](f32x16 (&S)[QBN], int buf) {
        const uint8_t* kt = kbuf + buf * G::K_BYTES + kread_off;
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) S[qb][r] = 0.f;
#pragma unroll
        for (int f = 0; f < NKF; ++f) {
            const u32x4 ka = k_operand(kt, f);
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) S[qb] = mfma16_q<QK_OP>(ka, Qf[qb][f >> 2], S[qb], f & 3);
        }
    };

    // keys whose mask bit is clear leave the softmax; element 4 kb + r is key 16 kb + 4 g + r of the tile
    auto mask_apply = [&](f32x16 (&S)[QBN], uint64_t mask) {
        const uint64_t mlane = mask >> (4 * g4);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool ok = (mlane >> (16 * kb + r)) & 1ull;
#pragma unroll
                for (int qb = 0; qb < QBN; ++qb) S[qb][4 * kb + r] = ok ? S[qb][4 * kb + r] : -INFINITY;
            }
    };

    // Row maxima of a score tile (relative to m_run once the loop runs), over all four lanes of a row.
    float mx_new[QBN];
    auto row_max = [&](const f32x16 (&S)[QBN]) {
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            float mx = S[qb][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S[qb][r]);
            mx_new[qb] = max_across_rows16(mx);
        }
    };
    // Raise the running maximum of the rows whose pending tile S (relative scores) tops the threshold:
    // m += shift, and everything expressed relative to m moves with it.  mx_new holds full row maxima.
    // The scores and the chain seed are moved ON THE MATRIX CORES: S -= shift is one more accumulation step
    // S += 1 * (-shift) per key block, with an all-ones A operand and a B operand that holds -shift of the
    // lane's query in its first two contraction slots (shift = hi + lo in the operand type) and zeros
    // elsewhere.  Every definition of S in the loop is then an MFMA that
    // accumulates in place; vector-ALU subtractions here made the register allocator give the changed scores
    // new registers and copy all 32 of them on the common path that changes none.
    // hi + lo ends where the operand type does: an fp16 pair holds no shift past 65504 (the row became NaN), a bf16 pair
    // is off by more than the threshold past 2^20, and scores of saturated operands reach 5e11.  A piece of the keys meets
    // such rises wherever it starts, so the forms with pieces, and the chained one, shift by all of it past there, on
    // fp32 MFMAs (an all-ones A operand, -shift in the first contraction slot of B): level in both, while the whole-tile
    // forms, which keep their key loop, took 2 to 5 % longer for what the compiler then made of it.
    auto shift_rows = [&](f32x16 (&S)[QBN]) {
        constexpr uint32_t kOnes = QK_OP == OP_F16 ? 0x3c003c00u : 0x3f803f80u;
        const u32x4 ones = mk4(kOnes, kOnes, kOnes, kOnes);
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            const float thr = EMPTY_ROWS ? empty_thr[qb] : kRescaleThr;
            const float want = mx_new[qb] > thr ? mx_new[qb] : 0.f;
            // hi + lo in the score operand type; what is applied is their exact fp32 sum
            const uint32_t hi_bits = pack2<QK_OP>(want, 0.f) & 0xffffu;
            const float hi = QK_OP == OP_F16 ? (float)__builtin_bit_cast(f16x2, hi_bits)[0] : bf16_lo(hi_bits);
            const uint32_t lo_bits = pack2<QK_OP>(want - hi, 0.f) & 0xffffu;
            const float lo = QK_OP == OP_F16 ? (float)__builtin_bit_cast(f16x2, lo_bits)[0] : bf16_lo(lo_bits);
            constexpr bool WIDE = PIECES || CHAIN;
            const float shift = WIDE && fabsf(want) > (QK_OP == OP_F16 ? 65504.0f : 131072.0f) ? want : hi + lo;
            float alpha = __builtin_amdgcn_exp2f(-shift);
            if constexpr (EMPTY_ROWS) {
                if (empty_thr[qb] != kRescaleThr) alpha = 1.f;  // (nothing to rescale; exp2 may be infinite)
                if (mx_new[qb] > thr) empty_thr[qb] = kRescaleThr;
            }
            m_run[qb] += shift;
            l_run[qb] *= alpha;
            if constexpr (WIDE) {
                const float bsh = g4 == 0 ? -shift : 0.f;
                negm[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, bsh, negm[qb], 0, 0, 0);
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    f32x4 x = {S[qb][4 * kb], S[qb][4 * kb + 1], S[qb][4 * kb + 2], S[qb][4 * kb + 3]};
                    x = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, bsh, x, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) S[qb][4 * kb + r] = x[r];
                }
            } else {
                // B operand: contraction slots 0 and 1 (lanes of row g = 0) = -hi, -lo
                const uint32_t neg = ((hi_bits | (lo_bits << 16)) ^ 0x80008000u);
                const u32x4 bsh = mk4(g4 == 0 ? neg : 0u, 0u, 0u, 0u);
                negm[qb] = mfma16<QK_OP>(ones, bsh, negm[qb]);
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) S[qb] = mfma16_q<QK_OP>(ones, bsh, S[qb], kb);
            }
#pragma unroll
            for (int og = 0; og < NOG; ++og)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[og][qb][r] *= alpha;
        }
    };

#ifndef DIT_PIPE16_LA
#define DIT_PIPE16_LA 6
#endif
    constexpr int LA = DIT_PIPE16_LA;  // LDS fragment reads issued this many fragments ahead of their MFMAs
    constexpr int NCH = 8 * QBN;       // softmax slices: two scores -> one dword of P
    // behind K' fragment f (its QBN score MFMAs) come the slices up to (f + 1) NCH / NKF: one at d128, two at d64 (half
    // as many with one query block); the maxima behind the V^T fragments likewise
    constexpr int CPA = (NCH + NKF - 1) / NKF;
#ifndef DIT_PIPE16_PRE
#define DIT_PIPE16_PRE 3
#endif
    // exp2 of a softmax slice runs this many slices ahead of its pack (at least one fragment's worth)
    constexpr int PRE = DIT_PIPE16_PRE < CPA ? CPA : DIT_PIPE16_PRE;
    static_assert(CPA * NKF >= NCH && PRE >= CPA, "every slice behind a fragment, its exponentials at least one ahead");
    static_assert(LA <= NKF && LA <= NVF, "lookahead too deep");

    const bool late = STAG && wave >= NW / 2;
    auto next_vslot = [](int s) { return s + 1 == VST ? 0 : s + 1; };
    // chained: parity of the number of key-tile steps taken before this query tile (the K' buffers alternate
    // along the whole stream, not per query tile)
    int par = 0;
    auto kslot = [&](int j) -> int {
        if constexpr (CHAIN) return (j + par) & 1;
        else return j & 1;
    };
    auto dma_interval = [&](int j, int vs) {
        if constexpr (CHAIN) {
            dma_tiles(stream_k, kslot(j), stream_v, next_vslot(vs));
            stream_advance();
        } else {
            dma_tiles(tile_of(j + 2), kslot(j), tile_of(j + 1), next_vslot(vs));
        }
    };

    // One pipelined iteration: Sc holds the relative scores of tile j (all <= threshold), Sn receives those of
    // tile j + 1.  vs = j % VST, the buffer V^T(j) sits in.  LATE (compile-time) selects where the barrier sits.
    // MASKED (compile-time): tile j + 1 may be the ragged last tile, or lie past the end.  The loop proper runs
    // the unmasked form; the last iterations of a sequence are separate copies, so that the steady state holds
    // no conditional change of the pending scores at all.  LAST (chained): the last key tile of a query tile; Sn receives
    // the first scores of the next one, from zero, and stays as it is.
    auto iteration = [&](auto late_tag, auto kind_tag, f32x16 (&Sc)[QBN], f32x16 (&Sn)[QBN], int j, int vs) {
        constexpr bool LATE = decltype(late_tag)::value;
        constexpr bool MASKED = decltype(kind_tag)::value == 1;
        constexpr bool LAST = decltype(kind_tag)::value == 2;
        const uint8_t* kt = kbuf + kslot(j + 1) * G::K_BYTES + kread_off;
        const uint8_t* vt = vbuf + vs * G::V_BYTES + vread_off;

        if constexpr (STAG && DIT_PIPE_PRIO == 1) __builtin_amdgcn_s_setprio(1);
        if constexpr (STAG && DIT_PIPE_PRIO == 2) __builtin_amdgcn_s_setprio(0);
        // ---- part A: S(j+1) on MFMA, P(j) and row sums on VALU ----
        u32x4 kf[NKF];
        u32x4 vf[NVF];
#pragma unroll
        for (int f = 0; f < LA; ++f) kf[f] = k_operand(kt, f);
        if constexpr (!LATE) dma_interval(j, vs);

        // slice c = (m, qb, w): dword w of the B operand of key group m for query block qb;
        // w < 2: scores 2w, 2w+1 of key block 2m; w >= 2: scores 2(w-2), 2(w-2)+1 of key block 2m+1
        uint32_t Pd[QBN][2][4];
        float ls[QBN][2];
        constexpr bool PKSUM = PV_OP == OP_F16 && !TWO;  // row sums over the rounded pairs, packed fp16 (see attn_pipe_body)
        f16x2 lsp[QBN][2];
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            ls[qb][0] = ls[qb][1] = 0.f;
            lsp[qb][0] = lsp[qb][1] = f16x2{(_Float16)0.f, (_Float16)0.f};
        }
        auto exp_slice = [&](int c) {
            const int m = c / (4 * QBN), qb = c / 4 % QBN, w = c % 4, e = 4 * (2 * m + (w >> 1)) + 2 * (w & 1);
            Sc[qb][e] = __builtin_amdgcn_exp2f(Sc[qb][e]);
            Sc[qb][e + 1] = __builtin_amdgcn_exp2f(Sc[qb][e + 1]);
        };
        auto pack_slice = [&](int c) {
            const int m = c / (4 * QBN), qb = c / 4 % QBN, w = c % 4, e = 4 * (2 * m + (w >> 1)) + 2 * (w & 1);
            const float e0 = Sc[qb][e], e1 = Sc[qb][e + 1];
            Pd[qb][m][w] = pack2<PV_OP>(e0, e1);
            if constexpr (PKSUM) {
                lsp[qb][w & 1] += __builtin_bit_cast(f16x2, Pd[qb][m][w]);
            } else if constexpr (TWO) {
                l_run[qb] += e0 + e1;
            } else {
                ls[qb][0] += e0;
                ls[qb][1] += e1;
            }
        };
#pragma unroll
        for (int c = 0; c < PRE; ++c) exp_slice(c);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < NKF; ++f) {
            const int ks = f >> 2, kb = f & 3;
            if (f + LA < NKF) kf[f + LA] = k_operand(kt, f + LA);
            // the last fragments of part A fetch the first V^T fragments of part B
            if (f >= NKF - LA) vf[f - (NKF - LA)] = v_operand(vt, f - (NKF - LA));
            Sn[0] = ks == 0 ? mfma16_q_init<QK_OP>(kf[f], Qf[0][ks], negm[0], Sn[0], kb)
                            : mfma16_q<QK_OP>(kf[f], Qf[0][ks], Sn[0], kb);
#pragma unroll
            for (int c = f * NCH / NKF; c < (f + 1) * NCH / NKF; ++c)
                if (c + PRE < NCH) exp_slice(c + PRE);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (QBN == 2)
                Sn[QBN - 1] = ks == 0 ? mfma16_q_init<QK_OP>(kf[f], Qf[QBN - 1][ks], negm[QBN - 1], Sn[QBN - 1], kb)
                                      : mfma16_q<QK_OP>(kf[f], Qf[QBN - 1][ks], Sn[QBN - 1], kb);
#pragma unroll
            for (int c = f * NCH / NKF; c < (f + 1) * NCH / NKF; ++c) pack_slice(c);
            __builtin_amdgcn_sched_barrier(0);
        }

        if constexpr (LATE) {  // the late half's barrier; its loads for the next interval follow at once
            dma_wait_and_sync();
            dma_interval(j + 1, next_vslot(vs));
            __builtin_amdgcn_sched_barrier(0);
        }

        if constexpr (STAG && DIT_PIPE_PRIO == 1) __builtin_amdgcn_s_setprio(0);
        if constexpr (STAG && DIT_PIPE_PRIO == 2) __builtin_amdgcn_s_setprio(1);
        // ---- part B: O += V^T(j) P(j) on MFMA, maxima of S(j+1) on VALU ----
        float pm[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        // slice c of the maxima: the two scores (kb, qb, r..r+1) with c = 8 kb + 4 qb + r / 2 ... any order will do
        auto max_slice = [&](int c) {
            const int kb = c / (2 * QBN), qb = c / 2 % QBN, e = 4 * kb + 2 * (c % 2);
            pm[c & 3] = max3(pm[c & 3], Sn[qb][e], Sn[qb][e + 1]);
        };
#pragma unroll
        for (int v = 0; v < NVF; ++v) {
            const int m = v / NCB, cb = v % NCB;
            if (v + LA < NVF) vf[v + LA] = v_operand(vt, v + LA);
            const auto& P0 = Pd[0][m];
            O[cb / 4][0] = mfma16_q<PV_OP>(vf[v], mk4(P0[0], P0[1], P0[2], P0[3]), O[cb / 4][0], cb % 4);
            // the first fragment leaves the last score MFMAs time to retire
            if (v >= 1) {
#pragma unroll
                for (int c = (v - 1) * NCH / NVF; c < v * NCH / NVF; ++c) max_slice(c);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (QBN == 2) {
                const auto& P1 = Pd[QBN - 1][m];
                O[cb / 4][QBN - 1] =
                    mfma16_q<PV_OP>(vf[v], mk4(P1[0], P1[1], P1[2], P1[3]), O[cb / 4][QBN - 1], cb % 4);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int c = (NVF - 1) * NCH / NVF; c < NCH; ++c) max_slice(c);
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            if constexpr (PKSUM) {
                const f16x2 t2 = lsp[qb][0] + lsp[qb][1];
                l_run[qb] += (float)t2[0] + (float)t2[1];
            } else if constexpr (!TWO) {
                l_run[qb] += ls[qb][0] + ls[qb][1];
            }
            asm volatile("" : "+v"(l_run[qb]));  // keeps the row-sum chain here (it would sink past the barrier)
        }
        // Common case: no score of the pending tile tops the threshold in ANY lane, which needs no exchange
        // between lanes at all; the full row maxima are only formed on the rare paths below.
        bool need;
        if constexpr (EMPTY_ROWS)  // (pm[0], pm[1]: query block 0)
            need = __any(fmaxf(pm[0], pm[1]) > empty_thr[0] || fmaxf(pm[2], pm[3]) > empty_thr[1]);
        else
            need = __any(fmaxf(fmaxf(pm[0], pm[1]), fmaxf(pm[2], pm[3])) > kRescaleThr);
        if constexpr (!LATE) dma_wait_and_sync();
        if constexpr (LAST) return;
        if constexpr (MASKED) {
            const uint64_t mnext = mask_of(j + 1);
            // A ragged tile takes the rescale path whatever its maxima say.  It need not (the maxima above were
            // taken before the mask: they can only call for a shift that is not needed, never miss one, and a masked
            // score is -inf, which every path below takes as it is), and the chained form, where the ragged tile is
            // one in eight, does not; the other forms keep the assignment: without it the compiler lays their key
            // loop out differently, instruction for instruction the same and 8 % slower on all-zero inputs.
            if (mnext != ~0ull) {
                mask_apply(Sn, mnext);
                if constexpr (!CHAIN) need = true;
            }
            // after the last tile these are scores of a stale buffer: never let them touch the state
            if constexpr (!CHAIN) need = need && j < last;
        }
        // (rows whose maximum stays under the threshold are shifted by zero)
        if (need) {
            row_max(Sn);
            shift_rows(Sn);
        }
    };

    // ---- prologue: tiles 0 (K, V) and 1 (K) start streaming, then Q is converted while they fly ----
    auto first_tiles = [&]() {
        if constexpr (CHAIN) {
            dma_tiles(stream_k, 0, stream_v, 0);  // (there if the sequence has no key too: read and not used)
            stream_advance();
            dma_tiles(stream_k, 1, stream_v, 1);  // (its V part: as below)
            stream_advance();
        } else if (n_steps > 0) {
            const int t1 = last > 0 ? 1 : 0;
            dma_tiles(0, 0, 0, 0);
            dma_tiles(t1, 1, 0, 1);  // K'(1); its V part lands in a buffer iteration 0 refills anyway
        }
    };
    // Query rows -> operand registers: normalise, rotate, fold scale*log2(e), round once (not the chained form, see
    // convert_q_area).  Rows, rotation entries and the per-token factor are requested before the first tiles, in one
    // go, and the arithmetic is one straight line per input type.  What bounds this stage is instructions and gathers
    // (two wavefronts per SIMD, four clocks an instruction, and some thirty clocks of the address unit a gather): with
    // a test of the input type, the normalisation and the rotation around every 16 bytes and a compare-and-select
    // saturation a workgroup of 8 wavefronts took 17,800 clocks from its start to its first scores (21,000 with the
    // normalisation), now 15,300 (16,700); 123.3 -> 119.5 us at 6,240 tokens x 4 heads, 333 -> 328 us at
    // 3,600 tokens x 40 heads, long sequences level.  Rotation entries two pairs a load (was one), the
    // pre-pack's requested ahead and, with 8 wavefronts, whole output rows at the end, whole calls, all three: 6,240 x 4
    // 100.0 -> 97.9 us, 3,600 x 40 318.6 -> 311.6, five packed requests x 12 3,997 -> 3,892, 32,760 x 12 5,139 -> 5,088, toy
    // grids level.
    auto start_q = [&](auto f32_tag) {
        constexpr bool F32 = decltype(f32_tag)::value;
        u32x4 raw[QBN][NKS][F32 ? 2 : 1];
        float2 cs[QBN][NKS][4];  // (cos, sin) of the lane's channel pairs at the row's position
        float2 edge[QBN][2];
        float rs[2] = {1.f, 1.f};
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            const int row = qt * BQ + wave * WR + qb * 16 + i16;
            const int qr = row < pv.Lq ? row : pv.Lq - 1;
            const int64_t base = pv.q_off + (int64_t)qr * a.sq_t + 8 * g4;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                if constexpr (F32) {
                    const u32x4* const src = reinterpret_cast<const u32x4*>(static_cast<const float*>(a.q) + base + 32 * ks);
                    raw[qb][ks][0] = src[0];
                    raw[qb][ks][1] = src[1];
                } else {
                    raw[qb][ks][0] = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.q) + base + 32 * ks);
                }
            }
            int pt, ph, pw;
            token_pos(qr, rg, pt, ph, pw);
            const RopeRow rr = rope_row(rg, pt, ph, pw);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int pp = 0; pp < 4; pp += 2) rope_two(a.tab, rg, rr, 16 * ks + 4 * g4 + pp, &cs[qb][ks][pp]);
            rope_edges(a.tab, rg, rr, edge[qb]);
            if (a.qn.mode == 2) rs[qb] = a.qn.rstd[pv.stat_off + qr];
        }
        first_tiles();
        float x[QBN][NKS][8];
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[qb][ks][e] = __uint_as_float(raw[qb][ks][e >> 2][e & 3]);
                } else {
                    widen8(raw[qb][ks][0], x[qb][ks]);
                }
            }
        if (a.qn.mode) {
            if (a.qn.mode == 1) {  // a row's channels are read by the four lanes (i, 0..3)
#pragma unroll
                for (int qb = 0; qb < QBN; ++qb) {
                    float ss = 0.f;
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                        for (int e = 0; e < 8; ++e) ss = fmaf(x[qb][ks][e], x[qb][ks][e], ss);
                    rs[qb] = 1.0f / sqrtf(sum_across_rows16(ss) * (1.0f / D) + a.qn.eps);
                }
            }
            float4 g[NKS][2];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) g[ks][0] = g[ks][1] = make_float4(1.f, 1.f, 1.f, 1.f);
            if (a.qn.gamma) {
                const float4* const src = reinterpret_cast<const float4*>(a.qn.gamma + (int64_t)pv.h * D + 8 * g4);
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    g[ks][0] = src[8 * ks];
                    g[ks][1] = src[8 * ks + 1];
                }
            }
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float4 ge = g[ks][e >> 2];
                        const float w = (e & 3) == 0 ? ge.x : (e & 3) == 1 ? ge.y : (e & 3) == 2 ? ge.z : ge.w;
                        x[qb][ks][e] *= rs[qb] * w;
                    }
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {  // (uniform: only the group of 16 pairs that holds an odd boundary is looked at)
            const int h0 = rg.hd[0], h01 = rg.hd[0] + rg.hd[1];
            if (((h0 & 1) && (h0 >> 4) == ks) || ((h01 & 1) && (h01 >> 4) == ks)) {
#pragma unroll
                for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
                    for (int pp = 0; pp < 4; pp += 2) rope_mend(rg, edge[qb], 16 * ks + 4 * g4 + pp, &cs[qb][ks][pp]);
            }
        }
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                float y[8];
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) {
                    const float2 r = rotate_pair(x[qb][ks][2 * pp], x[qb][ks][2 * pp + 1], cs[qb][ks][pp]);
                    y[2 * pp] = r.x * a.qscale;
                    y[2 * pp + 1] = r.y * a.qscale;
                }
                Qf[qb][ks] = pack8<QK_OP>(y);
            }
    };
    if constexpr (CHAIN) {
        first_tiles();
    } else {
        if (a.in_f32) start_q(std::true_type{});
        else start_q(std::false_type{});
    }

    constexpr std::integral_constant<int, 0> plain{};  // kinds of iteration
    constexpr std::integral_constant<int, 1> masked{};
    constexpr std::integral_constant<int, 2> last_of_tile{};
    // chained form: the rows of query tile `qtile` in this wavefront's area -> operand registers.  It takes 16-bit
    // query rows (the host sends fp32 rows and rotations to the other kernels): widen, normalise if asked to, scale,
    // round.  A row's four lanes (i, 0..3) hold its channels; the per-head statistic is their sum, the per-token one
    // comes from the table.
    auto convert_q_area = [&](int head, int qtile) {
        const int ln = opaque_lane();
        auto chunk = [&](int qb, int ks, float x[8]) {
            const int r = 16 * qb + (ln & 15);
            widen8(*reinterpret_cast<const u32x4*>(qarea + r * (D * 2) + (((4 * ks + (ln >> 4)) ^ (r & (QPR - 1))) << 4)), x);
        };
        float rs[2] = {1.f, 1.f};
        if (a.qn.mode == 2) {
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) {
                const int row = qtile * BQ + wave * WR + 16 * qb + (ln & 15);
                rs[qb] = a.qn.rstd[pv.stat_off + (row < pv.Lq ? row : pv.Lq - 1)];
            }
        } else if (a.qn.mode == 1) {
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) {
                float ss = 0.f;
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    float x[8];
                    chunk(qb, ks, x);
#pragma unroll
                    for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
                }
                rs[qb] = 1.0f / sqrtf(sum_across_rows16(ss) * (1.0f / D) + a.qn.eps);
            }
        }
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                float x[8];
                chunk(qb, ks, x);
                if (a.qn.mode) norm8(x, a.qn, rs[qb], head, D, 4 * ks + (ln >> 4));
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] *= a.qscale;
                Qf[qb][ks] = pack8<QK_OP>(x);
            }
    };
    // two softmaxes: the first result of query tile (h, qt) -> the output rows: the lane's 8 channels of blocks 2k, 2k + 1 go to
    // 16-byte piece 4k + g of its row, and from there into its own 16 bytes of LDS piece (qb, k)
    constexpr int NPK = D / 32;
    auto park_piece = [&](int ln, int qb, int k, bool& inside) -> uint8_t* {
        const int row = qt * BQ + wave * WR + 16 * qb + (ln & 15);
        inside = row < pv.Lq;
        const int64_t off = (int64_t)pv.b * a.so_b + (int64_t)h * a.so_h + (int64_t)(inside ? row : pv.Lq - 1) * a.so_t;
        return static_cast<uint8_t*>(a.out) + off * 2 + k * 64 + (ln >> 4) * 16;
    };
    auto park_rows = [&]() __attribute__((always_inline)) {
        const int ln = opaque_lane();
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            const float l = sum_across_rows16(l_run[qb]);
            const float inv = l > 0.f ? 1.0f / l : 0.f;
            bool inside;
            uint8_t* const dst = park_piece(ln, qb, 0, inside);
            if (inside) {
#pragma unroll
                for (int k = 0; k < NPK; ++k) {
                    uint32_t w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int cb = 2 * k + (i >> 1), e = 4 * (cb % 4) + 2 * (i & 1);
                        w[i] = pack2<OP_F16>(O[cb / 4][qb][e] * inv, O[cb / 4][qb][e + 1] * inv);
                    }
                    *reinterpret_cast<u32x4*>(dst + k * 64) = mk4(w[0], w[1], w[2], w[3]);
                }
            }
        }
    };
    auto request_parked = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows that the area held have been read
        const int ln = opaque_lane();
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            bool inside;
            const uint8_t* const src = park_piece(ln, qb, 0, inside);  // (past the end: some row, not used)
#pragma unroll
            for (int k = 0; k < NPK; ++k)
                __builtin_amdgcn_global_load_lds((gptr_t)(src + k * 64), (lptr_t)(qarea + (qb * NPK + k) * 1024), 16, 0, 0);
        }
    };
    if constexpr (!CHAIN) {
    if (n_steps > 0) {
        // scores of tile 0 become the first running maximum
        dma_wait_and_sync();
        f32x16 S0[QBN], S1[QBN];
        qk_tile(S0, kslot(0));
        __syncthreads();  // every wavefront has read K'(0) before iteration 0 streams K'(2) over it
        if constexpr (STAG) {
            if (late) dma_interval(0, 0);
        }
        if (mask_of(0) != ~0ull) mask_apply(S0, mask_of(0));
        row_max(S0);  // finite: a sequence has at least one key
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            m_run[qb] = mx_new[qb];
            if constexpr (EMPTY_ROWS) {
                if (mx_new[qb] == -INFINITY) {
                    m_run[qb] = 0.f;
                    empty_thr[qb] = -INFINITY;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) negm[qb][r] = -m_run[qb];
#pragma unroll
            for (int r = 0; r < 16; ++r) S0[qb][r] -= m_run[qb];
        }

        auto key_loop = [&](auto late_tag) {
            int j = 0, vs = 0;
            // iteration j produces the scores of tile j + 1: unmasked while j + 1 < last
            for (; j + 3 < n_steps; j += 2) {
                iteration(late_tag, plain, S0, S1, j, vs);
                vs = next_vslot(vs);
                iteration(late_tag, plain, S1, S0, j + 1, vs);
                vs = next_vslot(vs);
            }
            // the last one to three iterations
            if (j < n_steps) {
                iteration(late_tag, masked, S0, S1, j, vs);
                vs = next_vslot(vs);
                ++j;
            }
            if (j < n_steps) {
                iteration(late_tag, masked, S1, S0, j, vs);
                vs = next_vslot(vs);
                ++j;
            }
            if (j < n_steps) {
                iteration(late_tag, masked, S0, S1, j, vs);
                vs = next_vslot(vs);
            }
        };
        if (late) {
            key_loop(std::true_type{});
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
            key_loop(std::false_type{});
        }
    }

    }
    // ---- epilogue: the lane holds channels 16 cb + 4 g + r of its two queries ----
    auto store_rows = [&](bool parked) __attribute__((always_inline)) {
        // Stored from the accumulators a wavefront instruction writes sixteen 32-byte pieces of sixteen rows; with
        // an output as large as the input and a loop of eight steps that was a third of a query tile's time.  The
        // wavefront passes its 32 rows through a staging area of its own behind the tile buffers, STG bytes at a
        // time, and stores whole rows, 16 bytes a lane (pieces of a staged row swizzled with the row number).
        constexpr int STG = chain_stage_bytes<D>();
        uint8_t* const region = qarea;
        const int ln = opaque_lane();
        const int li = ln & 15, lg = ln >> 4;
        float inv[QBN];
#pragma unroll
        for (int qb = 0; qb < QBN; ++qb) {
            const float l = sum_across_rows16(l_run[qb]);
            inv[qb] = l > 0.f ? 1.0f / l : 0.f;
            const int row = qt * BQ + wave * WR + qb * 16 + li;
            if (a.lse && lg == 0 && row < pv.Lq) {
                const float v = l > 0.f ? (m_run[qb] + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
                a.lse[CHAIN ? ((int64_t)pv.b * a.H + h) * a.Lq + row : pv.lse_off + row] = v;
            }
        }
        const int64_t o_off = CHAIN ? (int64_t)pv.b * a.so_b + (int64_t)h * a.so_h : pv.o_off;
        auto stage_and_store = [&](auto es_tag) {
            constexpr int ES = decltype(es_tag)::value;  // bytes per output element
            constexpr int RB = D * ES;                   // bytes per staged row
            constexpr int PR = RB / 16;                  // 16-byte pieces per row
            constexpr int RPP = STG / RB < 16 ? STG / RB : 16;  // rows per pass: at most one 16-row block
            static_assert(RPP >= 1 && 16 % RPP == 0 && PR <= 64 && 64 % PR == 0 && (RPP * RB) % 1024 == 0,
                          "staging geometry");
            const int row0 = qt * BQ + wave * WR;
            const bool full = row0 + WR <= pv.Lq;  // wavefront-uniform
            // the first softmax's result, zero without one: read block by block before rows are staged over it (16 staged rows
            // take only the half of the area that held theirs)
            static_assert(!TWO || RPP * RB <= STG / 2, "the second block's first result stays in place");
            u32x4 first[TWO ? 2 : 1][TWO ? NPK : 1];
            auto read_first = [&](int qb) {
#pragma unroll
                for (int k = 0; k < NPK; ++k) {
                    first[qb][k] = *reinterpret_cast<const u32x4*>(region + (qb * NPK + k) * 1024 + ln * 16);
                    if (!parked) first[qb][k] = mk4(0u, 0u, 0u, 0u);
                }
                asm volatile("" ::: "memory");
            };
#pragma unroll
            for (int pass = 0; pass < WR / RPP; ++pass) {
                const int qb = pass * RPP / 16;
                if constexpr (TWO) read_first(qb);
                auto value = [&](int cb, int e) {
                    if constexpr (TWO) {
                        const uint32_t pair = first[qb][cb / 2][2 * (cb & 1) + (e >> 1)];  // (bit_cast of the element itself reads element 0)
                        const f16x2 t = __builtin_bit_cast(f16x2, pair);
                        return O[cb / 4][qb][4 * (cb % 4) + e] * inv[qb] + (float)t[e & 1];
                    } else {
                        return O[cb / 4][qb][4 * (cb % 4) + e] * inv[qb];
                    }
                };
                const int rr = li - (pass * RPP) % 16;  // this lane's row within the pass, if it has one
                if (rr >= 0 && rr < RPP) {
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const float o0 = value(cb, 0), o1 = value(cb, 1), o2 = value(cb, 2), o3 = value(cb, 3);
                        const int col = (16 * cb + 4 * lg) * ES;
                        uint8_t* const dst = region + rr * RB + (((col >> 4) ^ (rr & (PR - 1))) << 4) + (col & 15);
                        if constexpr (ES == 4) *reinterpret_cast<float4*>(dst) = make_float4(o0, o1, o2, o3);
                        else *reinterpret_cast<uint2*>(dst) = make_uint2(pack2<OP_BF16>(o0, o1), pack2<OP_BF16>(o2, o3));
                    }
                }
                // all of a pass's pieces are read back before the first is stored, and a tile that lies inside the
                // sequence stores without a row test: with a test per store each read sat in a branch of its own
                // and was waited for there, sixteen LDS round trips one after the other per query tile
                constexpr int NK = RPP * RB / 1024;
                static_assert(NK == 2 || NK % 4 == 0, "pieces are read back two or four at a time");
                u32x4 v[NK];
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    const int r = k * (64 / PR) + ln / PR, pc = ln % PR;
                    v[k] = *reinterpret_cast<const u32x4*>(region + r * RB + ((pc ^ (r & (PR - 1))) << 4));
                }
                // (four values the compiler must hold at once: left alone it sinks each read to its store)
                if constexpr (NK == 2) {
                    asm volatile("" : "+v"(v[0]), "+v"(v[1])::"memory");
                } else {
#pragma unroll
                    for (int k = 0; k < NK; k += 4)
                        asm volatile("" : "+v"(v[k]), "+v"(v[k + 1]), "+v"(v[k + 2]), "+v"(v[k + 3])::"memory");
                }
                uint8_t* const obase = static_cast<uint8_t*>(a.out) +
                                       (o_off + (int64_t)(row0 + pass * RPP + ln / PR) * a.so_t) * ES + (ln % PR) * 16;
                const int64_t kstride = (int64_t)(64 / PR) * a.so_t * ES;
                auto put = [&](int k) {
                    u32x4* const dst = reinterpret_cast<u32x4*>(obase + k * kstride);
                    if constexpr (ONCE) __builtin_nontemporal_store(v[k], dst);
                    else *dst = v[k];
                };
                if (full) {
#pragma unroll
                    for (int k = 0; k < NK; ++k) put(k);
                } else {
#pragma unroll
                    for (int k = 0; k < NK; ++k)
                        if (row0 + pass * RPP + k * (64 / PR) + ln / PR < pv.Lq) put(k);
                }
            }
        };
        if constexpr (TWO || ONCE) {
            stage_and_store(std::integral_constant<int, 2>());
        } else {
            if (a.out_f32) stage_and_store(std::integral_constant<int, 4>());
            else stage_and_store(std::integral_constant<int, 2>());
        }
    };
    if constexpr (CHAIN) {
    // query tiles of the chain, and the one after (h, qt)
    const int n_qt = pv.qt_count;
    int next_h = h, next_qt = qt;
    auto next_tile = [&]() {
        if (++next_qt == a.nQT) {
            next_qt = 0;
            ++next_h;
        }
    };
    auto query_tiles = [&](auto late_tag) __attribute__((always_inline)) {
        constexpr bool LATE = decltype(late_tag)::value;
        f32x16 S0[QBN], S1[QBN];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // rows and first tiles
        convert_q_area(h, qt);
        next_tile();
        if (n_qt > 1) request_q_lds(next_h, next_qt);
        __syncthreads();
        qk_tile(S0, 0);
        __syncthreads();  // every wavefront has read K'(0) before iteration 0 streams K'(2) over it
        if constexpr (LATE) dma_interval(0, 0);
        const uint64_t* const masks = a.tile_mask + (size_t)pv.b * a.nKT;
        const uint64_t mask_first = masks[TWO ? pv.skip_first + last : last];
        uint64_t mask_second = 0;
        if constexpr (TWO) mask_second = masks[pv.skip_second + pv.nKT - 1];
        last_mask = mask_first;
        int vs = 0, left = n_qt;
        bool second = false;  // two softmaxes: this pass is over the second sequence, the first result is parked
        while (left > 0) {
            // S0 = scores of the first key tile, from zero: they become the first running maximum
            if (mask_of(0) != ~0ull) mask_apply(S0, mask_of(0));
            row_max(S0);
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb) {
                m_run[qb] = mx_new[qb];
#pragma unroll
                for (int r = 0; r < 4; ++r) negm[qb][r] = -m_run[qb];
#pragma unroll
                for (int r = 0; r < 16; ++r) S0[qb][r] -= m_run[qb];
            }
            int j = 0;
            for (; j + 3 < n_steps; j += 2) {
                iteration(late_tag, plain, S0, S1, j, vs);
                vs = next_vslot(vs);
                iteration(late_tag, plain, S1, S0, j + 1, vs);
                vs = next_vslot(vs);
            }
            // two to go from here, the scores of the last one in S1 (copies, so that the registers' roles agree)
            if (j + 3 == n_steps) {
                iteration(late_tag, plain, S0, S1, j, vs);
                vs = next_vslot(vs);
                ++j;
#pragma unroll
                for (int qb = 0; qb < QBN; ++qb) S0[qb] = S1[qb];
            }
            if (j + 2 == n_steps) {
                iteration(late_tag, masked, S0, S1, j, vs);
                vs = next_vslot(vs);
                ++j;
            } else {
#pragma unroll
                for (int qb = 0; qb < QBN; ++qb) S1[qb] = S0[qb];
            }
            const bool again = TWO && !second && pv.n_first < pv.nKT;  // the second sequence follows, same rows
            if (!again && left > 1) {  // the rows of the next query tile (the last one's first scores are not used)
                // (with two key tiles or more the copy has been waited for at a barrier)
                if (pv.nKT == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                convert_q_area(next_h, next_qt);
            }
            if constexpr (TWO) {
                if (second) {  // (in the area at the barrier of the step below)
                    if (n_steps == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // its rows are written
                    request_parked();
                }
            }
#pragma unroll
            for (int qb = 0; qb < QBN; ++qb)
#pragma unroll
                for (int r = 0; r < 4; ++r) negm[qb][r] = 0.f;
            iteration(late_tag, last_of_tile, S1, S0, j, vs);
            vs = next_vslot(vs);
            par ^= n_steps & 1;
            if (again) {
                park_rows();
            } else {
                store_rows(second);
                h = next_h;
                qt = next_qt;
                --left;
                if (left > 1) {
                    next_tile();
                    request_q_lds(next_h, next_qt);
                }
            }
            if constexpr (TWO) {
                second = again;
                n_steps = again ? pv.nKT - pv.n_first : pv.n_first;
                last = n_steps - 1;
                last_mask = again ? mask_second : mask_first;
            }
            reset_state();
        }
        if constexpr (LATE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    if (n_steps > 0) {
        if constexpr (STAG) {
            if (late) query_tiles(std::true_type{});
            else query_tiles(std::false_type{});
        } else {
            query_tiles(std::false_type{});
        }
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the first rows, into the area the store stages in
        next_tile();
        for (int it = 0; it < n_qt; ++it) {
            store_rows(false);
            h = next_h;
            qt = next_qt;
            next_tile();
        }
    }
    } else {
    const int ln = opaque_lane();  // (nothing of the epilogue's addresses is held through the key loop)
    const int li = ln & 15, lg = ln >> 4;
#pragma unroll
    for (int qb = 0; qb < QBN; ++qb) {
        const int row = qt * BQ + wave * WR + qb * 16 + li;
        float l = l_run[qb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if constexpr (PIECES) {
            if (pv.piece >= 0) {  // in the lanes' own order: 1 KiB of consecutive bytes per store
                const int64_t blk = ((int64_t)pv.piece * NW + wave) * 2 + qb;
                float4* const dst = reinterpret_cast<float4*>(a.part_o) + blk * NCB * 64 + ln;
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) {
                    const int e = 4 * (cb % 4);
                    dst[cb * 64] = make_float4(O[cb / 4][qb][e], O[cb / 4][qb][e + 1], O[cb / 4][qb][e + 2],
                                               O[cb / 4][qb][e + 3]);
                }
                const bool empty = EMPTY_ROWS && empty_thr[qb] != kRescaleThr;
                if (lg == 0) a.part_ml[blk * 16 + li] = make_float2(empty ? -INFINITY : m_run[qb], l);
                continue;
            }
        }
        if constexpr (STAGED) continue;
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        if (row < pv.Lq) {
            const int64_t obase = pv.o_off + (int64_t)row * a.so_t;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                const int d0 = 16 * cb + 4 * lg;
                const int e = 4 * (cb % 4);
                const float o0 = O[cb / 4][qb][e] * inv, o1 = O[cb / 4][qb][e + 1] * inv;
                const float o2 = O[cb / 4][qb][e + 2] * inv, o3 = O[cb / 4][qb][e + 3] * inv;
                if (a.out_f32) {
                    *reinterpret_cast<float4*>(static_cast<float*>(a.out) + obase + d0) = make_float4(o0, o1, o2, o3);
                } else {
                    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + obase + d0) =
                        make_uint2(pack2<OP_BF16>(o0, o1), pack2<OP_BF16>(o2, o3));
                }
            }
            if (a.lse && lg == 0) {
                const float v = l > 0.f ? (m_run[qb] + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
                a.lse[pv.lse_off + row] = v;
            }
        }
    }
    if constexpr (STAGED) {
        if (!PIECES || pv.piece < 0) store_rows(false);
    }
    }
}

// One sequence per batch entry, all of the same length.
template <int D, int QK_OP, int PV_OP, int NW, int QBN>
__global__ void __launch_bounds__(64 * NW, 2) attn_fwd_pipe16_kernel(const AttnArgs a) {
    const int logical = xcd_contiguous_block();
    PipeView pv;
    const int bh = logical / a.nQT;
    pv.qt = logical % a.nQT;
    pv.b = bh / a.H;
    pv.h = bh - pv.b * a.H;
    pv.Lq = a.Lq;
    pv.Lk = a.Lk;
    pv.nKT = a.nKT;
    pv.tiles = a.tiles + (size_t)bh * a.nKT * TileGeom<D>::TILE_BYTES;
    pv.q_off = (int64_t)pv.b * a.sq_b + (int64_t)pv.h * a.sq_h;
    pv.o_off = (int64_t)pv.b * a.so_b + (int64_t)pv.h * a.so_h;
    pv.lse_off = ((int64_t)pv.b * a.H + pv.h) * a.Lq;
    pv.stat_off = (int64_t)pv.b * a.Lq;
    pv.Hg = a.rg.Hg;
    pv.Wg = a.rg.Wg;
    attn_pipe16_body<D, QK_OP, PV_OP, NW, false, false, false, QBN>(a, pv);
}

// The same with the query tiles of the last, partly filled round cut into pieces along the keys (AttnArgs::split):
// the first n_full workgroups take whole query tiles, the others one piece each, all pieces of one key range before
// those of the next so that neighbouring workgroups stream the same key tiles.
template <int D, int QK_OP, int PV_OP>
__global__ void __launch_bounds__(512, 2) attn_fwd_pipe16_split_kernel(const AttnArgs a) {
    const int n_full = a.split.n_full, n_tail = a.split.n_tail, n_piece = a.split.n_piece;
    const bool whole = (int)blockIdx.x < n_full;
    // (n_full is a multiple of 8: a workgroup's XCD is its index modulo 8 on both sides)
    const int logical = whole ? xcd_contiguous(blockIdx.x, n_full) : xcd_contiguous(blockIdx.x - n_full, n_tail * n_piece);
    PipeView pv;
    pv.piece = whole ? -1 : logical;
    const int tile = whole ? logical : n_full + logical % n_tail;
    const int bh = tile / a.nQT;
    pv.qt = tile % a.nQT;
    pv.b = bh / a.H;
    pv.h = bh - pv.b * a.H;
    // key tiles [k0, k1) of the sequence; n_piece <= nKT
    const int s = whole ? 0 : logical / n_tail, ns = whole ? 1 : n_piece;
    const int k0 = (int)((int64_t)a.nKT * s / ns), k1 = (int)((int64_t)a.nKT * (s + 1) / ns);
    pv.Lq = a.Lq;
    pv.nKT = k1 - k0;
    pv.Lk = (a.Lk < k1 * kBK ? a.Lk : k1 * kBK) - k0 * kBK;
    pv.tiles = a.tiles + ((size_t)bh * a.nKT + k0) * TileGeom<D>::TILE_BYTES;
    pv.q_off = (int64_t)pv.b * a.sq_b + (int64_t)pv.h * a.sq_h;
    pv.o_off = (int64_t)pv.b * a.so_b + (int64_t)pv.h * a.so_h;
    pv.lse_off = ((int64_t)pv.b * a.H + pv.h) * a.Lq;
    pv.stat_off = (int64_t)pv.b * a.Lq;
    pv.Hg = a.rg.Hg;
    pv.Wg = a.rg.Wg;
    attn_pipe16_body<D, QK_OP, PV_OP, 8, false, true>(a, pv);
}

// Puts the pieces of a query tile together: out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s, M = max_s m_s.  A
// wavefront takes 16 rows (block rb of the tile), in the layout the pieces were left in; memory-bound (it reads every
// piece once; writing, reading and the launch together cost what 3 + 0.037 key-tile steps a piece would, see
// choose_split).  6,240 tokens x 4 heads, whole call: 120 -> 101 us.  Pieces: first, first + stride, ...
template <int D>
__device__ __forceinline__ void combine_rows(const AttnArgs& a, int64_t first, int stride, int n_piece, int rb, int row,
                                             int Lq, int64_t o_off, int64_t lse_off) {
    constexpr int NCB = D / 16;
    const int lane = threadIdx.x & 63, i16 = lane & 15, g4 = lane >> 4;
    float m = -INFINITY;
    for (int s = 0; s < n_piece; ++s) m = fmaxf(m, a.part_ml[((first + (int64_t)s * stride) * 16 + rb) * 16 + i16].x);
    float l = 0.f;
    float4 o[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) o[cb] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < n_piece; ++s) {
        const int64_t blk = (first + (int64_t)s * stride) * 16 + rb;
        const float2 ml = a.part_ml[blk * 16 + i16];
        const float4* const src = reinterpret_cast<const float4*>(a.part_o) + blk * NCB * 64 + lane;
        float4 x[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) x[cb] = src[cb * 64];
        // (a piece of -inf scores only, bf16 score operands, weighs nothing, also where there is no other)
        const float w = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - m);
        l = fmaf(w, ml.y, l);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            o[cb].x = fmaf(w, x[cb].x, o[cb].x);
            o[cb].y = fmaf(w, x[cb].y, o[cb].y);
            o[cb].z = fmaf(w, x[cb].z, o[cb].z);
            o[cb].w = fmaf(w, x[cb].w, o[cb].w);
        }
    }
    if (row >= Lq) return;
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const int64_t obase = o_off + (int64_t)row * a.so_t + 4 * g4;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        const float o0 = o[cb].x * inv, o1 = o[cb].y * inv, o2 = o[cb].z * inv, o3 = o[cb].w * inv;
        if (a.out_f32)
            *reinterpret_cast<float4*>(static_cast<float*>(a.out) + obase + 16 * cb) = make_float4(o0, o1, o2, o3);
        else
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + obase + 16 * cb) =
                make_uint2(pack2<OP_BF16>(o0, o1), pack2<OP_BF16>(o2, o3));
    }
    if (a.lse && g4 == 0)
        a.lse[lse_off + row] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
}

template <int D>
__global__ void __launch_bounds__(256) attn_combine_kernel(const AttnArgs a) {
    const int rb = (blockIdx.x & 3) * 4 + (threadIdx.x >> 6);
    const int t = blockIdx.x >> 2, tile = a.split.n_full + t;
    const int bh = tile / a.nQT, qt = tile % a.nQT, b = bh / a.H, h = bh - b * a.H;
    combine_rows<D>(a, t, a.split.n_tail, a.split.n_piece, rb, qt * 256 + rb * 16 + (threadIdx.x & 15), a.Lq,
                    (int64_t)b * a.so_b + (int64_t)h * a.so_h, (int64_t)bh * a.Lq);
}

template <int D>
__global__ void __launch_bounds__(256) attn_combine_varlen_kernel(const AttnArgs a, const VarlenTable vt) {
    const int rb = (blockIdx.x & 3) * 4 + (threadIdx.x >> 6);
    int t = blockIdx.x >> 2, r = 0;
    for (; r < vt.n; ++r) {
        const int tiles = vt.r[r].n_piece > 1 ? a.H * vt.r[r].nQT : 0;
        if (t < tiles) break;
        t -= tiles;
    }
    if (r == vt.n) return;
    const ReqDesc& rq = vt.r[r];
    const int h = t / rq.nQT, qt = t - h * rq.nQT;
    combine_rows<D>(a, rq.piece0 + h * rq.n_piece * rq.nQT + qt, rq.nQT, rq.n_piece, rb,
                    qt * 256 + rb * 16 + (threadIdx.x & 15), rq.L, (int64_t)rq.tok0 * a.so_t + (int64_t)h * a.so_h,
                    (int64_t)h * vt.total_tokens + rq.tok0);
}

// Packed requests of different lengths: work distribution in varlen_view.  PIECES: some requests' tiles are computed
// in pieces (8 wavefronts only).
template <int D, int QK_OP, int PV_OP, int NW, bool PIECES, int QBN>
__global__ void __launch_bounds__(64 * NW, 2) attn_fwd_pipe16_varlen_kernel(const AttnArgs a, const VarlenTable vt) {
    PipeView pv;
    if (!varlen_view<D>(a, vt, pv)) return;  // uniform over the workgroup, before any barrier
    attn_pipe16_body<D, QK_OP, PV_OP, NW, false, PIECES, false, QBN>(a, pv);
}

// Cross-attention with one joint softmax per request: workgroups chain `qch` query tiles of one request, head by head.
// The pre-pack leaves a request's attending keys densely in its tiles 0 .. count-1 (without a mask or counts all keys
// attend), so only the last of them is partial; count and that tile's mask come from the
// workspace.  Workgroup order: request fastest, then the chains in the order of their query tiles, so that the workgroups
// an XCD holds at a time share a handful of (request, head) tile sets in its L2 and requests of different lengths are
// interleaved.  (Workgroups that walk a 256th of ALL query tiles each, in one round, have 20 heads in work on an XCD at a
// time: 1,530 us where this order takes 1,480; striding them over the XCD's share so that they stay together costs a start
// per request and index arithmetic that small calls feel.)
// TWO: the tiles of the two sequences stand from image 0 and from image nTA on, the tile counts of both together and of
// the first come from the workspace; a sequence without a key has no pass.
template <int D, int QK_OP, int PV_OP, int NW, bool TWO, int QBN, bool ONCE>
__global__ void __launch_bounds__(64 * NW, 2) attn_fwd_pipe16_chain_kernel(const AttnArgs a, int qch) {
    const int logical = xcd_contiguous_block();
    PipeView pv;
    const int chain = logical / a.B;
    pv.b = logical - chain * a.B;
    const int tile0 = chain * qch;
    pv.h = tile0 / a.nQT;
    pv.qt = tile0 - pv.h * a.nQT;
    pv.qt_count = a.H * a.nQT - tile0 < qch ? a.H * a.nQT - tile0 : qch;
    pv.Lq = a.Lq;
    pv.Lk = a.Lk;
    pv.nKT = a.tile_count[pv.b];
    pv.tiles = a.tiles + ((size_t)(pv.b * a.H + pv.h) * a.nKT) * TileGeom<D>::TILE_BYTES;
    pv.stat_off = (int64_t)pv.b * a.Lq;
    pv.Hg = a.rg.Hg;
    pv.Wg = a.rg.Wg;
    if constexpr (TWO) {
        const int first = a.tile_count_a[pv.b];
        pv.n_first = first > 0 ? first : pv.nKT;
        pv.skip_first = first > 0 || pv.nKT == 0 ? 0 : a.nTA;
        pv.skip_second = first < pv.nKT ? a.nTA - first : 0;
    }
    attn_pipe16_body<D, QK_OP, PV_OP, NW, true, false, TWO, QBN, ONCE>(a, pv);
}

// qch: query tiles per workgroup
template <int D, int QK_OP, int PV_OP, int NW, bool TWO, int QBN = 2, bool ONCE = false>
hipError_t launch_attn_pipe16_chain_inst(const AttnArgs& a, int qch, hipStream_t s) {
    auto kern = attn_fwd_pipe16_chain_kernel<D, QK_OP, PV_OP, NW, TWO, QBN, ONCE>;
    constexpr int smem = chain_lds_bytes<D, NW>();
    static std::atomic<uint64_t> attr_set{0};
    hipError_t e = allow_dynamic_lds(kern, smem, attr_set);
    if (e != hipSuccess) return e;
    const int64_t chains = ((int64_t)a.H * a.nQT + qch - 1) / qch;
    hipLaunchKernelGGL(kern, dim3((unsigned)(chains * a.B)), dim3(64 * NW), smem, s, a, qch);
    return hipGetLastError();
}

template <int D, int QK_OP, int PV_OP, int NW, int QBN>
hipError_t launch_attn_pipe16_inst(const AttnArgs& a, hipStream_t s) {
    auto kern = attn_fwd_pipe16_kernel<D, QK_OP, PV_OP, NW, QBN>;
    constexpr int smem = NW == 8 ? chain_lds_bytes<D, NW>() : pipe_lds_bytes<D, NW>();
    static std::atomic<uint64_t> attr_set{0};
    hipError_t e = allow_dynamic_lds(kern, smem, attr_set);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((int64_t)a.nQT * a.B * a.H));
    hipLaunchKernelGGL(kern, grid, dim3(64 * NW), smem, s, a);
    return hipGetLastError();
}

template <int D, int QK_OP, int PV_OP>
hipError_t launch_attn_pipe16_split_inst(const AttnArgs& a, hipStream_t s) {
    auto kern = attn_fwd_pipe16_split_kernel<D, QK_OP, PV_OP>;
    constexpr int smem = chain_lds_bytes<D, 8>();
    static std::atomic<uint64_t> attr_set{0};
    hipError_t e = allow_dynamic_lds(kern, smem, attr_set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.split.n_full + a.split.n_tail * a.split.n_piece)), dim3(512), smem, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(attn_combine_kernel<D>, dim3((unsigned)(4 * a.split.n_tail)), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int D, int QK_OP, int PV_OP, int NW, bool PIECES, int QBN>
hipError_t launch_attn_pipe16_varlen_inst(const AttnArgs& a, const VarlenTable& vt, hipStream_t s) {
    auto kern = attn_fwd_pipe16_varlen_kernel<D, QK_OP, PV_OP, NW, PIECES, QBN>;
    constexpr int smem = NW == 8 ? chain_lds_bytes<D, NW>() : pipe_lds_bytes<D, NW>();
    static std::atomic<uint64_t> attr_set{0};
    hipError_t e = allow_dynamic_lds(kern, smem, attr_set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * vt.queue_len)), dim3(64 * NW), smem, s, a, vt);
    e = hipGetLastError();
    if constexpr (PIECES) {
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(attn_combine_varlen_kernel<D>, dim3((unsigned)(4 * vt.split_tiles)), dim3(256), 0, s, a, vt);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace dit
