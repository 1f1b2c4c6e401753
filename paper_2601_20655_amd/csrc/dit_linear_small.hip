// Dense projection y[M, N] = x[M, K] w[N, K]^T + bias[N] where 256 x 256 tiles (dit_linear.hip) would leave most of the
// chip idle: few token rows, few features, or a tile count just past a multiple of the compute units.  One smaller
// tile per workgroup, walking K in steps of 64 through a ring of LDS stages filled by the load-to-LDS DMA.
//
// Same operand roles as the big kernel: w rows ride the A operand of v_mfma_f32_16x16x32_bf16, token rows the B
// operand; a lane (i, g) ends with token i of a block and features 4g .. 4g+3.
//
// What bounds it: no one unit.  769 x 10,240 x 5,120 in 160 x 256 tiles (counters, on the 200 compute units that have
// one): 171,500 clocks for 80 steps, the matrix cores busy in 60 % of them (the big kernel: 82 to 85 %), the LDS serving
// fragment reads in 28 % (4 clocks for a wavefront's 1 KiB; 32 %), a quarter of the wavefronts' time in waits: LDS holds
// three stages of so large a tile, and a step has one barrier.  So a small tile costs more per flop than a big one, and
// is taken only where it fills the chip better (choose_linear_form).
#include <type_traits>

#include "dit_attn_device.h"
#include "dit_attn_internal.h"

namespace dit {

namespace {

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<I + 1, N>(f);
    }
}

// 2 x 4 wavefronts (tokens x features), TB and FB 16-token and 16-feature blocks per wavefront
template <int TB, int FB>
struct LinTile {
    static constexpr int BM = 32 * TB, BN = 64 * FB;
    static constexpr int STAGE = (BM + BN) * 128;  // bytes of one step: 64 contraction indices of every row
    // Stages: as many as hide a trip to memory behind steps this short, within the LDS of one compute unit (large
    // tiles) or half of it (two workgroups per unit)
    static constexpr bool PAIR = STAGE <= 26 * 1024;
    static constexpr int FIT = (PAIR ? 80 : 160) * 1024 / STAGE;
    static constexpr int S = FIT > 6 ? 6 : FIT;
    static_assert(S >= 3, "at least two steps ahead");
    // DMA instructions per wavefront and step: FULL of 8 rows, and half of one more if TB is odd
    static constexpr int FULL = FB + TB / 2, LOADS = FULL + (TB & 1);
};

template <int TB, int FB, bool OUT_F32>
__global__ void __launch_bounds__(512, (LinTile<TB, FB>::PAIR ? 4 : 2)) linear_tile_kernel(const LinearArgs a) {
    using T = LinTile<TB, FB>;
    constexpr int S = T::S;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int wt = wave & 1, wf = wave >> 1;

    // contiguous ranges of tiles per XCD, token tiles fastest: the workgroups of an XCD share the rows of w
    int tm, tn;
    {
        const int nblk = gridDim.x, xcd = blockIdx.x & 7;
        const int chunk = nblk >> 3, rem = nblk & 7;
        const int logical = xcd * chunk + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
        tm = logical % a.nTM;
        tn = logical / a.nTM;
    }

    // A stage is the tile's BN rows of w, then its BM rows of x, 128 bytes each; the DMA moves 8 rows an instruction
    // and fills LDS in lane order, so the bank swizzle (piece p of row r in slot p ^ ((r >> 1) & 7)) is in which piece
    // a lane fetches.  Rows past the end are clamped to the last one; their products are not stored.
    const int r8 = lane >> 3;
    auto src_of = [&](int chunk) __attribute__((always_inline)) -> const uint8_t* {  // of 8 rows, step 0
        const bool is_w = chunk < T::BN / 8;
        const int r = 8 * (is_w ? chunk : chunk - T::BN / 8) + r8;
        const int piece = (lane & 7) ^ ((r >> 1) & 7);
        const int row0 = is_w ? tn * T::BN : tm * T::BM, end = is_w ? a.N : a.M;
        const int row = row0 + r < end ? row0 + r : end - 1;
        return reinterpret_cast<const uint8_t*>(is_w ? a.w + (int64_t)row * a.ldw : a.x + (int64_t)row * a.ldx) + piece * 16;
    };
    constexpr int FULL = T::FULL;
    const uint8_t* src[T::LOADS];
#pragma unroll
    for (int i = 0; i < FULL; ++i) src[i] = src_of(wave + 8 * i);
    if constexpr (TB & 1) src[FULL] = src_of(8 * FULL + (wave >> 1));  // half a chunk per wavefront
    f32x4 acc[FB][TB];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[fb][tb][r] = 0.f;

    const int sw = (lr >> 1) & 7;
    const int wread = (wf * 16 * FB + lr) * 128;
    const int xread = (T::BN + wt * 16 * TB + lr) * 128;
    // fragment i of a slice of 32 contraction indices: first the FB of w, then the TB of x
    auto read_fragment = [&](u32x4 (&W)[FB], u32x4 (&X)[TB], auto i, int stage, int ks) __attribute__((always_inline)) {
        constexpr int I = decltype(i)::value;
        const uint8_t* const base = smem + stage * T::STAGE + (((4 * ks + lg) ^ sw) * 16);
        if constexpr (I < FB) W[I] = *reinterpret_cast<const u32x4*>(base + wread + I * 2048);
        else X[I - FB] = *reinterpret_cast<const u32x4*>(base + xread + (I - FB) * 2048);
    };
    // All but the youngest S - 2 stages requested have arrived, and every wavefront has got as far.  (The bare barrier:
    // __syncthreads() would drain the loads that are meant to stay in flight.)
    auto sync_stage = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * T::LOADS) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    const int nK = a.K / kLinBK;
    // S - 1 stages are requested ahead; past the end of K the last step is requested again (into a stage nobody reads
    // any more), so that the number of loads in flight stays the constant the waits count on
    int requested = 0;
    auto request_piece = [&](auto i, int stage) __attribute__((always_inline)) {
        constexpr int I = decltype(i)::value;
        uint8_t* const dst = smem + stage * T::STAGE;
        src[I] += requested > 0 && requested < nK ? 128 : 0;  // on from the step requested before
        if constexpr (I < FULL) {
            __builtin_amdgcn_global_load_lds((gptr_t)src[I], (lptr_t)(dst + (wave + 8 * I) * 1024), 16, 0, 0);
        } else {
            if ((lane >> 5) == (wave & 1))
                __builtin_amdgcn_global_load_lds((gptr_t)src[I], (lptr_t)(dst + (8 * FULL + (wave >> 1)) * 1024), 16, 0, 0);
        }
    };
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        static_for<0, T::LOADS>([&](auto i) __attribute__((always_inline)) { request_piece(i, s); });
        ++requested;
    }
    sync_stage();
    u32x4 W0[FB], X0[TB], W1[FB], X1[TB];
    constexpr int R = FB + TB;  // fragments of a slice
    static_for<0, R>([&](auto i) __attribute__((always_inline)) { read_fragment(W0, X0, i, 0, 0); });
    // While one slice is multiplied, token block by token block, the next one is read: nothing ahead of the first block
    // (the wait for its own fragments would wait for what was just asked for too) nor of the last one (whose MFMAs
    // cover the youngest reads), PER fragments ahead of each block between.  (Left to the compiler the reads sank
    // behind the MFMAs and were waited for there: 641 x 3,320 x 1,664 14.6 -> 12.8 us, 3,600 x 5,120 x 5,120 166 -> 159.)
    constexpr int GAPS = TB > 2 ? TB - 2 : 1, PER = (R + GAPS - 1) / GAPS, LPER = (T::LOADS + GAPS - 1) / GAPS;
    int stage = 0, free_stage = S - 1;
    for (int k = 0; k < nK; ++k) {
        const int next = stage + 1 == S ? 0 : stage + 1;
        auto slice = [&](u32x4 (&W)[FB], u32x4 (&X)[TB], u32x4 (&Wn)[FB], u32x4 (&Xn)[TB], int nstage, auto ksn) __attribute__((always_inline)) {
            constexpr int KSN = decltype(ksn)::value;  // slice being read: 1 of this step, or 0 of the next
            static_for<0, TB>([&](auto tbc) __attribute__((always_inline)) {
                constexpr int tb = decltype(tbc)::value, gap = tb - 1;
                if constexpr (gap >= 0 && gap < GAPS) {
                    constexpr int r0 = gap * PER < R ? gap * PER : R, r1 = r0 + PER < R ? r0 + PER : R;
                    static_for<r0, r1>([&](auto i) __attribute__((always_inline)) { read_fragment(Wn, Xn, i, nstage, KSN); });
                    constexpr int l0 = gap * LPER < T::LOADS ? gap * LPER : T::LOADS;
                    constexpr int l1 = l0 + LPER < T::LOADS ? l0 + LPER : T::LOADS;
                    // the stage read one step ago is free: every wavefront passed a barrier behind its last read of it
                    if constexpr (KSN == 1)
                        static_for<l0, l1>([&](auto i) __attribute__((always_inline)) { request_piece(i, free_stage); });
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int fb = 0; fb < FB; ++fb) acc[fb][tb] = mfma16<OP_BF16>(W[fb], X[tb], acc[fb][tb]);
                __builtin_amdgcn_sched_barrier(0);
                // step k + 1 has arrived, everybody has read step k (its fragments have been waited for)
                if constexpr (KSN == 0 && tb == 0) sync_stage();
            });
            if constexpr (TB == 1) {
                static_for<0, R>([&](auto i) __attribute__((always_inline)) { read_fragment(Wn, Xn, i, nstage, KSN); });
                if constexpr (KSN == 1)
                    static_for<0, T::LOADS>([&](auto i) __attribute__((always_inline)) { request_piece(i, free_stage); });
            }
        };
        slice(W0, X0, W1, X1, stage, std::integral_constant<int, 1>());
        ++requested;
        slice(W1, X1, W0, X0, next, std::integral_constant<int, 0>());  // (behind the last step: unused)
        free_stage = stage;
        stage = next;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- store: 16 token rows at a time through an area of the wavefront's own, so that rows leave in 16-byte pieces
    // (Tried: non-temporal stores.  769 x 10,240 x 5,120 72.1 -> 70.6 us on the operands of the call before, 89.4 ->
    // 88.7 on new ones, but level with the kernel that reads the rows next: cross-attention of 256 queries on them 92.7
    // and 92.8.)
    constexpr int ES = OUT_F32 ? 4 : 2;
    constexpr int RB = 16 * FB * ES;  // bytes of a staged row: the wavefront's features
    constexpr int PR = RB / 16;       // pieces per row
    constexpr int NP = 16 * PR;       // pieces per pass
    static_assert(8 * 16 * RB <= S * T::STAGE && (PR & (PR - 1)) == 0, "staging geometry");
    uint8_t* const area = smem + wave * 16 * RB;
    // where piece c of staged row r lies: spread over the banks by the row number
    auto slot = [](int r, int c) { return c ^ (r & (PR - 1)); };
    float b[FB][4];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
        const int n0 = tn * T::BN + (wf * FB + fb) * 16 + 4 * lg;
        uint2 bb = make_uint2(0u, 0u);
        if (a.bias && n0 < a.N) bb = *reinterpret_cast<const uint2*>(a.bias + n0);
        b[fb][0] = bf16_lo(bb.x);
        b[fb][1] = bf16_hi(bb.x);
        b[fb][2] = bf16_lo(bb.y);
        b[fb][3] = bf16_hi(bb.y);
    }
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
            const float y0 = acc[fb][tb][0] + b[fb][0], y1 = acc[fb][tb][1] + b[fb][1];
            const float y2 = acc[fb][tb][2] + b[fb][2], y3 = acc[fb][tb][3] + b[fb][3];
            const int col = (16 * fb + 4 * lg) * ES;
            uint8_t* const dst = area + lr * RB + slot(lr, col >> 4) * 16 + (col & 15);
            if constexpr (OUT_F32) *reinterpret_cast<float4*>(dst) = make_float4(y0, y1, y2, y3);
            else *reinterpret_cast<uint2*>(dst) = make_uint2(pack2<OP_BF16>(y0, y1), pack2<OP_BF16>(y2, y3));
        }
        asm volatile("" ::: "memory");  // (one wavefront's LDS accesses complete in order)
#pragma unroll
        for (int p0 = 0; p0 < NP; p0 += 64) {
            const int p = p0 + lane;
            const int r = p / PR, c = p % PR;
            const int m = tm * T::BM + (wt * TB + tb) * 16 + r;
            const int n = tn * T::BN + wf * FB * 16 + c * (16 / ES);
            // N is a multiple of 8: a piece of a row is inside or outside as a whole
            if ((NP >= 64 || p < NP) && m < a.M && n < a.N) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(area + r * RB + slot(r, c) * 16);
                *reinterpret_cast<u32x4*>(static_cast<uint8_t*>(a.y) + ((int64_t)m * a.ldy + n) * ES) = v;
            }
        }
        asm volatile("" ::: "memory");
    }
}

template <int TB, int FB, bool OUT_F32>
hipError_t launch_tile(LinearArgs a, hipStream_t s) {
    using T = LinTile<TB, FB>;
    auto kern = linear_tile_kernel<TB, FB, OUT_F32>;
    constexpr int smem = T::S * T::STAGE;
    static std::atomic<uint64_t> attr_set{0};
    hipError_t e = allow_dynamic_lds(kern, smem, attr_set);
    if (e != hipSuccess) return e;
    a.nTM = (a.M + T::BM - 1) / T::BM;
    a.nTN = (a.N + T::BN - 1) / T::BN;
    if ((int64_t)a.nTM * a.nTN > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)a.nTM * a.nTN)), dim3(512), smem, s, a);
    return hipGetLastError();
}

// Every tile that is built, with the microseconds of one step where workgroups have a compute unit to themselves and
// where two share one (0: they cannot), and those of a workgroup's start and store.  Fitted to runs over 31 shapes
// (M 1 .. 32,760, N 256 .. 15,360, K 256 .. 5,120) before the reads and loads of a step were spread over its token
// blocks, which took up to 12 % off the larger ones: they decide for the big kernel a little too often.  The big kernel:
// 1.0 to 1.2 a step, 3.5 a tile and 4 a call.
struct Form {
    int tb, fb;
    double step, step2, ends;
};
constexpr Form kForms[] = {{1, 1, 0.20, 0.35, 2.5}, {2, 1, 0.215, 0.36, 2.5}, {2, 2, 0.33, 0.55, 3.0}, {4, 2, 0.47, 0.0, 3.0},
                           {3, 4, 0.74, 0.0, 3.5},  {4, 4, 0.76, 0.0, 4.0},   {5, 4, 1.05, 0.0, 4.0}};

}  // namespace

// The tile the estimate says is fastest (10 TB + FB), 0 for the big kernel, which keeps what is not 5 % slower there.
// Measured, us a call one after the other on the same operands: M x N x K = 769 x 10,240 x 5,120: 98 in 256 x 256 tiles
// (160 of them), 80 in 160 x 256 (with other work between the calls 98 and 88); 769 x 5,120 x 5,120: 82 and 56 (96 x 256);
// 512 x 3,072 x 1,536: 28 and 9 (64 x 128); 172 x 3,664 x 3,072: 51 and 11 (64 x 64); 1 x 15,360 x 5,120: 80 and 23;
// 3,600 x 5,120 x 5,120: 193 and 161 (160 x 256); kept: 14,040 x 1,536 x 1,536 (66), 3,600 x 15,360 x 5,120 (430).
int choose_linear_form(int M, int N, int K, int cus) {
    const double nK = K / kLinBK;
    auto tiles_of = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t big = tiles_of(kLinBM, kLinBN), full = big / cus, rest = big % cus;
    double best = 0.95 * (7.0 + full * (1.2 * nK + 3.5) + (rest == 0 ? 0.0 : (rest <= cus / 2 ? 1.0 : 1.2) * nK + 3.5));
    int form = 0;
    for (const Form& f : kForms) {
        const int64_t tiles = tiles_of(32 * f.tb, 64 * f.fb);
        const int slots = f.step2 > 0.0 ? 2 * cus : cus;
        const int64_t rounds = tiles / slots, left = tiles % slots;
        const double full_step = f.step2 > 0.0 ? f.step2 : f.step;
        const double t = 3.0 + rounds * (full_step * nK + f.ends) +
                         (left == 0 ? 0.0 : (left <= cus ? f.step : full_step) * nK + f.ends);
        if (t < best) {
            best = t;
            form = 10 * f.tb + f.fb;
        }
    }
    return form;
}

hipError_t launch_linear_small(const LinearArgs& a, int form, hipStream_t s) {
#define DIT_TILE(TB, FB) \
    if (form == 10 * TB + FB) return a.out_f32 ? launch_tile<TB, FB, true>(a, s) : launch_tile<TB, FB, false>(a, s);
    DIT_TILE(1, 1)
    DIT_TILE(2, 1)
    DIT_TILE(2, 2)
    DIT_TILE(4, 2)
    DIT_TILE(3, 4)
    DIT_TILE(4, 4)
    DIT_TILE(5, 4)
#undef DIT_TILE
    return hipErrorInvalidValue;
}

}  // namespace dit
