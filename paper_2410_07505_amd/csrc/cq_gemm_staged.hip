// W8A8 linear layer for few tokens, small outputs and any layout: output tiles from 16 x 16 to 128 x 128 whose
// contraction is split over the waves of a block.
//
// The ring kernel (cq_gemm.hip) works on 256 x 256 tiles: at 16 tokens it multiplies 240 rows of padding, and a
// 256 x 4096 output gives it 32 half tiles for 256 CUs.  Here a block's 8 waves are WM x WN wave tiles of 16 MT tokens x
// 16 NT channels times WK shares of the contraction; the WK partial sums (int32, so their order cannot matter) meet in
// LDS at the end.  The tile is chosen so that one round of blocks covers the chip (launch_w8a8_staged).
// What bounds it: what a CU takes in.  Its L2 delivers 64 bytes per clock where it hits; with the requests of a layer, whose
// tiles share rows across the CUs, loads alone reach 41 to 44 (25 TB/s over the chip), so a step costs (TM + TN) x 128 bytes of
// that; a decode step of a large layer is bound by the weights' way from HBM.  Every tile pays some 3.5 us besides (launch and
// first requests), partial sums and stores another 1 to 3.
#include <algorithm>
#include <type_traits>

#include "cq_gemm_common.h"

namespace cq {
namespace {

// 16 bytes at p, any alignment
__device__ __forceinline__ v4i load16(const int8_t* p) {
    v4i v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
// bytes [kb, kb + 16) of a row of I >= 16 bytes, bytes past the row's end as zero; nothing outside the row is read
__device__ __forceinline__ v4i load16_tail(const int8_t* row, int kb, int I) {
    const int at = min(kb, I - 16), sh = kb - at;
    unsigned __int128 w = __builtin_bit_cast(unsigned __int128, load16(row + at));
    w = sh >= 16 ? 0 : w >> (8 * (sh & 15));
    return __builtin_bit_cast(v4i, w);
}

// A step is 64 WK contraction bytes; wave share wk multiplies slab wk of it.  A slot holds one step:
// [WK / 2][TM + TN rows][128 bytes], chunk c of row R at chunk c ^ ((R >> 1) & 7), so that the 16 rows a fragment read
// covers fall on distinct banks.  LDS row 16 ni + f of a wave's weight rows holds its channel NT f + ni (the loader picks
// the rows; a request covers whole 128-byte lines of 8 rows).
// At step kt the fragments of kt are in registers; behind the step's barrier slot kt % S is free (step kt + S is
// requested into it) and step kt + 1 has landed (its fragments are read while kt is multiplied): one barrier a step.
// DMA: operands aligned to 16 bytes with I % 16 == 0 go straight to LDS; pieces past a row's end come from a zero
// block.  Otherwise (I >= 16) they pass through registers, loaded unaligned two steps before they are stored: 512 x 2752 x
// 4096 takes 13.7 us in the first form, 512 x 2756 x 4096 15.0 us in the second (whether rows start on a word or a byte makes
// 1 us; with one step in registers, and the row's end dealt with in every step, which spilled, 19.9 us).
// ONCE: the weights' requests are non-temporal.
template <int MT, int NT, int WM, int WN, int WK, int S, bool DMA, bool ONCE>
__global__ void __launch_bounds__(64 * kSplitWaves)
gemm_i8_staged_kernel(const int8_t* __restrict__ qx, const float* __restrict__ row_scale, const int8_t* __restrict__ qw,
                      const float* __restrict__ w_scale, int T, int I, int O, uint16_t* __restrict__ Y, int64_t ldy,
                      int32_t* __restrict__ acc_debug, int tiles_m, int total, bool vec_out) {
    static_assert(WM * WN * WK == kSplitWaves && WK % 2 == 0, "8 waves, whole 128-byte lines");
    constexpr int TM = 16 * MT * WM, TN = 16 * NT * WN, kRows = TM + TN;
    constexpr int kStepK = 64 * WK, kSlot = kRows * kStepK;
    constexpr int N = kSlot / 1024 / kSplitWaves;             // 1 KiB requests per wave and step
    static_assert(N * 1024 * kSplitWaves == kSlot, "the waves share a step evenly");
    extern __shared__ __align__(16) int8_t lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = wave % (WM * WN), wk = wave / (WM * WN);
    const int wm = w / WN, wn = w % WN;
    const int fr = lane & 15, chunk = lane >> 4;
    const int nk = (I + kStepK - 1) / kStepK;
    // A request holds its wave for about 100 cycles: with many requests a step waves 0-3 (one per SIMD) make them before
    // they multiply and waves 4-7 after, so that one wave of every SIMD multiplies meanwhile; with the short steps of WK = 2
    // all waves make them after (1024 x 4096 x 4096 24.5 -> 23.0 us, 1000 x 2750 x 4090 through registers 26.5 -> 25.1).
    const bool early = WK > 2 && wave < 4;

    const int per_xcd = (total + kXcds - 1) / kXcds;
    for (int i = blockIdx.x / kXcds; i < per_xcd; i += gridDim.x / kXcds) {
        const int L = (blockIdx.x % kXcds) * per_xcd + i;
        if (L >= total) break;                                // block-uniform
        const int tile_n = L / tiles_m;
        const int m0 = (L - tile_n * tiles_m) * TM, n0 = tile_n * TN;

        // request n of this wave fills LDS rows 8 g .. 8 g + 7 of a slot, g = wave N + n; lane l's 16 bytes are physical
        // chunk l & 7 of row 8 g + (l >> 3)
        const int8_t* src[N];
        int kb[N];                                            // first contraction byte of the lane's piece in step 0
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int g = wave * N + n, R_all = 8 * g + (lane >> 3);
            const int sub = R_all / kRows, R = R_all % kRows;
            kb[n] = sub * 128 + (((lane & 7) ^ ((R >> 1) & 7)) * 16);
            if (R < TM) {
                src[n] = qx + (int64_t)min(m0 + R, T - 1) * I + kb[n];
            } else {
                const int b = R - TM, grp = b / (16 * NT), in = b % (16 * NT);
                src[n] = qw + (int64_t)min(n0 + grp * 16 * NT + NT * (in & 15) + (in >> 4), O - 1) * I + kb[n];
            }
        }
        // Steps are taken from the end of the contraction: step 0 is its last, partly filled stretch, so that only the
        // prologue deals with pieces past a row's end.
        auto load_step = [&](v4i (&r)[N], int kt) {           // register form: this wave's pieces of a step (kt > 0)
            const int koff = (nk - 1 - kt) * kStepK;
#pragma unroll
            for (int n = 0; n < N; ++n) r[n] = load16(src[n] + koff);
        };
        auto commit = [&](const v4i (&r)[N], int slot) {
#pragma unroll
            for (int n = 0; n < N; ++n)
                *reinterpret_cast<v4i*>(lds + slot * kSlot + (wave * N + n) * 1024 + lane * 16) = r[n];
        };
        auto request = [&](int kt, int slot) {                // DMA: straight to LDS (kt > 0)
            const int koff = (nk - 1 - kt) * kStepK;
            const int8_t* dst = lds + slot * kSlot + wave * N * 1024;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                if (ONCE && (8 * (wave * N + n)) % kRows >= TM) request_1k<true>(src[n] + koff, dst + n * 1024);   // (scalar)
                else request_1k(src[n] + koff, dst + n * 1024);
            }
        };

        struct Frags {
            v4i a[MT], b[NT];
        };
        const int sub_base = (wk >> 1) * kRows * 128;
        const int sw = (((wk & 1) * 4 + chunk) ^ ((fr >> 1) & 7)) * 16;
        const int a_off = sub_base + (wm * 16 * MT + fr) * 128 + sw, b_off = sub_base + (TM + wn * 16 * NT + fr) * 128 + sw;
        auto read = [&](Frags& f, int slot) {
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) f.b[ni] = *reinterpret_cast<const v4i*>(lds + slot * kSlot + b_off + ni * 2048);
#pragma unroll
            for (int mi = 0; mi < MT; ++mi) f.a[mi] = *reinterpret_cast<const v4i*>(lds + slot * kSlot + a_off + mi * 2048);
        };
        v4i acc[MT][NT];
#pragma unroll
        for (int mi = 0; mi < MT; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) acc[mi][ni] = v4i{0, 0, 0, 0};

        // The scales first, held until the end.  (Behind the first requests, or a few steps before the end, the waits for
        // requests become waits for more of them: FP6 32 x 5120 x 20480 15.5 us, 15.8 and 17.3.  The fence keeps the loads here.)
        // Not under 64 x 64 tiles, whose first requests then start later than their end gains: 134 x 512 x 3544 4.9 us so, 4.7 with the
        // scales loaded at the end, 639 x 128 x 960 4.45 : 4.3.
        constexpr bool kScalesLast = TM == 64 && TN == 64;
        TileScales<MT, NT, WK> scales;
        if (!kScalesLast) {
            tile_scales<MT, NT, WN, WK>(scales, row_scale, w_scale, T, O, m0, n0, w, wk, lane);
            asm volatile("" ::: "memory");
        }
        // prologue: steps 0 .. S - 1 requested (register form: loaded together and stored; steps S and S + 1 on their way
        // into the two register sets)
        v4i r0[N], r1[N];
        const int last = (nk - 1) * kStepK;                   // where step 0 starts
        if (DMA) {
            const int8_t* dst = lds + wave * N * 1024;
#pragma unroll
            for (int n = 0; n < N; ++n)
                request_1k(last + kb[n] < I ? static_cast<const void*>(src[n] + last) : static_cast<const void*>(&g_zero_piece),
                           dst + n * 1024);
#pragma unroll
            for (int s = 1; s < S; ++s)
                if (s < nk) request(s, s);
        } else {
            v4i pre[S][N];
#pragma unroll
            for (int n = 0; n < N; ++n) pre[0][n] = load16_tail(src[n] - kb[n], last + kb[n], I);
#pragma unroll
            for (int s = 1; s < S; ++s)
                if (s < nk) load_step(pre[s], s);
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (s < nk) commit(pre[s], s);
            if (S < nk) load_step(r0, S);
            if (S + 1 < nk) load_step(r1, S + 1);
        }
        if (!DMA) __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, 0));
        else if (nk >= S) __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 1) * N, 15));     // step 0 has landed
        else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
        step_barrier();
        Frags f0, f1;
        read(f0, 0);

        // FULL: a step whose requests and reads all exist; the others, at the contraction's end, ask.  The wait for this wave's
        // LDS reads has to stand on every path by itself: as part of the one or the other wait the compiler sees a way
        // around it, and puts a wait for *all* reads, the next step's too, in front of this step's matrix instructions.
        int slot = 0;                                         // slot of step kt
        auto step = [&](auto full_c, int kt, Frags& cur, Frags& nxt, v4i (&r)[N]) {
            constexpr bool FULL = decltype(full_c)::value;
            // this wave's reads of step kt are done and its share of step kt + 1 has landed (steps kt + 2 .. kt + S - 1
            // may still be in flight; near the end, where there are fewer, all of them)
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(DMA && FULL ? (S - 2) * N : 63, 0));
            if (DMA && !FULL) {
                if (kt + S - 1 < nk) __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 2) * N, 15));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
            }
            step_barrier();
            auto fetch = [&]() {
                if (FULL || kt + S < nk) {
                    if (DMA) {
                        request(kt + S, slot);
                    } else {
                        commit(r, slot);
                        if (FULL || kt + S + 2 < nk) load_step(r, kt + S + 2);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            const int next_slot = slot + 1 == S ? 0 : slot + 1;
            if (early) fetch();
            if (FULL || kt + 1 < nk) read(nxt, next_slot);
#pragma unroll
            for (int mi = 0; mi < MT; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_i32_16x16x64_i8(cur.a[mi], cur.b[ni], acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (!early) fetch();
            slot = next_slot;
        };
        using yes = std::integral_constant<bool, true>;
        using no = std::integral_constant<bool, false>;
        // (full steps only where there are many: for smaller tiles their code costs more, fetched once, than they save)
        constexpr bool kFullSteps = TM * TN >= 8192;
        constexpr int kAhead = DMA ? S : S + 2;               // a step asks for the one this many on
        int kt = 0;
        for (; kFullSteps && kt + 1 + kAhead < nk; kt += 2) {
            step(yes{}, kt, f0, f1, r0);
            step(yes{}, kt + 1, f1, f0, r1);
        }
        for (; kt < nk; kt += 2) {
            step(no{}, kt, f0, f1, r0);
            if (kt + 1 < nk) step(no{}, kt + 1, f1, f0, r1);
        }
        __syncthreads();                                      // the ring is free: it holds the partial sums now
        if (kScalesLast) tile_scales<MT, NT, WN, WK>(scales, row_scale, w_scale, T, O, m0, n0, w, wk, lane);
        sum_and_store<MT, NT, WM, WN, WK>(acc, lds, scales, w, wk, lane, T, O, Y, ldy, acc_debug, m0, n0, vec_out);
        __syncthreads();
    }
}

template <int MT, int NT, int WM, int WN, int WK, int S, bool DMA, bool ONCE = false>
hipError_t launch_staged(const int8_t* qx, const float* row_scale, const int8_t* qw, const float* w_scale, int T, int I,
                         int O, uint16_t* Y, int64_t ldy, int32_t* acc_debug, hipStream_t stream) {
    constexpr int TM = 16 * MT * WM, TN = 16 * NT * WN;
    constexpr int kRing = S * (TM + TN) * 64 * WK, kParts = kPartsBytes<MT, NT, WM, WN, WK>, kLds = kRing > kParts ? kRing : kParts;
    const int tiles_m = (T + TM - 1) / TM;
    const int64_t total = (int64_t)tiles_m * ((O + TN - 1) / TN);
    if (total >= (int64_t)1 << 31) return hipErrorInvalidValue;
    const bool vec_out = O % NT == 0 && ldy % NT == 0 && reinterpret_cast<uintptr_t>(Y) % (2 * NT) == 0;
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_i8_staged_kernel<MT, NT, WM, WN, WK, S, DMA, ONCE>), kLds, allowed);
    if (e != hipSuccess) return e;
    const int64_t blocks = std::min<int64_t>((total + kXcds - 1) / kXcds * kXcds, (int64_t)1 << 20);
    gemm_i8_staged_kernel<MT, NT, WM, WN, WK, S, DMA, ONCE><<<dim3((unsigned)blocks), dim3(64 * kSplitWaves), kLds, stream>>>(
        qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, tiles_m, (int)total, vec_out);
    return hipGetLastError();
}

// Contractions shorter than one 16-byte piece: a thread per output.
__global__ void __launch_bounds__(256)
gemm_i8_short_kernel(const int8_t* __restrict__ qx, const float* __restrict__ row_scale, const int8_t* __restrict__ qw,
                     const float* __restrict__ w_scale, int T, int I, int O, uint16_t* __restrict__ Y, int64_t ldy,
                     int32_t* __restrict__ acc_debug) {
    const int64_t n = (int64_t)T * O;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t r = i / O, k = i - r * O;
        int v = 0;
        for (int j = 0; j < I; ++j) v += (int)qx[r * I + j] * (int)qw[k * I + j];
        float y = (float)v * row_scale[r];
        y = rounded_f32(y * w_scale[k]);
        Y[r * ldy + k] = (uint16_t)f2h(y);
        if (acc_debug) acc_debug[i] = v;
    }
}

}  // namespace

// Tile kinds by what a CU has to take in for one byte of the contraction of one tile (TM + TN rows).  The cost of a launch is the
// rounds of tiles over the CUs times that; of equal ones the smaller tile is taken.  Measured at I = 4096 (us, best kind
// first): 16 x 4096 4.7 (16 x 16), 5.7 (32 x 32), 7.1 (32 x 64); 64 x 4096 7.1 (32 x 32), 7.2 (32 x 64), 9.1 (64 x 64);
// 64 x 11008 11.6 (64 x 64), 12.7 (32 x 64), 16.6 (32 x 32); 256 x 4096 10.5 (64 x 64), 11.7 (32 x 64), 12.6 (64 x 128);
// 512 x 4096 14.7 (64 x 128), 18.2 (128 x 128), 19.4 (64 x 64); the rule picks the first of each.  Off the 16-byte layout
// likewise: 128 x 2750 x 4090 9.1 (32 x 64), 10.2 (64 x 64), 13.1 (32 x 32); 509 x 2750 x 4090 17.5 (64 x 128), 18.6
// (64 x 64), 21.0 (128 x 128); 1000 x 2750 x 4090 24.7 (128 x 128), 34.2 (64 x 128).
static const int kKinds[][2] = {{16, 16}, {32, 32}, {32, 64}, {64, 64}, {64, 128}, {128, 128}};
constexpr int kNumKinds = 6;

static bool staged_dma(const int8_t* qx, const int8_t* qw, int I) {
    return reinterpret_cast<uintptr_t>(qx) % 16 == 0 && reinterpret_cast<uintptr_t>(qw) % 16 == 0 && I % 16 == 0;
}

static int best_kind(int T, int O, int n_cu, int64_t* cost) {
    int best = -1;
    for (int k = 0; k < kNumKinds; ++k) {
        const int tm = kKinds[k][0], tn = kKinds[k][1];
        const int64_t tiles = (int64_t)((T + tm - 1) / tm) * ((O + tn - 1) / tn);
        const int64_t c = (tiles + n_cu - 1) / n_cu * (tm + tn);
        if (best < 0 || c < *cost) {
            best = k;
            *cost = c;
        }
    }
    return best;
}

// The time of the launch in the unit of the kinds' cost (one operand row and one byte of the contraction; 75000 of them are
// about 1 us), with what a round of tiles takes besides: first requests, partial sums, stores.  Fitted to launches of 1 to 6
// rounds with I from 128 to 8192; at that time one round of 64 x 64 tiles took 4.2 us + 1.45 us per 1024 bytes of I, of 64 x 128 6.0 + 2.4,
// of 128 x 128 6.6 + 3.5.  Now, from 1024 to 4096 bytes, 4.4 + 1.6, 5.9 + 2.2 and 6.0 + 3.9.  More than 2048 tokens under 128 x 128 tiles
// are left to the ring: every XCD walks one column of tiles there and fetches all the activations (4096 x 4096 x 1024 25.4 us against
// 25.3; 2048 x 4096 x 2048 22.5 : 25.8).
int64_t w8a8_staged_time(int T, int I, int O, int n_cu) {
    static const int kRound[kNumKinds] = {82000, 142000, 90000, 187000, 329000, 351000};
    int64_t cost = 0;
    const int kind = best_kind(T, O, n_cu, &cost);
    if (kind == kNumKinds - 1 && T > 2048) return INT64_MAX;
    return cost * I + cost / (kKinds[kind][0] + kKinds[kind][1]) * kRound[kind];
}

hipError_t launch_w8a8_staged(const int8_t* qx, const float* row_scale, const int8_t* qw, const float* w_scale, int T, int I,
                              int O, uint16_t* Y, int64_t ldy, int32_t* acc_debug, int n_cu, hipStream_t stream) {
    if (I < 16) {
        const int64_t blocks = std::min<int64_t>(((int64_t)T * O + 255) / 256, (int64_t)1 << 20);
        gemm_i8_short_kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug);
        return hipGetLastError();
    }
    const bool dma = staged_dma(qx, qw, I);
    int64_t cost;
    // the steps and slots of a kind: as much of the contraction per barrier, and as many slots, as the LDS allows; through
    // registers shorter steps and fewer slots, which leave the registers for two steps on their way (512 x 2756 x 4096 with
    // 64 x 128 tiles: 15.5 us with WK 2 and 3 slots, 15.7 with 4, 19.1 with WK 4)
    // Weights that one row of tiles reads once and that no cache keeps are requested non-temporally: 16 x 8192 x 28672 44.2 ->
    // 37.9 us (6.2 TB/s), 64 x 8192 x 28672 52.6 -> 47.7, 32 x 8192 x 22016 42.2 -> 37.8, but 16 x 4096 x 22016 (86 MiB, part of which
    // the memory-side cache keeps from one call to the next) 18.5 -> 21.3.  The kinds without such an instance request plainly: they
    // are not the fastest ones for these up-projections.  (Down-projections take some of them, 16 x 28672 x 8192 the 16 x 16
    // tiles; on 16 x 8192 x 28672 non-temporal requests took them from 45.2 to 42.7 us, 32 x 32 from 51.3 to 45.8, 64 x 64 from 48.3
    // to 43.9.)
    const int kind = best_kind(T, O, n_cu, &cost);
    const bool once = dma && T <= kKinds[kind][0] && (int64_t)O * I > (int64_t)128 << 20;
#define CQ_STAGED(MT, NT, WM, WN, WK, S, ...) \
    launch_staged<MT, NT, WM, WN, WK, S, __VA_ARGS__>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream)
    switch (kind) {
        case 0: return dma ? CQ_STAGED(1, 1, 1, 1, 8, 4, true) : CQ_STAGED(1, 1, 1, 1, 8, 2, false);
        case 1: return dma ? CQ_STAGED(2, 2, 1, 1, 8, 4, true) : CQ_STAGED(2, 2, 1, 1, 8, 2, false);
        case 2: return once ? CQ_STAGED(2, 2, 1, 2, 4, 3, true, true) : dma ? CQ_STAGED(2, 2, 1, 2, 4, 3, true) : CQ_STAGED(2, 2, 1, 2, 4, 2, false);
        case 3: return dma ? CQ_STAGED(2, 4, 2, 1, 4, 4, true) : CQ_STAGED(2, 2, 2, 2, 2, 2, false);
        case 4: return once ? CQ_STAGED(4, 4, 1, 2, 4, 3, true, true) : dma ? CQ_STAGED(4, 4, 1, 2, 4, 3, true) : CQ_STAGED(2, 4, 2, 2, 2, 3, false);
        default: return once ? CQ_STAGED(4, 4, 2, 2, 2, 3, true, true) : dma ? CQ_STAGED(4, 4, 2, 2, 2, 3, true) : CQ_STAGED(4, 4, 2, 2, 2, 2, false);
    }
#undef CQ_STAGED
}

}  // namespace cq
