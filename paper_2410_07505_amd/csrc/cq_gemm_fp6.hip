// A4W4 linear layer on the FP6 matrix instruction (the W4A4 rows of the paper's accuracy tables).
//
// gfx950 has no INT4 matrix instruction, but the f8f6f4 matrix instructions multiply 6-bit floats at
// twice the INT8 rate, and every INT4 code q in [-7, 7] is exactly representable in FP6 E2M3
// (1 sign, 2 exponent, 3 mantissa bits, bias 1: 0, 1, 2, 3, 4, 5, 6, 7 are 0b000000, 0b001000,
// 0b010000, 0b010100, 0b011000, 0b011010, 0b011100, 0b011110).  Products are integers of at most
// 49 and the accumulator is binary32, so a dot product over I <= 2^18 channels stays below 2^24
// and is exact: the result equals the integer GEMM bit for bit, and the scale epilogue is the
// same sequence of binary32 operations as in the INT8 path.
//
// Operand format ("FP6 fragments"), produced by pack_fp6_kernel.  A fragment holds 32 rows x 64 K elements: lane
// slot s (0..63) is the 32 consecutive K elements [32 (s >> 5), +32) of row (s & 31) as one 192-bit little-endian
// stream (element j in bits [6j, 6j + 6)).  A matrix of R rows and K columns is stored as [ceil(R/32)][K/64]
// fragments of 1536 bytes, each fragment as a 1024-byte plane (64 slots x 16 bytes: bits [0, 128) of every
// slot's stream) followed by a 512-byte plane (64 slots x 8 bytes: bits [128, 192)); rows past R are zero.
// The weight operand uses the same fragments with its rows in a different order (pack_fp6_kernel<.., true>):
// inside every group of 64 output channels, stored row 16 n + f holds channel 4 f + n, so that the 16 rows of
// the kernel's weight tile n are the channels 4 f + n and a lane ends up with four adjacent channels.
//
// The matrix instruction is v_mfma_f32_16x16x128_f8f6f4: lane l supplies row (l & 15) and the 32 consecutive K
// elements of chunk l >> 4 of a 128-element K step, i.e. slot 16 p + (l & 15) + 32 (c & 1) of fragment c >> 1
// of the two fragments along K, for the rows [16 p, 16 p + 16) of a 32-row block: one 16-byte and one 8-byte
// LDS read per lane and tile.  (Which K positions a lane's elements take inside the instruction does not matter
// for a dot product, as long as both operands are read the same way.)  The 16-byte reads of 16 lanes are
// consecutive; for the 8-byte reads, of which the LDS serves 32 lanes per cycle, the two halves of a fragment's
// second plane would fall on the same banks, so in LDS the two 128-byte pieces of that plane's second half
// change places (done by the global -> LDS requests, which pick their 16 source bytes per lane).
// The 16 x 16 x 128 instruction instead of 32 x 32 x 64: half the accumulator register traffic per multiply-add
// (a loop fed from LDS sustains about 5 % more with it), and the accumulator layout the direct epilogue wants.
//
// The kernel follows the INT8 ring kernel's schedule with 6-bit operands: 256 x 256 block tile,
// 8 waves of 128 x 64 (8 x 4 tiles of 16 x 16), K step 128 elements (two fragments along K, 24 KiB per operand).
// The smaller operands leave room for a ring of six LDS slots, i.e. three tiles in flight: requests
// run two to three steps ahead (described at the kernel).  Per K step a wave issues 32 matrix
// instructions (half the cycles of the INT8 kernel for the same K) against 18 KiB of LDS reads,
// so this kernel is bound by operand movement rather than by the matrix pipe.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "cq_gemm_common.h"

namespace cq {
namespace {

constexpr int kFragBytes = 1536;                     // 32 rows x 64 elements x 6 bits
constexpr int kFragLo = 1024;                        // first plane: 64 lanes x 16 bytes
constexpr int kF6Slot = 8 * 2 * kFragBytes;          // 24 KiB: 256 rows x 128 elements
constexpr int kF6Slots = 6;
constexpr int kF6Ring = kF6Slots * kF6Slot;         // 144 KiB
constexpr int kF6Lds = kF6Ring + 8 * 512;           // ... and the epilogue's row factors behind it
static_assert(kF6Lds <= 160 * 1024, "LDS budget of a gfx950 CU");

// ---- packing ---------------------------------------------------------------------------------
// One thread builds one lane's 24 bytes of one fragment.  SRC 8: int8 codes [R][K]; SRC 4: packed
// two's-complement nibbles [R][K/2], even column in the low nibble.  Codes are clamped to +-7.
// WEIGHTS: stored row 64 g + 16 n + f holds row 64 g + 4 f + n of the source (see the head of this file).
template <int SRC, bool WEIGHTS>
__global__ void pack_fp6_kernel(const uint8_t* __restrict__ src, int R, int K, uint8_t* __restrict__ dst,
                                int64_t n_slots) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n_slots) return;
    const int lane = (int)(idx & 63);
    const int64_t frag = idx >> 6;
    const int KB = K / 64;
    const int kb = (int)(frag % KB), rb = (int)(frag / KB);
    const int stored = rb * 32 + (lane & 31);
    const int row = WEIGHTS ? (stored & ~63) + 4 * (stored & 15) + ((stored >> 4) & 3) : stored;
    const int k0 = kb * 64 + 32 * (lane >> 5);
    uint32_t w[6] = {0u, 0u, 0u, 0u, 0u, 0u};
    if (row < R) {
        int8_t q[32];
        if (SRC == 8) {
            const uint4* p = reinterpret_cast<const uint4*>(src + (int64_t)row * K + k0);
            const uint4 v0 = p[0], v1 = p[1];
            const uint32_t u[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
            for (int j = 0; j < 32; ++j) q[j] = (int8_t)((u[j >> 2] >> (8 * (j & 3))) & 0xFFu);
        } else {
            const uint4 v = *reinterpret_cast<const uint4*>(src + (int64_t)row * (K / 2) + k0 / 2);
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                const int nib = (int)((u[j >> 3] >> (4 * (j & 7))) & 0xFu);
                q[j] = (int8_t)((nib ^ 8) - 8);                     // sign-extend 4 bits
            }
        }
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            const int v = q[j];
            const int mag = min(v < 0 ? -v : v, 7);
            // E2M3 patterns of 0..7, one per byte
            const uint32_t e = (uint32_t)((0x1E1C1A1814100800ull >> (8 * mag)) & 0xFFu) | (v < 0 ? 32u : 0u);
            const int bit = 6 * j;
            w[bit >> 5] |= e << (bit & 31);
            if ((bit & 31) > 26) w[(bit >> 5) + 1] |= e >> (32 - (bit & 31));
        }
    }
    uint8_t* f = dst + frag * kFragBytes;
    *reinterpret_cast<uint4*>(f + lane * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint2*>(f + kFragLo + lane * 8) = make_uint2(w[4], w[5]);
}

// s_waitcnt vmcnt(n), lgkmcnt(0) for a wave-uniform n in [0, 12] (the instruction takes an immediate)
__device__ __forceinline__ void wait_vmcnt_upto(int n) {
    switch (n) {
        case 0: __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0)); break;
        case 1: __builtin_amdgcn_s_waitcnt(waitcnt_imm(1, 0)); break;
        case 2: __builtin_amdgcn_s_waitcnt(waitcnt_imm(2, 0)); break;
        case 3: __builtin_amdgcn_s_waitcnt(waitcnt_imm(3, 0)); break;
        case 4: __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 0)); break;
        case 5: __builtin_amdgcn_s_waitcnt(waitcnt_imm(5, 0)); break;
        case 6: __builtin_amdgcn_s_waitcnt(waitcnt_imm(6, 0)); break;
        case 7: __builtin_amdgcn_s_waitcnt(waitcnt_imm(7, 0)); break;
        case 8: __builtin_amdgcn_s_waitcnt(waitcnt_imm(8, 0)); break;
        case 9: __builtin_amdgcn_s_waitcnt(waitcnt_imm(9, 0)); break;
        case 10: __builtin_amdgcn_s_waitcnt(waitcnt_imm(10, 0)); break;
        case 11: __builtin_amdgcn_s_waitcnt(waitcnt_imm(11, 0)); break;
        default: __builtin_amdgcn_s_waitcnt(waitcnt_imm(12, 0)); break;
    }
}

// ---- fragments: LDS -> registers ---------------------------------------------------------------
struct frag6 {
    uint4 lo;
    uint2 hi;
};

__device__ __forceinline__ v8i as_operand(const frag6& f) {
    v8i v;
    v[0] = (int)f.lo.x; v[1] = (int)f.lo.y; v[2] = (int)f.lo.z; v[3] = (int)f.lo.w;
    v[4] = (int)f.hi.x; v[5] = (int)f.hi.y;
    v[6] = 0; v[7] = 0;
    return v;
}

// Where a piece of a fragment sits in LDS: the two 128-byte pieces of the second plane's second half change places
// (fragment-local byte offsets [1280, 1408) and [1408, 1536)); everything else is where the operand format has it.
__device__ __forceinline__ int lds_place(int frag_offset) {
    return frag_offset >= 1280 ? frag_offset ^ 128 : frag_offset;      // 1280 = 10 * 128: the xor swaps the two pieces
}

// Per-lane read offsets inside a slot, for the 16 x 16 tile made of the rows [16 p, 16 p + 16) of a 32-row block:
// lane l = row (l & 15), K chunk c = l >> 4 -> fragment c >> 1 along K, slot 16 p + (l & 15) + 32 (c & 1).
struct FragLane {
    int lo[2];             // 16-byte piece, p = 0 / 1
    int hi[2][2];          // 8-byte piece, [p][row block even / odd]
};
__device__ __forceinline__ FragLane frag_lane(int lane) {
    const int r = lane & 15, c = lane >> 4;
    FragLane f;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int slot = 16 * p + r + 32 * (c & 1);
        f.lo[p] = (c >> 1) * kFragBytes + slot * 16;
        f.hi[p][0] = (c >> 1) * kFragBytes + lds_place(kFragLo + slot * 8);
        // The odd row block's offset goes through an empty asm so that the compiler cannot see that it is the even
        // one's plus a constant: it would otherwise pair the 8-byte reads of two row blocks into one instruction
        // and then has to move the halves of its result next to each tile's 16-byte piece, waiting for the read first.
        f.hi[p][1] = f.hi[p][0] + 2 * kFragBytes;
        asm volatile("" : "+v"(f.hi[p][1]));
    }
    return f;
}
// tile `tile` (16 rows) of the operand rows that start at row block rb0 (even) of the slot
__device__ __forceinline__ frag6 read_tile(const int8_t* slot, int rb0, int tile, const FragLane& fl) {
    const int8_t* f_even = slot + (rb0 + ((tile >> 1) & ~1)) * (2 * kFragBytes);
    frag6 r;
    r.lo = *reinterpret_cast<const uint4*>(f_even + ((tile >> 1) & 1) * (2 * kFragBytes) + fl.lo[tile & 1]);
    r.hi = *reinterpret_cast<const uint2*>(f_even + fl.hi[tile & 1][(tile >> 1) & 1]);
    return r;
}

// Activation fragment first, as in the INT8 kernel (weights first runs 3 to 4 % slower): the accumulator tile has the
// instruction's natural orientation (lane l: channel l & 15 of the weight tile, tokens 4 (l >> 4) + register).
// Format 2 = FP6 E2M3 for both operands; scale operands 0 select the unscaled instruction.
__device__ __forceinline__ v4f mfma6(const frag6& a, const frag6& b, v4f acc) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(a), as_operand(b), acc, 2, 2, 0, 0, 0, 0);
}

// s_waitcnt vmcnt(n + 32), lgkmcnt(0) for a wave-uniform n in [0, 12]: the same with the 32 stores of the block's
// previous tile still allowed in flight
__device__ __forceinline__ void wait_vmcnt_upto_after_stores(int n) {
    static_assert(kEpilogue16Stores == 32, "the store count of the shared epilogue");
    switch (n) {
        case 0: __builtin_amdgcn_s_waitcnt(waitcnt_imm(32, 0)); break;
        case 1: __builtin_amdgcn_s_waitcnt(waitcnt_imm(33, 0)); break;
        case 2: __builtin_amdgcn_s_waitcnt(waitcnt_imm(34, 0)); break;
        case 3: __builtin_amdgcn_s_waitcnt(waitcnt_imm(35, 0)); break;
        case 4: __builtin_amdgcn_s_waitcnt(waitcnt_imm(36, 0)); break;
        case 5: __builtin_amdgcn_s_waitcnt(waitcnt_imm(37, 0)); break;
        case 6: __builtin_amdgcn_s_waitcnt(waitcnt_imm(38, 0)); break;
        case 7: __builtin_amdgcn_s_waitcnt(waitcnt_imm(39, 0)); break;
        case 8: __builtin_amdgcn_s_waitcnt(waitcnt_imm(40, 0)); break;
        case 9: __builtin_amdgcn_s_waitcnt(waitcnt_imm(41, 0)); break;
        case 10: __builtin_amdgcn_s_waitcnt(waitcnt_imm(42, 0)); break;
        case 11: __builtin_amdgcn_s_waitcnt(waitcnt_imm(43, 0)); break;
        default: __builtin_amdgcn_s_waitcnt(waitcnt_imm(44, 0)); break;
    }
}

// One output tile of 256 tokens x 256 channels starting at (m0, n0).  `prefetched`: the block's previous tile has
// requested this tile's first half tiles already; (next_m0, next_n0): the tile this one does that for (next_m0 < 0:
// none).
template <bool DEBUG, bool STREAM>
__device__ __forceinline__ void f6_tile(const uint8_t* __restrict__ qx6, const float* __restrict__ row_scale,
                                        const uint8_t* __restrict__ qw6, const float* __restrict__ w_scale, int T, int I,
                                        int O, uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_debug,
                                        int m0, int n0, int8_t* lds, bool prefetched, int next_m0, int next_n0) {
    constexpr int WN = 4, WTN = 64, G = 4;

    // (the thread id goes through an empty asm: the lane-dependent offsets below are then worked out again for every
    // tile of the block's walk instead of being kept, and spilled, across the whole loop over tiles)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int KB = I / 64;                        // fragments along K
    const int nk = I / 128;                       // K steps
    // Six LDS slots hold three tiles: half tile h (A(kt) = 2 kt, B(kt) = 2 kt + 1) lives in slot
    // h % 6, so requests run two to three steps ahead of their use (the loads' latency from the
    // memory-side cache is longer than one step).
    //   waves 0-3 ("early"): request B(kt+2) before the barrier of step kt; its slot was B(kt-1)'s,
    //                        released at barrier kt-1;
    //   waves 4-7 ("late"):  request A(kt+3) after the barrier of step kt (the early waves take a
    //                        share of it, see the loader below); its slot was A(kt)'s, which nobody
    //                        reads after that barrier.
    // One wave of every SIMD multiplies while its mate is held in load issue, as in the INT8 kernel.
    const bool late = wave >= 4;

    // ---- loader: a slot (half tile) is 24 instructions of 1 KiB.  Instruction n fills bytes
    // [1024 (n % 3), +1024) of the two consecutive fragments (3072 bytes) of row block n / 3 in LDS; a lane's
    // 16 bytes come from where lds_place puts them.  Row blocks past the end of a ragged operand are replaced
    // by the last valid one: what lands there only feeds outputs the epilogue drops.
    //   B(kt+2), before the barrier: early wave lw issues instructions 6 lw .. 6 lw + 5;
    //   A(kt+3), after the barrier:  late wave lw issues kLateA of them, early wave lw the other
    //                                kEarlyA = 6 - kLateA (the late waves are the critical path of a
    //                                step, the early ones would otherwise idle at the barrier).
    const int lw = wave & 3;
    constexpr int kEarlyA = 2, kLateA = 6 - kEarlyA;   // 0 / 6 measured ~4 % slower, 1..3 alike
    auto src_of = [&](const uint8_t* base, int first_rb, int last_rb, int n, int ln) {
        const int rb = min(first_rb + n / 3, last_rb);
        const int pair_offset = (n % 3) * 1024 + ln * 16;                    // where the 16 bytes land, in the pair
        const int frag = pair_offset >= kFragBytes ? 1 : 0;
        // (lds_place is its own inverse)
        return base + (int64_t)rb * KB * kFragBytes + frag * kFragBytes + lds_place(pair_offset - frag * kFragBytes);
    };
    const uint8_t* src_b[6];                      // early waves only
    const uint8_t* src_a[kLateA > kEarlyA ? kLateA : kEarlyA];
    const int n_a = late ? kLateA : kEarlyA;      // this wave's share of an A half tile ...
    const int a_first = late ? kLateA * lw : 4 * kLateA + kEarlyA * lw;   // ... starting at this instruction
    auto set_sources = [&](int tile_m0, int tile_n0) {
        // (worked out from scratch at each of the two calls rather than kept in registers in between)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        // (the weight operand always has whole groups of 64 channels, i.e. an even number of row blocks)
#pragma unroll
        for (int ii = 0; ii < 6; ++ii) src_b[ii] = src_of(qw6, tile_n0 / 32, 2 * ((O + 63) / 64) - 1, 6 * lw + ii, ln);
#pragma unroll
        for (int ii = 0; ii < (kLateA > kEarlyA ? kLateA : kEarlyA); ++ii)
            src_a[ii] = src_of(qx6, tile_m0 / 32, (T + 31) / 32 - 1, a_first + min(ii, n_a > 0 ? n_a - 1 : 0), ln);
    };
    set_sources(m0, n0);
    auto issue_b = [&](int kt, int slot) {        // early waves
        int8_t* dst = lds + slot * kF6Slot + lw * (6 * 1024);
        const int64_t koff = (int64_t)kt * (2 * kFragBytes);
#pragma unroll
        for (int ii = 0; ii < 6; ++ii) request_1k(src_b[ii] + koff, dst + ii * 1024);
    };
    auto issue_a = [&](int kt, int slot) {        // all waves, n_a instructions each
        int8_t* dst = lds + slot * kF6Slot + a_first * 1024;
        const int64_t koff = (int64_t)kt * (2 * kFragBytes);
        if (late) {
#pragma unroll
            for (int ii = 0; ii < kLateA; ++ii) request_1k(src_a[ii] + koff, dst + ii * 1024);
        } else {
#pragma unroll
            for (int ii = 0; ii < kEarlyA; ++ii) request_1k(src_a[ii] + koff, dst + ii * 1024);
        }
    };
    // requests of this wave that may still be in flight when tile kt+1 has to be complete: its share
    // of A(kt+2) and, for the early waves, B(kt+2)
    const int pend_a = n_a;

    const int a_rb = wm * 4, b_rb = wn * 2;       // first row block of this wave inside the A / B slot
    const FragLane fl = frag_lane(lane);

    v4f acc[8][G];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int ni = 0; ni < G; ++ni)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.0f;

    // prologue, oldest first: B0 A0 B1 A1 A2 (B by the early waves only); tile 0 must have landed,
    // the rest may still be in flight -- and, when the block's previous tile made these requests before its
    // epilogue, so may that tile's 32 stores, which are this wave's newest requests (the counter is decremented in
    // the order of issue)
    auto issue_prologue = [&]() {
        if (!late) issue_b(0, 1);
        issue_a(0, 0);
        if (nk > 1) {
            if (!late) issue_b(1, 3);
            issue_a(1, 2);
        }
        if (nk > 2) issue_a(2, 4);
    };
    {
        const int later = (nk > 1 ? (late ? 0 : 6) + pend_a : 0) + (nk > 2 ? pend_a : 0);
        if (!prefetched) {
            issue_prologue();
            wait_vmcnt_upto(later);
        } else {
            wait_vmcnt_upto_after_stores(later);
        }
    }
    __builtin_amdgcn_s_barrier();

    int sa = 0, sb = 1;
    auto adv = [](int v) { v += 2; return v >= kF6Slots ? v - kF6Slots : v; };

    // Fragment registers: the activation tiles 0-3 and 4-7 of a step alternate (a_lo, a_hi), the four weight tiles
    // are replaced one by one as the step's second half finishes with them.  A step is two phases of 16 matrix
    // instructions, walked weight tile by weight tile:
    //   phase 1: tokens 0-63   (a_lo x bf) while a_hi of this step is read;
    //   [requests, waits and the step's barrier]
    //   phase 2: tokens 64-127 (a_hi x bf) while a_lo and then bf of the next step are read, each weight tile
    //            after the four instructions that used its predecessor.
    frag6 a_lo[4], a_hi[4], bf[G];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) a_lo[mi] = read_tile(lds + sa * kF6Slot, a_rb, mi, fl);
#pragma unroll
    for (int ni = 0; ni < G; ++ni) bf[ni] = read_tile(lds + sb * kF6Slot, b_rb, ni, fl);

    // The arguments that only the epilogue uses are brought into registers here.  Left to the compiler their scalar
    // loads stay pending into the loop, and while one is pending every wait for an LDS read at the head of the loop has
    // to be a wait for all of them (scalar loads return out of order, on the same counter): the first matrix
    // instruction of a step then waits for the last read of the step before.
    asm volatile("" ::"s"(row_scale), "s"(w_scale), "s"(Y), "s"(ldy), "s"(acc_debug), "s"(T), "s"(O));
    auto k_step = [&](int kt, auto ahead2_c, auto ahead3_c, auto prefetch_c) {
        constexpr bool AHEAD2 = decltype(ahead2_c)::value;      // kt + 2 < nk
        constexpr bool AHEAD3 = decltype(ahead3_c)::value;      // kt + 3 < nk
        constexpr bool PREFETCH = decltype(prefetch_c)::value;  // kt + 1 < nk
        const int8_t* As = lds + sa * kF6Slot;
        const int na = adv(sa), nb = adv(sb);                   // slots of tile kt+1
        // phase 1
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) a_hi[mi] = read_tile(As, a_rb, 4 + mi, fl);
#pragma unroll
        for (int ni = 0; ni < G; ++ni)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[mi][ni] = mfma6(a_lo[mi], bf[ni], acc[mi][ni]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {                           // 8 reads, one after each of the first 8 instructions
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        __builtin_amdgcn_sched_barrier(0);
        // Before the barrier every wave makes sure its share of tile kt+1 has landed; requests are
        // served in order, so it is enough that at most the newest ones (its share of A(kt+2) and
        // B(kt+2)) are still in flight.  lgkmcnt(0): this wave's reads of tile kt are done (its slots
        // are handed over at the barrier).
        if (!late && AHEAD2) issue_b(kt + 2, adv(nb));          // B(kt+2) -> slot of B(kt-1)
        // (Constants to choose from: the general wait, a chain of compares and branches over the counts, stood in front of
        // every step's barrier; 4096 x 4096 x 4096 35.2 -> 34.1 us, 4096 x 8192 x 8192 124.7 -> 122.7.)
        if (AHEAD2) {
            // (in a prefetched tile's first step the previous tile's stores are still younger than tile 1's requests)
            const bool stores = prefetched && kt == 0;
            if (late) {
                if (stores) __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLateA + kEpilogue16Stores, 0));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLateA, 0));
            } else {
                if (stores) __builtin_amdgcn_s_waitcnt(waitcnt_imm(kEarlyA + 6 + kEpilogue16Stores, 0));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(kEarlyA + 6, 0));
            }
        } else {
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
        }
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (AHEAD3) issue_a(kt + 3, sa);                        // A(kt+3) -> slot of A(kt)
        __builtin_amdgcn_sched_barrier(0);
        // phase 2
        if (PREFETCH) {
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) a_lo[mi] = read_tile(lds + na * kF6Slot, a_rb, mi, fl);
        }
#pragma unroll
        for (int ni = 0; ni < G; ++ni) {
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[4 + mi][ni] = mfma6(a_hi[mi], bf[ni], acc[4 + mi][ni]);
            if (PREFETCH) bf[ni] = read_tile(lds + nb * kF6Slot, b_rb, ni, fl);
        }
        if (PREFETCH) {
            // reads 1-8 (a_lo) behind instructions 1-8, the weight tiles' behind 9-14, the last tile's after 16
#pragma unroll
            for (int i = 0; i < 14; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        sa = na;
        sb = nb;
    };
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;
    int kt = 0;
    for (; kt + 3 < nk; ++kt) k_step(kt, yes{}, yes{}, yes{});
    if (kt + 2 < nk) {
        k_step(kt, yes{}, no{}, yes{});
        ++kt;
    }
    if (kt + 1 < nk) {
        k_step(kt, no{}, no{}, yes{});
        ++kt;
    }
    EpilogueScales16<G> scales;
    epilogue16_load_scales<G>(scales, row_scale, w_scale, T, O, m0 + wm * 128, n0 + wn * WTN, lane);
    __builtin_amdgcn_sched_barrier(0);              // requested now, in flight during the last step
    k_step(kt, no{}, no{}, no{});

    // Every wave is past the last step's barrier and all requests have landed: the ring is free.  The prologue of the
    // block's next tile is requested now and travels while this tile's results are scaled and stored; the row
    // factors of the epilogue sit behind the ring.  (Not with DEBUG: the number of stores in flight is not fixed then.)
    if (!DEBUG && next_m0 >= 0) {
        set_sources(next_m0, next_n0);
        issue_prologue();
    }
    float* a_lds = reinterpret_cast<float*>(lds + kF6Ring + wave * 512);
    epilogue16_store<WTN, G, DEBUG, STREAM>(acc, a_lds, scales, Y, ldy, acc_debug, T, O, m0 + wm * 128, n0 + wn * WTN, lane);
    __builtin_amdgcn_sched_barrier(0);
}

// One block per CU (a block fills a CU's LDS) walks over several tiles, as in the INT8 kernel: block b belongs to XCD
// b % 8 and takes positions i, i + per, ... of that XCD's contiguous range of the tile walk, i = b / 8, per =
// gridDim.x / 8.
template <bool DEBUG, bool STREAM>
__global__ void __launch_bounds__(512)
gemm_f6_ring_kernel(const uint8_t* __restrict__ qx6, const float* __restrict__ row_scale,
                    const uint8_t* __restrict__ qw6, const float* __restrict__ w_scale, int T, int I, int O,
                    uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_debug, int tiles_m,
                    int tiles_n) {
    extern __shared__ __align__(16) int8_t lds[];
    const int xcd = blockIdx.x % kXcds, first = blockIdx.x / kXcds, per = gridDim.x / kXcds;
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + kXcds - 1) / kXcds;
    bool prefetched = false;
    for (int i = first; i < per_xcd; i += per) {
        const int L = xcd * per_xcd + i;
        if (L >= total) break;
        int tile_m, tile_n, next_m = -1, next_n = -1;
        tile_of_index(L, tiles_m, tiles_n, tile_m, tile_n);
        const bool has_next = i + per < per_xcd && L + per < total;
        if (has_next) tile_of_index(L + per, tiles_m, tiles_n, next_m, next_n);
        f6_tile<DEBUG, STREAM>(qx6, row_scale, qw6, w_scale, T, I, O, Y, ldy, acc_debug, tile_m * BM, tile_n * BN, lds,
                               prefetched, has_next ? next_m * BM : -1, next_n * BN);
        prefetched = has_next && !DEBUG;
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Smaller tiles for few tokens and small outputs, as in the INT8 path (gemm_i8_staged_kernel, whose schedule this is):
// 8 waves = WM x WN wave tiles of 16 MT tokens x 64 channels times WK shares of the contraction, whose partial sums
// meet in LDS.  A step is 128 WK elements; a slot holds [WK][(TM + TN) / 32 row blocks][two fragments along K].  Bound, as
// there, by what a CU takes in from its L2, and for a decode step by the weights' way from HBM.
// MU: the first activation tiles of a wave, which alone hold tokens (T <= 16 in tiles of 32, half of whose partial sums would change
// hands for nothing: 1 x 384 x 2728 5.7 -> 5.5 us, 16 x 512 x 1024 6.0 -> 5.8).
// ---------------------------------------------------------------------------------------------------------------
template <int MT, int WM, int WN, int WK, int S, bool ONCE, int MU>
__global__ void __launch_bounds__(64 * kSplitWaves)
gemm_f6_staged_kernel(const uint8_t* __restrict__ qx6, const float* __restrict__ row_scale,
                      const uint8_t* __restrict__ qw6, const float* __restrict__ w_scale, int T, int I, int O,
                      uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_debug, int tiles_m, int total) {
    static_assert(WM * WN * WK == kSplitWaves && MT % 2 == 0, "8 waves, whole row blocks");
    static_assert(MU == MT || (MU < MT && WM == 1), "the first tiles of the block's rows");
    constexpr int NT = 4, TM = 16 * MT * WM, TN = 64 * WN;
    constexpr int kRbA = TM / 32, kRb = (TM + TN) / 32, kPair = 2 * kFragBytes;
    constexpr int kSlot = WK * kRb * kPair, kRequests = kSlot / 1024;
    constexpr int N = (kRequests + kSplitWaves - 1) / kSplitWaves;        // per wave and step (the last one may be made twice)
    extern __shared__ __align__(16) int8_t lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = wave % (WM * WN), wk = wave / (WM * WN);
    const int wm = w / WN, wn = w % WN;
    const int64_t row_bytes = (int64_t)(I / 64) * kFragBytes;             // a row block's fragments
    const int nk128 = I / 128, nk = (nk128 + WK - 1) / WK;
    const bool early = WK > 2 && wave < 4;                               // see gemm_i8_staged_kernel
    const FragLane fl = frag_lane(lane);

    const int per_xcd = (total + kXcds - 1) / kXcds;
    for (int i = blockIdx.x / kXcds; i < per_xcd; i += gridDim.x / kXcds) {
        const int L = (blockIdx.x % kXcds) * per_xcd + i;
        if (L >= total) break;                                           // block-uniform
        const int tile_n = L / tiles_m;
        const int m0 = (L - tile_n * tiles_m) * TM, n0 = tile_n * TN;

        // request id = wave N + n of a step: KiB id % 3 of the pair of fragments of row block (id / 3) % kRb, share
        // id / (3 kRb).  Row blocks past the end are replaced by the last one (its outputs are dropped).
        const uint8_t* src[N];
        int share[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int id = min(wave * N + n, kRequests - 1), rb = (id / 3) % kRb;
            share[n] = id / (3 * kRb);
            const int pair_offset = (id % 3) * 1024 + lane * 16;
            const int frag = pair_offset >= kFragBytes ? 1 : 0;
            const uint8_t* base = rb < kRbA ? qx6 + min(m0 / 32 + rb, (T + 31) / 32 - 1) * row_bytes
                                            : qw6 + min(n0 / 32 + rb - kRbA, 2 * ((O + 63) / 64) - 1) * row_bytes;
            src[n] = base + frag * kFragBytes + lds_place(pair_offset - frag * kFragBytes) + share[n] * kPair;
        }
        // steps are taken from the end of the contraction: step 0 is its last, partly filled stretch, where shares past
        // the end read zeros
        auto request = [&](int kt, int slot) {                           // kt > 0
            const int64_t koff = (int64_t)(nk - 1 - kt) * (WK * kPair);
            const int8_t* dst = lds + slot * kSlot;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int id = min(wave * N + n, kRequests - 1);
                if (ONCE && (id / 3) % kRb >= kRbA) request_1k<true>(src[n] + koff, dst + id * 1024);
                else request_1k(src[n] + koff, dst + id * 1024);
            }
        };
        auto request_first = [&]() {
            const int64_t koff = (int64_t)(nk - 1) * (WK * kPair);
#pragma unroll
            for (int n = 0; n < N; ++n)
                request_1k((nk - 1) * WK + share[n] < nk128 ? static_cast<const void*>(src[n] + koff) : static_cast<const void*>(&g_zero_piece),
                           lds + min(wave * N + n, kRequests - 1) * 1024);
        };
        struct Frags {
            frag6 a[MU], b[NT];
        };
        const int share_base = wk * kRb * kPair;
        auto read = [&](Frags& f, int slot) {
            const int8_t* s = lds + slot * kSlot + share_base;
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) f.b[ni] = read_tile(s, kRbA + 2 * wn, ni, fl);
#pragma unroll
            for (int mi = 0; mi < MU; ++mi) f.a[mi] = read_tile(s, wm * MT / 2, mi, fl);
        };
        v4f acc[MU][NT];
#pragma unroll
        for (int mi = 0; mi < MU; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) acc[mi][ni] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

        // The scales first, held until the end.  (Behind the first requests, or a few steps before the end, the waits for
        // requests become waits for more of them: FP6 32 x 5120 x 20480 15.5 us, 15.8 and 17.3.  The fence keeps the loads here.)
        TileScales<MU, NT, WK> scales;
        tile_scales<MU, NT, WN, WK>(scales, row_scale, w_scale, T, O, m0, n0, w, wk, lane);
        asm volatile("" ::: "memory");
        request_first();
#pragma unroll
        for (int s = 1; s < S; ++s)
            if (s < nk) request(s, s);
        if (nk >= S) __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 1) * N, 15));           // step 0 has landed
        else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
        step_barrier();
        Frags f0, f1;
        read(f0, 0);

        int slot = 0;                                                    // slot of step kt
        auto step = [&](auto full_c, int kt, Frags& cur, Frags& nxt) {   // (see gemm_i8_staged_kernel)
            constexpr bool FULL = decltype(full_c)::value;
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(FULL ? (S - 2) * N : 63, 0));
            if (!FULL) {
                if (kt + S - 1 < nk) __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 2) * N, 15));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
            }
            step_barrier();
            const int next_slot = slot + 1 == S ? 0 : slot + 1;
            if (early && (FULL || kt + S < nk)) request(kt + S, slot);
            __builtin_amdgcn_sched_barrier(0);
            if (FULL || kt + 1 < nk) read(nxt, next_slot);
#pragma unroll
            for (int mi = 0; mi < MU; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) acc[mi][ni] = mfma6(cur.a[mi], cur.b[ni], acc[mi][ni]);
            __builtin_amdgcn_sched_barrier(0);
            if (!early && (FULL || kt + S < nk)) request(kt + S, slot);
            __builtin_amdgcn_sched_barrier(0);
            slot = next_slot;
        };
        using yes = std::integral_constant<bool, true>;
        using no = std::integral_constant<bool, false>;
        // (full steps only where there are many: for smaller tiles their code costs more, fetched once, than they save)
        constexpr bool kFullSteps = TM * TN >= 8192;
        int kt = 0;
        for (; kFullSteps && kt + 1 + S < nk; kt += 2) {
            step(yes{}, kt, f0, f1);
            step(yes{}, kt + 1, f1, f0);
        }
        for (; kt < nk; kt += 2) {
            step(no{}, kt, f0, f1);
            if (kt + 1 < nk) step(no{}, kt + 1, f1, f0);
        }
        __syncthreads();                                                 // the ring is free: it holds the partial sums now
        sum_and_store<MU, NT, WM, WN, WK>(acc, lds, scales, w, wk, lane, T, O, Y, ldy, acc_debug, m0, n0, true);
        __syncthreads();
    }
}

template <int MT, int WM, int WN, int WK, int S, bool ONCE = false, int MU = MT>
hipError_t launch_f6_staged(const uint8_t* qx6, const float* row_scale, const uint8_t* qw6, const float* w_scale, int T, int I,
                            int O, uint16_t* Y, int64_t ldy, int32_t* acc_debug, hipStream_t stream) {
    constexpr int TM = 16 * MT * WM, TN = 64 * WN;
    constexpr int kRing = S * WK * (TM + TN) / 32 * 2 * kFragBytes, kParts = kPartsBytes<MU, 4, WM, WN, WK>;
    constexpr int kLds = kRing > kParts ? kRing : kParts;
    static_assert(kLds <= 160 * 1024, "LDS budget of a gfx950 CU");
    const int tiles_m = (T + TM - 1) / TM;
    const int64_t total = (int64_t)tiles_m * ((O + TN - 1) / TN);
    if (total >= (int64_t)1 << 31) return hipErrorInvalidValue;
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_f6_staged_kernel<MT, WM, WN, WK, S, ONCE, MU>), kLds, allowed);
    if (e != hipSuccess) return e;
    const int64_t blocks = std::min<int64_t>((total + kXcds - 1) / kXcds * kXcds, (int64_t)1 << 20);
    gemm_f6_staged_kernel<MT, WM, WN, WK, S, ONCE, MU><<<dim3((unsigned)blocks), dim3(64 * kSplitWaves), kLds, stream>>>(
        qx6, row_scale, qw6, w_scale, T, I, O, Y, ldy, acc_debug, tiles_m, (int)total);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Tiles of 256 tokens x 32 NT channels (128, 192, 320 or 384), for outputs that 256 x 256 tiles do not divide over the CUs (the rule
// and what both take stand at w4a4_wide_tile): the structure of gemm_i8_wide_kernel (cq_gemm_wide.hip) on FP6 fragments.
//   8 waves in 4 x 2, wave tiles of 64 x 16 NT; a step is 128 elements, 4 + NT fragments for 4 NT matrix instructions (LDS reads
//   and writes of a step keep the LDS busy for 1050 / 1270 / 1780 / 2020 cycles, the matrix instructions the matrix cores for 510 /
//   770 / 1280 / 1540).
//   NT is even: a block's 32 NT channels are NT / 2 whole groups of 64.  Wave wn has NT / 4 of them to itself; of the one in the
//   middle that NT = 6 and 10 leave it takes the weight tiles 2 wn and 2 wn + 1.
//   LDS, NT = 10, 12: two buffers of activations, three slots of weights (141 / 160 KB).  The barrier near the end of step kt stands
//   behind the last reads of tile kt; what tile kt occupied is then requested for the activations of kt + 2 and the weights of
//   kt + 3, by the waves 0 to 3 at once, by 4 to 7 at the end of the step.  The weights are what no cache holds: with two slots of them 4096 x
//   4096 x 5120 takes 52.6 us instead of 49.2 where nothing is left in the caches, 4096 x 8192 x 5120 90.7 instead of 85.2.
//   NT = 4, 6: four / three slots of both (147 / 129 KB), since the steps are short: with the buffers of the others 2048 x 4096 x 5120
//   in tiles of 192 takes 37.2 us instead of 30.8 there, the ring 33.0.
// STREAM: Y is stored as a stream (see y_stays_cached), here nt alone: a wave writes a line in pieces, which have to meet in the L2.
//   With the ring's sc1 nt whole layers of 4096 x 5120 x 13824 and 2048 x 8192 x 28672 take 171 us and 231 instead of 158 and 220.
// ---------------------------------------------------------------------------------------------------------------
typedef int v6i __attribute__((ext_vector_type(6)));

// acc += a x b with the result in the same registers (see cq_gemm_wide.hip)
__device__ __forceinline__ void mfma6_in_place(v4f& acc, const v6i& a, const v6i& b) {
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:2 blgp:2" : "+v"(acc) : "v"(a), "v"(b));
}

// 16 bytes per lane from base + offset (base: scalar) to LDS at dst + 16 lane
__device__ __forceinline__ void request_at(const uint8_t* base, uint32_t offset, const int8_t* dst) {
    const uint32_t lds_off = (uint32_t)(uintptr_t)((lptr_t)dst);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 sc0" : : "v"(offset), "s"(base), "s"(lds_off) : "m0");
}

template <int NT, bool STREAM>
__global__ void __launch_bounds__(512)
gemm_f6_wide_kernel(const uint8_t* __restrict__ qx6, const float* __restrict__ row_scale, const uint8_t* __restrict__ qw6,
                    const float* __restrict__ w_scale, int T, int I, int O, uint16_t* __restrict__ Y, int64_t ldy, int tiles_m,
                    int tiles_n) {
    static_assert(NT % 2 == 0, "whole groups of 64 channels per block");
    constexpr int F = NT / 4, P = NT % 4 / 2;                // groups of 64 channels a wave has to itself, and shares
    constexpr int WTN = 16 * NT, BNW = 2 * WTN, kPair = 2 * kFragBytes;
    constexpr int kSets = NT < 12 ? 4 : 3;                   // weight tiles in registers: read kSets - 1 ahead (12: no room for more)
    constexpr bool kDeep = NT < 10;                          // the operands' tiles in kSlots slots each, requested kSlots - 1 steps ahead
    constexpr int kSlots = NT == 4 ? 4 : 3, kSlotsA = kDeep ? kSlots : 2;
    constexpr int kTileA = 8 * kPair, kTileB = NT * kPair, kReq = (8 + NT) * 3;  // LDS bytes; 1 KiB requests
    constexpr int N = (kReq + 7) / 8;                        // ... of a wave at most: ids wave, wave + 8, ...
    extern __shared__ __align__(16) int8_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nk = I / 128;
    const bool early = wave < 4;
    const bool all = wave < kReq - 8 * (N - 1);              // this wave has N requests, the others N - 1 (scalar)
    const int64_t row_bytes = (int64_t)(I / 64) * kFragBytes;

    const int total = tiles_m * tiles_n, per_xcd = (total + kXcds - 1) / kXcds;
    for (int i = blockIdx.x / kXcds; i < per_xcd; i += gridDim.x / kXcds) {
        const int L = (blockIdx.x % kXcds) * per_xcd + i;
        if (L >= total) break;                               // block-uniform
        int tile_m, tile_n;
        tile_of_index(L, tiles_m, tiles_n, tile_m, tile_n);
        const int m0 = tile_m * BM, n0 = tile_n * BNW;
        int tl = lane;                                       // (worked out for every tile, not kept and spilled)
        asm volatile("" : "+v"(tl));

        // request id: KiB id % 3 of the pair of fragments of row block id / 3; row blocks past an operand's end are replaced by its last
        const int a_last = (T + 31) / 32 - 1, b_last = 2 * ((O + 63) / 64) - 1;
        const uint8_t* src[N];                               // (scalar)
        uint32_t off[3];                                     // lane's bytes of ids wave, wave + 8, wave + 16, and every 24
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int id = wave + 8 * n, rb = id / 3;
            src[n] = rb < 8 ? qx6 + min(m0 / 32 + rb, a_last) * row_bytes : qw6 + min(n0 / 32 + rb - 8, b_last) * row_bytes;
            if (n < 3) {
                const int pair_offset = (id - 3 * rb) * 1024 + tl * 16, frag = pair_offset >= kFragBytes ? 1 : 0;
                off[n] = frag * kFragBytes + lds_place(pair_offset - frag * kFragBytes);
            }
        }
        auto request_a = [&](int kt, int buf) {              // ids 0 to 23
            const int8_t* dst = lds + buf * kTileA + wave * 1024;
#pragma unroll
            for (int n = 0; n < 3; ++n) request_at(src[n] + (int64_t)kt * kPair, off[n], dst + n * 8192);
        };
        auto request_b = [&](int kt, int slot) {             // slot: its byte offset from the first one
            const int8_t* dst = lds + (kSlotsA - 1) * kTileA + slot + wave * 1024;         // (n = 3: kTileA more)
#pragma unroll
            for (int n = 3; n < N; ++n)
                if (n < N - 1 || all) request_at(src[n] + (int64_t)kt * kPair, off[n % 3], dst + n * 8192);
        };

        v4f acc[4][NT];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                acc[mi][ni] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                asm volatile("" : "+v"(acc[mi][ni]));        // here, far ahead of the first matrix instruction
            }

        // the epilogue's scales: 256 row factors and, behind them, the steps of 64 ceil(NT / 2) channels
        int8_t* const scales = lds + kSlotsA * kTileA + kSlots * kTileB;
        if (wave < 4) request_words(row_scale + min(m0 + wave * 64 + tl, T - 1), scales + wave * 256);
        if (wave < NT / 2) request_words(w_scale + min(n0 + wave * 64 + tl, O - 1), scales + (4 + wave) * 256);
        if (kDeep) {
#pragma unroll
            for (int t = 0; t < kSlots; ++t)
                if (t < nk) {
                    request_a(t, t);
                    request_b(t, t * kTileB);
                }
            if (nk < kSlots) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
            else if (all) __builtin_amdgcn_s_waitcnt(waitcnt_imm((kSlots - 1) * N, 15));          // tile 0 has landed
            else __builtin_amdgcn_s_waitcnt(waitcnt_imm((kSlots - 1) * (N - 1), 15));
        } else {
            request_a(0, 0);
            request_b(0, 0);
            if (nk > 1) {
                request_b(1, kTileB);
                request_a(1, 1);
            }
            if (nk > 2) {
                request_b(2, 2 * kTileB);
                if (all) __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * N - 3, 15));          // tile 0 has landed
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * N - 5, 15));
            } else {
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
            }
        }
        step_barrier();

        // LDS addresses of a lane's fragment pieces: 16 bytes and 8 bytes, the latter for the two halves p of a row block
        // (frag_lane; the first half's 16 bytes are 256 further on in the second).  Through an empty asm, as in the INT8 kernel.
        struct At {
            uint32_t lo, hi[2];
        };
        At a_at, f_at, p_at;                                 // activations, a wave's own groups, the shared group
        {
            const int r = tl & 15, c = tl >> 4, slot = r + 32 * (c & 1);
            const uint32_t base = (uint32_t)(uintptr_t)((lptr_t)lds) + (c >> 1) * kFragBytes;
            auto at = [&](At& x, uint32_t o) {
                x = At{base + o + slot * 16, {base + o + lds_place(kFragLo + slot * 8), base + o + lds_place(kFragLo + (16 + slot) * 8)}};
                asm volatile("" : "+v"(x.lo), "+v"(x.hi[0]), "+v"(x.hi[1]));
            };
            at(a_at, wm * 2 * kPair);
            at(f_at, kSlotsA * kTileA + 2 * wn * (F + P) * kPair);
            at(p_at, kSlotsA * kTileA + (2 * F + wn) * kPair);
        }
        typedef int v2i __attribute__((ext_vector_type(2)));
        typedef __attribute__((address_space(3))) const v4i* lo_ptr;
        typedef __attribute__((address_space(3))) const v2i* hi_ptr;
        auto read = [&](v6i& f, const At& at, int tile, int buf_bytes) {      // 16 rows: half tile & 1 of row block tile >> 1
            const v4i lo = ((lo_ptr)at.lo)[(buf_bytes + (tile >> 1) * kPair + (tile & 1) * 256) / 16];
            const v2i hi = ((hi_ptr)at.hi[tile & 1])[(buf_bytes + (tile >> 1) * kPair) / 8];
            f = v6i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y};
        };
        v6i af[4], bf[kSets];
        auto read_a = [&](int buf, int mi) { read(af[mi], a_at, mi, kDeep ? 0 : buf * kTileA); };
        auto read_b = [&](int set, int s) {                  // of the slot that f_at and p_at stand at
            if (s < 4 * F) read(bf[set], f_at, s, 0);
            else read(bf[set], p_at, s - 4 * F, 0);
        };
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) read_a(0, mi);
#pragma unroll
        for (int s = 0; s < kSets - 1; ++s) read_b(s, s);

        int slot = 0;                                        // of the weights of step kt
        int slot_a = 0;                                      // kDeep: number of the slot of both operands
        // Step kt, its activations in buffer PAR.  FULL: tiles up to kt + 3 exist.  The last two weight tiles are multiplied activation tile by
        // activation tile, so that the next step's activations replace this one's as they are done with.
        auto k_step = [&](int kt, auto par_c, auto full_c) {
            constexpr int PAR = decltype(par_c)::value;
            constexpr bool FULL = decltype(full_c)::value;
            constexpr int kFirst = PAR * NT;                 // the sets rotate on through the two steps
            const bool land = FULL || kt + 1 < nk, more_a = FULL || kt + kSlotsA < nk, more_b = FULL || kt + kSlots < nk;
            const int freed = slot, on = slot == (kSlots - 1) * kTileB ? -(kSlots - 1) * kTileB : kTileB;
            const int freed_a = kDeep ? slot_a : PAR;
            auto ask = [&]() {                               // into what step kt leaves
                if (more_a) request_a(kt + kSlotsA, freed_a);
                if (more_b) request_b(kt + kSlots, freed);
            };
            auto turn = [&]() {
                // this wave's reads of tile kt are done and its requests for kt + 1 have landed: only the weights of kt + 2 may be under
                // way (kDeep: both operands of kt + 2 to kt + kSlots - 1)
                if (kDeep ? !(FULL || kt + kSlots - 1 < nk) : !more_a) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
                else if (all) __builtin_amdgcn_s_waitcnt(waitcnt_imm(kDeep ? (kSlots - 2) * N : N - 3, 0));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(kDeep ? (kSlots - 2) * (N - 1) : N - 4, 0));
                step_barrier();
                if (early) ask();
                slot += on;
                if (kDeep) {
                    const int on_a = slot_a == kSlots - 1 ? -(kSlots - 1) : 1;
                    slot_a += on_a;
                    a_at.lo += on_a * kTileA, a_at.hi[0] += on_a * kTileA, a_at.hi[1] += on_a * kTileA;
                }
                f_at.lo += on, f_at.hi[0] += on, f_at.hi[1] += on;
                if (P) p_at.lo += on, p_at.hi[0] += on, p_at.hi[1] += on;
                __builtin_amdgcn_sched_barrier(0);
            };
#pragma unroll
            for (int s = 0; s < NT - 2; ++s) {
                if (s == NT + 1 - kSets) turn();             // (three sets: behind this loop)
                if (s + kSets - 1 < NT) read_b((kFirst + s + kSets - 1) % kSets, s + kSets - 1);
                else if (land) read_b((kFirst + s + kSets - 1) % kSets, s + kSets - 1 - NT);
#pragma unroll
                for (int mi = 0; mi < 4; ++mi) mfma6_in_place(acc[mi][s], af[mi], bf[(kFirst + s) % kSets]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (kSets == 3) turn();
            if (land) read_b((kFirst + NT + kSets - 3) % kSets, kSets - 3);
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) {
                mfma6_in_place(acc[mi][NT - 2], af[mi], bf[(kFirst + NT - 2) % kSets]);
                mfma6_in_place(acc[mi][NT - 1], af[mi], bf[(kFirst + NT - 1) % kSets]);
                if (land) read_a(PAR ^ 1, mi);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (land) read_b((kFirst + NT + kSets - 2) % kSets, kSets - 2);
            if (!early) ask();
            __builtin_amdgcn_sched_barrier(0);
        };
        using even = std::integral_constant<int, 0>;
        using odd = std::integral_constant<int, 1>;
        using yes = std::integral_constant<bool, true>;
        using no = std::integral_constant<bool, false>;
        int kt = 0;
        for (; kt + kSlots + 1 < nk; kt += 2) {
            k_step(kt, even{}, yes{});
            k_step(kt + 1, odd{}, yes{});
        }
        for (; kt < nk; kt += 2) {
            k_step(kt, even{}, no{});
            if (kt + 1 < nk) k_step(kt + 1, odd{}, no{});
        }
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");    // the last matrix instructions' results ...
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)                      // ... are read behind this
            asm volatile("" : "+v"(acc[0][ni]), "+v"(acc[1][ni]), "+v"(acc[2][ni]), "+v"(acc[3][ni]));

        // Scale and store: 64 rows of the block's 32 NT channels as a raw buffer that ends at the last valid element
        int el = lane;
        asm volatile("" : "+v"(el));
        const int fr = el & 15, grp = el >> 4;
        const int row0 = m0 + wm * 64;
        const int first_four = 64 * wn * (F + P) + 4 * fr, first_pair = 64 * F + 4 * fr + 2 * wn;     // channels of the block
        const float* const row_f = reinterpret_cast<const float*>(scales) + wm * 64 + 4 * grp;
        const float* const step_f = reinterpret_cast<const float*>(scales) + BM;
        float s_own[NT];
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) s_own[ni] = step_f[ni < 4 * F ? first_four + 64 * (ni >> 2) + (ni & 3) : first_pair + ni - 4 * F];
        const int n_rows = min(64, T - row0), n_cols = min(BNW, O - n0), pitch = (int)ldy * 2;
        const int bytes = n_rows > 0 && n_cols > 0 ? (n_rows - 1) * pitch + n_cols * 2 : 0;
        const __amdgpu_buffer_rsrc_t yb = __builtin_amdgcn_make_buffer_rsrc(Y + (int64_t)row0 * ldy + n0, 0, bytes, 0x00020000);
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
            const float4 a4 = *reinterpret_cast<const float4*>(row_f + 16 * mi);
            const float a_own[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y[NT];
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) {
                    y[ni] = acc[mi][ni][r] * a_own[r];
                    y[ni] = rounded_f32(y[ni] * s_own[ni]);
                }
                const uint32_t row_off = (uint32_t)((16 * mi + 4 * grp + r) * pitch);
                // O % 8 == 0: the channels of a group exist or not together
                auto offset_of = [&](int c) { return (int)(c < n_cols ? row_off + 2 * c : 0x80000000u); };
                typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int g = 0; g < F; ++g)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2v{pack_half2(y[4 * g], y[4 * g + 1]), pack_half2(y[4 * g + 2], y[4 * g + 3])}, yb,
                                                          offset_of(first_four + 64 * g), 0, STREAM ? 2 : 0);
                if (P) __builtin_amdgcn_raw_buffer_store_b32(pack_half2(y[NT - 2], y[NT - 1]), yb, offset_of(first_pair), 0, STREAM ? 2 : 0);
            }
        }
        step_barrier();                                      // (every wave is past its last read of the tile's LDS)
    }
}

template <int NT, bool STREAM>
hipError_t launch_f6_wide(const uint8_t* qx6, const float* row_scale, const uint8_t* qw6, const float* w_scale, int T, int I, int O,
                          uint16_t* Y, int64_t ldy, int cu_blocks, hipStream_t stream) {
    constexpr int kSlots = NT == 4 ? 4 : 3, kLds = ((NT < 10 ? kSlots : 2) * 8 + kSlots * NT) * 2 * kFragBytes + (4 + NT / 2) * 256;
    static_assert(kLds <= 160 * 1024, "LDS of a gfx950 CU");
    static std::atomic<uint64_t> allowed{0};
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_f6_wide_kernel<NT, STREAM>), kLds, allowed);
    if (e != hipSuccess) return e;
    const int tiles_m = (T + BM - 1) / BM, tiles_n = (O + 32 * NT - 1) / (32 * NT), total = tiles_m * tiles_n;
    const int blocks = std::min(cu_blocks, (total + kXcds - 1) / kXcds * kXcds);
    gemm_f6_wide_kernel<NT, STREAM><<<dim3((unsigned)blocks), dim3(512), kLds, stream>>>(qx6, row_scale, qw6, w_scale, T, I, O, Y, ldy, tiles_m, tiles_n);
    return hipGetLastError();
}

// Which tile of the kernel above: 16-column weight tiles per wave (NT), or 0 for the ring's 256 x 256 tiles.  Measured with operands and
// results that nothing has left in the caches.  One round of 256 x 128 tiles is ahead of the ring, which half of the CUs have no tile in
// then, at every contraction (us, ring : here, I = 512, 1024, 2048, 4096, 8192):
//   1000 x I x 5120 (80 ring tiles, 160 of 256 x 128)           9.8 : 8.2     12.4 : 10.2   18.6 : 15.4   31.0 : 25.1   54 : 42
//   2048 x I x 4096 (128, 256)                                  11.1 : 10.1   14.5 : 12.8   20.7 : 18.3   32.2 : 27.7   56 : 46
// one round of 256 x 192 tiles only at long ones:
//   2048 x I x 5120 (160, 216 of 256 x 192)                     11.6 : 11.5   14.8 : 14.4   21.2 : 20.3   33.0 : 30.8   56 : 51
//   2048 x I x 6144 (192, 256)                                  12.3 : 12.8   15.8 : 19.1   22.2 : 23.3   34.6 : 33.2   60 : 55
// Where the ring needs more
// than one round over the CUs, in hundredths of a round of them: a round of 256 x 320 takes 126, of 256 x 384 139, from I = 4096 on
// (where first tiles and stores weigh less) 124 and 133:
//   4096 x I x 5120 (320 ring tiles, one round of 256 x 320)    21.8 : 17.0   28.8 : 21.8   42.5 : 31.2   67.3 : 49.1   120 : 85
//   2048 x I x 11008 (344, one round of 256 x 384)              22.8 : 18.0   30.1 : 22.9   43.0 : 32.7   68.1 : 51.9   120 : 92
//   4096 x I x 10240 (640, two rounds of 256 x 320)             28.6 : 31.2   39.4 : 39.8   59.3 : 55.8   99 : 87       187 : 158
//   4096 x I x 11008 (688, two of 256 x 384)                    32.5 : 33.6   43.2 : 43.3   62.2 : 61.0   102 : 95      191 : 174
//   4096 x I x 13824 (864, three of 256 x 320)                  38.0 : 41.4   51.8 : 53.4   78.5 : 76.4   131 : 121     246 : 222
//   4096 x I x 16384 (1024, three of 256 x 384)                                              85.3 : 85.4   145 : 142     270 : 260
//   4096 x I x 20480 (1280, four of 256 x 320)                                              103 : 105     176 : 169     333 : 312
//   4096 x I x 28672 (1792, five of 256 x 384)                  62.7 : 69.3   89.6 : 92.8   140 : 138     242 : 228
// so more than one round only from I = 2048 on (the ring requests a block's next tile under the stores of the last, here they
// follow each other).  With as many rounds as the ring the wider tiles lose: 4096 x 4096 x 4096 38.7 : 47.0, 256 x 256
// tiles in this kernel 42.1.
int w4a4_wide_tile(int T, int I, int O, int n_cu) {
    if (T < 256) return 0;
    auto rounds = [&](int bn) { return ((int64_t)((T + BM - 1) / BM) * ((O + bn - 1) / bn) + n_cu - 1) / n_cu; };
    if (rounds(128) == 1) return 4;
    if (rounds(192) == 1 && I >= 4096) return 6;
    if (rounds(BN) < 2) return 0;
    int64_t cost = 100 * rounds(BN);
    int nt = 0;
    for (const auto& [tiles, unit] : {std::pair<int, int>{10, I < 4096 ? 126 : 124}, {12, I < 4096 ? 139 : 133}}) {
        const int64_t r = rounds(32 * tiles);
        if ((r == 1 || I >= 2048) && r * unit < cost) {
            cost = r * unit;
            nt = tiles;
        }
    }
    return nt;
}

}  // namespace

int64_t fp6_packed_bytes(int64_t R, int64_t K) { return ((R + 31) / 32) * (K / 64) * (int64_t)kFragBytes; }
int64_t fp6_packed_weight_bytes(int64_t O, int64_t K) { return fp6_packed_bytes(((O + 63) / 64) * 64, K); }

hipError_t launch_pack_fp6(const void* codes, int src_format, bool weights, int R, int K, void* packed,
                           hipStream_t stream) {
    const int64_t row_blocks = weights ? 2 * (((int64_t)R + 63) / 64) : ((int64_t)R + 31) / 32;
    const int64_t n_slots = row_blocks * (K / 64) * 64;
    if (!grid_fits((n_slots + 255) / 256, 256)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((n_slots + 255) / 256)), block(256);
    const uint8_t* src = static_cast<const uint8_t*>(codes);
    uint8_t* dst = static_cast<uint8_t*>(packed);
    if (src_format == 8) {
        if (weights) pack_fp6_kernel<8, true><<<grid, block, 0, stream>>>(src, R, K, dst, n_slots);
        else pack_fp6_kernel<8, false><<<grid, block, 0, stream>>>(src, R, K, dst, n_slots);
    } else {
        if (weights) pack_fp6_kernel<4, true><<<grid, block, 0, stream>>>(src, R, K, dst, n_slots);
        else pack_fp6_kernel<4, false><<<grid, block, 0, stream>>>(src, R, K, dst, n_slots);
    }
    return hipGetLastError();
}

hipError_t launch_w4a4_linear(const void* qx6, const float* row_scale, const void* qw6, const float* w_scale, int T,
                              int I, int O, uint16_t* Y, int64_t ldy, int32_t* acc_debug, hipStream_t stream) {
    const int tiles_m = (T + BM - 1) / BM, tiles_n = (O + BN - 1) / BN;
    if (!grid_fits((int64_t)tiles_m * tiles_n + kXcds, 512)) return hipErrorInvalidValue;
    if (ldy >= ((int64_t)1 << 22)) return hipErrorInvalidValue;      // the epilogue's 32-bit byte offsets
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + kXcds - 1) / kXcds;
    int n_cu = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
        n_cu = 256;
    const uint8_t* qx = static_cast<const uint8_t*>(qx6);
    const uint8_t* qw = static_cast<const uint8_t*>(qw6);
    // Small tiles: the kind with the fewest rounds of tiles over the CUs times rows (TM + TN) a CU takes in per step, of equal
    // ones the larger tile.  Measured at I = 4096 (us; ring first, then 32 x 64, 64 x 64, 64 x 128, 128 x 128): 32 x 4096 26 : 7.7
    // 8.6 10.9 14.1; 256 x 4096 26 : 14.9 9.1 11.5 14.6; 512 x 4096 27 : 28 16.8 12.3 15.5; 1024 x 4096 28 : 57 32 24.0 18.1;
    // 2048 x 4096 (two rounds of the last) 31 : 123 76 48 34; and 32 x 5120 x 20480 32 : 21.7 21.0 15.5 17.3.
    static const int kinds[4][2] = {{128, 128}, {64, 128}, {64, 64}, {32, 64}};
    int64_t cost = INT64_MAX;
    int kind = -1;
    for (int k = 0; k < 4; ++k) {
        const int tm = kinds[k][0], tn = kinds[k][1];
        const int64_t tiles = (int64_t)((T + tm - 1) / tm) * ((O + tn - 1) / tn), c = (tiles + n_cu - 1) / n_cu * (tm + tn);
        if (c < cost) {
            cost = c;
            kind = k;
        }
    }
    // Taken where they are faster than the ring's rounds of 256 x 256 tiles, in that unit times the contraction (100000 are about
    // 1 us): up to 192 always, beyond with the fixed part of larger tiles or more rounds.  Around the line, us, small tiles : ring: 512 x
    // 128 x 4096 5.7 : 7.1 (192); 1024 x I x 4096 (256) 7.3 : 7.6 at I = 128, 8.1 : 9.3 at 512, 9.3 : 12.1 at 1024, 17.7 : 28.5 at 4096;
    // 60 x I x 33024 (384) 10.0 : 9.0 at 512, 18.0 : 18.0 at 2048, 57 : 52 at 8192; 16 x I x 98304 (576, two rounds of the
    // ring) 16.1 : 17.9 at 512, 57 : 74 at 4096; 128 x I x 81920 (768) 21.3 : 19.5 at 512, 66 : 76 at 4096.  The 930 was fitted to
    // earlier forms of the small tiles, so the line lies on the ring's side.
    const int64_t rounds = (total + n_cu - 1) / n_cu;
    const int64_t ring_time = rounds * ((int64_t)500 * I + 110000) - (int64_t)100 * I;
    // One round of 256 x 128 tiles (w4a4_wide_tile) is ahead of two rounds of 128 x 128 at every contraction, and of one of them at short
    // ones; the ring is behind both then.  128 x 128 : 256 x 128 : ring, us: 1000 x I x 4096 7.3 : 6.2 : 7.6 at I = 128, 8.0 : 7.7 : 9.3 at 512, 8.5 :
    // 8.25 : 9.9 at 640, 8.5 : 8.7 : 10.6 at 768, 9.0 : 9.2 : 11.2 at 896, 17.7 : 22.5 : 28.6 at 4096; 500 x I x 8192 8.4 : 8.2 : 10.0 at 640, 8.5 : 8.6 :
    // 10.6 at 768; 2000 x I x 2048 8.4 : 8.2 : 9.9 and 8.5 : 8.6 : 10.6.
    const int cu_blocks = n_cu >= kXcds ? n_cu / kXcds * kXcds : kXcds;      // the larger tiles: one block per CU, a multiple of the XCDs
    int wide = acc_debug ? 0 : w4a4_wide_tile(T, I, O, cu_blocks);
    const bool one_round = wide == 4 && cost <= 256;                         // of either
    if (one_round && I > 640) wide = 0;
    if (cost > 192 && (wide == 4 || (!one_round && cost * (I + 930) >= ring_time))) kind = -1;
    // weights that one row of tiles reads once and that no cache keeps: see launch_w8a8_staged (32 x 8192 x 28672 33.9 -> 32.2
    // us, 64 x 8192 x 28672 35.3 -> 34.1)
    const bool once = kind >= 0 && T <= kinds[kind][0] && (int64_t)O * I / 4 * 3 > (int64_t)128 << 20;
    switch (kind) {
        case 0:
            return once ? launch_f6_staged<4, 2, 2, 2, 3, true>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream)
                        : launch_f6_staged<4, 2, 2, 2, 3>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream);
        case 1:
            return once ? launch_f6_staged<2, 2, 2, 2, 4, true>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream)
                        : launch_f6_staged<2, 2, 2, 2, 4>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream);
        case 2: return launch_f6_staged<2, 2, 1, 4, 3>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream);
        case 3:
            return T <= 16 ? launch_f6_staged<2, 1, 1, 8, 2, false, 1>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream)
                           : launch_f6_staged<2, 1, 1, 8, 2>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, stream);
        default: break;
    }
    const bool stream_y = !y_stays_cached(T, O);
    switch (wide) {                                          // (one round of the first two is at most 24 MiB of Y)
        case 4: return launch_f6_wide<4, false>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream);
        case 6: return launch_f6_wide<6, false>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream);
        case 10:
            return stream_y ? launch_f6_wide<10, true>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream)
                            : launch_f6_wide<10, false>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream);
        case 12:
            return stream_y ? launch_f6_wide<12, true>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream)
                            : launch_f6_wide<12, false>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, cu_blocks, stream);
        default: break;
    }
    // four instances: with or without the raw accumulators, Y streamed to memory or left in the caches
    using kernel_t = void (*)(const uint8_t*, const float*, const uint8_t*, const float*, int, int, int, uint16_t*, int64_t,
                              int32_t*, int, int);
    static const kernel_t kernels[4] = {&gemm_f6_ring_kernel<false, false>, &gemm_f6_ring_kernel<false, true>,
                                        &gemm_f6_ring_kernel<true, false>, &gemm_f6_ring_kernel<true, true>};
    static std::atomic<uint64_t> lds_allowed[4];
    const int which = (acc_debug ? 2 : 0) + (stream_y ? 1 : 0);
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernels[which]), kF6Lds, lds_allowed[which]);
    if (e != hipSuccess) return e;
    const int blocks = std::min(cu_blocks, per_xcd * kXcds);
    kernels[which]<<<dim3((unsigned)blocks), dim3(512), kF6Lds, stream>>>(
        qx, row_scale, qw, w_scale, T, I, O, Y, ldy, acc_debug, tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace cq
