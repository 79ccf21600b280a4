// W8A8 linear layer for outputs that 256 x 256 tiles do not divide over the CUs but tiles of 256 tokens x 32 NT channels (160,
// 192, 288, 320 or 352) do in one round.
//
// 2048 x 4096 x 11008 is 344 tiles of 256 x 256: one round of 256 CUs and a second one, of half tiles, that costs 0.42 of a
// round; in tiles of 256 x 352 it is 256 tiles, one round of 1.37.  160 tiles of 256 x 256 leave 96 CUs idle; in tiles of
// 256 x 160 they are 256.  Against gemm_i8_ring_kernel (us): 2048 x 4096 x 11008 71.2 -> 67.2, 2048 x 4096 x 9216 67.8 -> 56.2, 2048 x
// 4096 x 10240 69.1 -> 61.5, 4096 x 5120 x 5120 91 -> 78, 2048 x 1024 x 9216 24.5 -> 21.9, 1024 x 4096 x 11008 40.6 -> 36.9, 1024 x
// 4096 x 8448 39.9 -> 32.7, 1024 x 1024 x 8448 15.7 -> 13.7.
//   - 8 waves in 4 x 2, wave tiles of 64 x 16 NT: 4 x NT accumulator tiles of 16 x 16 (176 registers with NT = 11).  A slab of
//     64 contraction bytes costs a wave 4 + NT fragment reads for 4 NT matrix instructions, 0.34 each with NT = 11 and 0.375 in
//     the 256 x 256 kernel.  With all CUs at work both are bound by the power of the matrix instructions and of
//     feeding them; what this one gains is the CUs that would idle.
//   - LDS holds two tiles, (256 + 32 NT) rows x 128 bytes each (2 x 76 KiB).  Behind the barrier near the end of step kt, where
//     the last fragments of tile kt are in registers, its half of the LDS takes the requests for tile kt + 2, which have
//     a whole step to land.  Waves 0-3, one per SIMD, make theirs before the step's last matrix instructions and waves 4-7
//     after, so that one wave of every SIMD multiplies meanwhile.
//   - Weight fragments are read three weight tiles ahead, into four sets of registers that rotate through the 2 NT
//     weight tiles of a step, the activation fragments of the next slab while one is multiplied.
//   - The scales wait in LDS, requested before the first operands.
#include <algorithm>
#include <type_traits>

#include "cq_gemm_common.h"

namespace cq {
namespace {

constexpr int BK = 128;

// Which of a wave's 16 NT channels fragment row f of its weight tile ni holds: tiles go in fours (then a pair, then one) whose
// rows are interleaved, so that a lane's accumulators are 4 (2, 1) adjacent channels.
template <int NT>
__device__ __forceinline__ int wide_channel(int ni, int f) {
    constexpr int kFours = NT / 4 * 4, kPairs = kFours + (NT - kFours) / 2 * 2;
    if (ni < kFours) return (ni >> 2) * 64 + 4 * f + (ni & 3);
    if (ni < kPairs) return kFours * 16 + 2 * f + (ni - kFours);
    return kPairs * 16 + f;
}

// 16 bytes per lane from base + offset (base: scalar) to LDS at dst + 16 lane
__device__ __forceinline__ void request_at(const int8_t* base, uint32_t offset, const int8_t* dst) {
    const uint32_t lds_off = (uint32_t)(uintptr_t)((lptr_t)dst);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 sc0" : : "v"(offset), "s"(base), "s"(lds_off) : "m0");
}

// acc += a x b with the result in the same registers.  Left to choose, the compiler gives most of the results registers of their
// own, for which there is no room, and spills.  It does not know the assembly for a matrix instruction: what writes acc by
// vector instructions before, or reads it after, has to keep the distance by itself.
__device__ __forceinline__ void mfma_in_place(v4i& acc, const v4i& a, const v4i& b) {
    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

template <int NT>
__global__ void __launch_bounds__(512)
gemm_i8_wide_kernel(const int8_t* __restrict__ qx, const float* __restrict__ row_scale, const int8_t* __restrict__ qw,
                    const float* __restrict__ w_scale, int T, int I, int O, uint16_t* __restrict__ Y, int64_t ldy, int tiles_m,
                    int tiles_n) {
    constexpr int WTN = 16 * NT, BNW = 2 * WTN;              // channels of a wave, of a block
    constexpr int kTile = (BM + BNW) * BK;                   // LDS bytes of one tile
    constexpr int kReq = (BM + BNW) / 8;                     // 1 KiB requests of one tile
    constexpr int N = (kReq + 7) / 8;                        // ... of a wave at most: ids wave, wave + 8, ...
    constexpr int kSeq = 2 * NT;                             // weight tiles of a step: two slabs
    extern __shared__ __align__(16) int8_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int fr = lane & 15, grp = lane >> 4;
    const int nk = I / BK;
    const bool early = wave < 4;
    const bool all = wave < kReq - 8 * (N - 1);              // this wave has N requests, the others N - 1 (scalar)

    const int total = tiles_m * tiles_n, per_xcd = (total + kXcds - 1) / kXcds;
    for (int i = blockIdx.x / kXcds; i < per_xcd; i += gridDim.x / kXcds) {
        const int L = (blockIdx.x % kXcds) * per_xcd + i;
        if (L >= total) break;                               // block-uniform
        int tile_m, tile_n;
        tile_of_index(L, tiles_m, tiles_n, tile_m, tile_n);
        const int m0 = tile_m * BM, n0 = tile_n * BNW;

        // request id fills LDS rows 8 id .. 8 id + 7 of a tile: lane l's 16 bytes are physical chunk l & 7 of row 8 id + (l >> 3),
        // logical chunk (l & 7) ^ ((row >> 1) & 7).  Rows past the end of an operand are replaced by its last one.
        const int8_t* a_base = qx + (int64_t)m0 * I;
        const int8_t* b_base = qw + (int64_t)n0 * I;
        uint32_t off[N];
        int load_lane = lane;
        asm volatile("" : "+v"(load_lane));
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int R = 8 * (wave + 8 * n) + (load_lane >> 3);
            const int chunk = ((load_lane & 7) ^ ((R >> 1) & 7)) * 16;
            int row;
            if (n < BM / 64) {
                row = min(R, T - 1 - m0);
            } else {
                const int b = R - BM, w = b / WTN, in = b - w * WTN;
                row = min(w * WTN + wide_channel<NT>(in >> 4, in & 15), O - 1 - n0);
            }
            off[n] = (uint32_t)row * (uint32_t)I + (uint32_t)chunk;
        }
        auto request = [&](int kt, int buf) {
            const int8_t* dst = lds + buf * kTile + wave * 1024;
#pragma unroll
            for (int n = 0; n < N; ++n)
                if (n < N - 1 || all) request_at((n < BM / 64 ? a_base : b_base) + (int64_t)kt * BK, off[n], dst + n * 8192);
        };

        v4i acc[4][NT];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                acc[mi][ni] = v4i{0, 0, 0, 0};
                asm volatile("" : "+v"(acc[mi][ni]));      // here, far ahead of the first matrix instruction
            }

        // the epilogue's scales: 256 row factors and, behind them, the steps of 64 ceil(NT / 2) channels
        int8_t* const scales = lds + 2 * kTile;
        if (wave < 4) request_words(row_scale + min(m0 + wave * 64 + load_lane, T - 1), scales + wave * 256);
        if (wave < (NT + 1) / 2) request_words(w_scale + min(n0 + wave * 64 + load_lane, O - 1), scales + (4 + wave) * 256);
        request(0, 0);
        if (nk > 1) {
            request(1, 1);
            if (all) __builtin_amdgcn_s_waitcnt(waitcnt_imm(N, 15));          // tile 0 has landed
            else __builtin_amdgcn_s_waitcnt(waitcnt_imm(N - 1, 15));
        } else {
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
        }
        step_barrier();

        const int sw = (grp ^ ((fr >> 1) & 7)) * 16;
        // LDS addresses of this lane's fragment rows in the two tiles and slabs.  They go through an empty asm: of what it can see
        // through the compiler keeps every sum with a tile's offset in a register of its own, and spills.
        typedef __attribute__((address_space(3))) const v4i* frag_ptr;
        uint32_t a_at[2][2], b_at[2][2];
#pragma unroll
        for (int buf = 0; buf < 2; ++buf)
#pragma unroll
            for (int slab = 0; slab < 2; ++slab) {
                const uint32_t base = (uint32_t)(uintptr_t)((lptr_t)lds) + buf * kTile + (sw ^ (slab * 64));
                a_at[buf][slab] = base + (wm * 64 + fr) * BK;
                b_at[buf][slab] = base + (BM + wn * WTN + fr) * BK;
                asm volatile("" : "+v"(a_at[buf][slab]), "+v"(b_at[buf][slab]));
            }
        v4i af[2][4], bf[4];
        auto read_a = [&](int buf, int slab, int mi) { af[slab][mi] = ((frag_ptr)a_at[buf][slab])[mi * 16 * BK / 16]; };
        auto read_b = [&](int set, int buf, int s) {         // weight tile s % NT of slab s / NT
            bf[set] = ((frag_ptr)b_at[buf][s / NT])[(s % NT) * 16 * BK / 16];
        };
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) read_a(0, 0, mi);
#pragma unroll
        for (int s = 0; s < 3; ++s) read_b(s, 0, s);

        // Step kt on buffer PAR.  FULL: tiles kt + 1 and kt + 2 exist.
        auto k_step = [&](int kt, auto par_c, auto full_c) {
            constexpr int PAR = decltype(par_c)::value;
            constexpr bool FULL = decltype(full_c)::value;
            constexpr int kFirst = PAR * kSeq;               // the sets rotate on through the two steps
            constexpr int kSlab1 = NT > 6 ? 2 : 1;           // where the second slab's activations are read
            const bool land = FULL || kt + 1 < nk, more = FULL || kt + 2 < nk;
#pragma unroll
            for (int s = 0; s < kSeq; ++s) {
                if (s == kSeq - 3) {
                    // this wave's reads of tile kt are done and its requests for kt + 1 have landed
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
                    step_barrier();
                    if (early && more) request(kt + 2, PAR);
                    __builtin_amdgcn_sched_barrier(0);
                    if (land) {
#pragma unroll
                        for (int mi = 0; mi < 4; ++mi) read_a(PAR ^ 1, 0, mi);
                    }
                }
                if (s + 3 < kSeq) read_b((kFirst + s + 3) % 4, PAR, s + 3);
                else if (land) read_b((kFirst + s + 3) % 4, PAR ^ 1, s + 3 - kSeq);
                if (s >= kSlab1 && s < kSlab1 + 4) read_a(PAR, 1, s - kSlab1);
#pragma unroll
                for (int mi = 0; mi < 4; ++mi) mfma_in_place(acc[mi][s % NT], af[s / NT][mi], bf[(kFirst + s) % 4]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!early && more) request(kt + 2, PAR);
            __builtin_amdgcn_sched_barrier(0);
        };
        using even = std::integral_constant<int, 0>;
        using odd = std::integral_constant<int, 1>;
        using yes = std::integral_constant<bool, true>;
        using no = std::integral_constant<bool, false>;
        int kt = 0;
        for (; kt + 3 < nk; kt += 2) {
            k_step(kt, even{}, yes{});
            k_step(kt + 1, odd{}, yes{});
        }
        for (; kt < nk; kt += 2) {
            k_step(kt, even{}, no{});
            if (kt + 1 < nk) k_step(kt + 1, odd{}, no{});
        }
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // the last matrix instructions' results (see mfma_in_place) ...
#pragma unroll
        for (int ni = 0; ni < NT; ++ni)                      // ... are read behind this
            asm volatile("" : "+v"(acc[0][ni]), "+v"(acc[1][ni]), "+v"(acc[2][ni]), "+v"(acc[3][ni]));

        // Scale and store: the wave's 64 x 16 NT outputs as a raw buffer that ends at the last valid element (rows past T are
        // dropped by its range check; a lane whose channels lie past O points beyond it).
        // (lane-dependent values are worked out here for every tile; kept across the loop over tiles they would be spilled)
        int tile_lane = lane;
        asm volatile("" : "+v"(tile_lane));
        const int fr = tile_lane & 15, grp = tile_lane >> 4;
        const int row0 = m0 + wm * 64, col0 = n0 + wn * WTN;
        const float* const row_f = reinterpret_cast<const float*>(scales) + wm * 64 + 4 * grp;
        const float* const step_f = reinterpret_cast<const float*>(scales) + BM + wn * WTN;
        float s_own[NT];
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) s_own[ni] = step_f[wide_channel<NT>(ni, fr)];
        const int n_rows = min(64, T - row0), n_cols = min(WTN, O - col0), pitch = (int)ldy * 2;
        const int bytes = n_rows > 0 && n_cols > 0 ? (n_rows - 1) * pitch + n_cols * 2 : 0;
        const __amdgpu_buffer_rsrc_t yb = __builtin_amdgcn_make_buffer_rsrc(Y + (int64_t)row0 * ldy + col0, 0, bytes, 0x00020000);
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
            const float4 a4 = *reinterpret_cast<const float4*>(row_f + 16 * mi);
            const float a_own[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y[NT];
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) {
                    y[ni] = (float)acc[mi][ni][r] * a_own[r];
                    y[ni] = rounded_f32(y[ni] * s_own[ni]);
                }
                const uint32_t row_off = (uint32_t)((16 * mi + 4 * grp + r) * pitch);
                // O % 8 == 0: the channels of a group exist or not together
                auto offset_of = [&](int ni) {
                    const int c = wide_channel<NT>(ni, fr);
                    return (int)(c < n_cols ? row_off + 2 * c : 0x80000000u);
                };
                typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
                constexpr int kFours = NT / 4 * 4;
#pragma unroll
                for (int ni = 0; ni < kFours; ni += 4)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2v{pack_half2(y[ni], y[ni + 1]), pack_half2(y[ni + 2], y[ni + 3])}, yb, offset_of(ni), 0, 0);
                if (NT % 4 >= 2)
                    __builtin_amdgcn_raw_buffer_store_b32(pack_half2(y[kFours], y[NT % 4 >= 2 ? kFours + 1 : 0]), yb, offset_of(kFours), 0, 0);
                if (NT % 2)
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)f2h(y[NT - 1]), yb, offset_of(NT - 1), 0, 0);
            }
        }
        step_barrier();                                      // (every wave is past its last read of the tile's LDS)
    }
}

}  // namespace

// The tile width (as NT) for an output, and the time of its one round in hundredths of a round of 256 x 256 tiles; 0 if none
// gets by with one round.  Measured at I = 1024 and 4096 (us, 256 x 256: 18 and 49): NT 5 13.7-14.2 and 33-35, 6 14.4-15.2 and
// 37-39, 9 21.1-21.9 and 54-56, 10 23.0 and 61.5, 11 25.2 and 67.2 (7 and 8: never ahead by more than 2 %).
int w8a8_wide_tile(int T, int O, int n_cu, int* units) {
    static const int kTiles[][2] = {{5, 75}, {6, 80}, {9, 117}, {10, 126}, {11, 137}};
    for (const auto& k : kTiles) {
        const int w = 32 * k[0];
        if ((int64_t)((T + BM - 1) / BM) * ((O + w - 1) / w) <= n_cu) {
            *units = k[1];
            return k[0];
        }
    }
    return 0;
}

hipError_t launch_w8a8_wide(const int8_t* qx, const float* row_scale, const int8_t* qw, const float* w_scale, int T, int I, int O,
                            uint16_t* Y, int64_t ldy, int nt, int n_cu, hipStream_t stream) {
    auto run = [&](auto nt_c) {
        constexpr int NT = decltype(nt_c)::value, kLds = 2 * (BM + 32 * NT) * BK + (4 + (NT + 1) / 2) * 256;
        static_assert(kLds <= 160 * 1024, "LDS of a gfx950 CU");
        static std::atomic<uint64_t> allowed{0};
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&gemm_i8_wide_kernel<NT>), kLds, allowed);
        if (e != hipSuccess) return e;
        const int tiles_m = (T + BM - 1) / BM, tiles_n = (O + 32 * NT - 1) / (32 * NT), total = tiles_m * tiles_n;
        const int cu_blocks = n_cu >= kXcds ? n_cu / kXcds * kXcds : kXcds;
        const int blocks = std::min(cu_blocks, (total + kXcds - 1) / kXcds * kXcds);
        gemm_i8_wide_kernel<NT><<<dim3((unsigned)blocks), dim3(512), kLds, stream>>>(qx, row_scale, qw, w_scale, T, I, O, Y, ldy, tiles_m, tiles_n);
        return hipGetLastError();
    };
    switch (nt) {
        case 5: return run(std::integral_constant<int, 5>{});
        case 6: return run(std::integral_constant<int, 6>{});
        case 9: return run(std::integral_constant<int, 9>{});
        case 10: return run(std::integral_constant<int, 10>{});
        default: return run(std::integral_constant<int, 11>{});
    }
}

}  // namespace cq
