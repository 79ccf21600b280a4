// Pieces shared by the matrix-core GEMM kernels (INT8 codes, and INT4 codes carried as FP6).
#pragma once
#include "cq_kernels.h"

namespace cq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int BM = 256, BN = 256;   // block tile (tokens x output channels)
constexpr int kXcds = 8;            // block ids are dealt round-robin to this many L2 domains
constexpr int kGroupM = 4;          // tile-rows walked together (8, 16 and 1 measured slower)

// s_waitcnt immediate for gfx9-family encodings: vmcnt in bits 3:0 and 15:14, expcnt 6:4 (7 = no
// wait), lgkmcnt 11:8 (15 = no wait)
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 0xF) | ((vm >> 4) << 14) | (7 << 4) | (lgkm << 8); }

// Block id -> output tile.  Consecutive block ids land on different XCDs, so ids are first
// de-interleaved by XCD (each XCD gets a contiguous range of tiles, hence its own L2 sees a compact
// patch), then walked in groups of kGroupM tile-rows so that concurrently resident tiles share A
// rows and B columns.  Returns false for the padding blocks of the last XCD range.
// position L of the walk -> tile
__device__ __forceinline__ void tile_of_index(int L, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int group_sz = kGroupM * tiles_n;
    const int g = L / group_sz;
    const int gm = min(kGroupM, tiles_m - g * kGroupM);
    const int in_g = L - g * group_sz;
    tile_m = g * kGroupM + in_g % gm;
    tile_n = in_g / gm;
}
__device__ __forceinline__ bool tile_of_block(int block, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int total = tiles_m * tiles_n;
    const int per_xcd = (total + kXcds - 1) / kXcds;
    const int L = (block % kXcds) * per_xcd + block / kXcds;
    if (L >= total) return false;
    tile_of_index(L, tiles_m, tiles_n, tile_m, tile_n);
    return true;
}

// Store policy of Y in the ring kernels: up to 64 MiB it is written with plain stores, beyond that written through as a
// stream (see epilogue16_store).  Measured in a layer step: 2048 x 11008 outputs (43 MiB) 84.1 -> 82.5 us for the matrix
// kernel with plain stores and no change after it; 4096 x 20480 (160 MiB) and 4096 x 28672 (224 MiB) make the
// absmax call that follows 1.5 and 6 us slower with plain stores.
inline bool y_stays_cached(int T, int O) { return (int64_t)T * O * 2 <= (int64_t)64 << 20; }

// ---- Epilogue of the ring kernels, whose accumulator tiles are 16 x 16 (v_mfma_i32_16x16x64_i8 for INT8 codes,
// v_mfma_f32_16x16x128_f8f6f4 for INT4 codes carried as FP6; row0 / col0: first token / channel of the wave): lane l
// holds channel l & 15 of each tile and, in register r, token 4 (l >> 4) + r.  The kernel assigns the rows of its G weight tiles so that lane l's channels
// are the G consecutive ones G (l & 15) + ni: the G binary16 results of one token are 2 G adjacent bytes of Y, the
// 16 lanes of a group cover 32 G contiguous bytes of a token row (whole 128-byte lines for G = 4), and they are
// stored straight from registers, with no pass through LDS.  The wave's outputs are addressed as one raw buffer that
// ends with the last valid element, so the hardware's range check drops the rows past T; a lane whose channels lie
// past O gets an offset beyond any buffer.  No store is predicated: a wave always issues exactly 32 of them, which
// the kernel's hand-counted waits rely on.
// A lane needs the row factors of 4 consecutive tokens at a time; they go through 512 bytes of wave-private LDS
// (each lane requests two of its wave's 128 before the last step of the contraction).
template <int G>
struct EpilogueScales16 {
    float a_own[2];        // row factors of tokens row0 + lane and row0 + 64 + lane
    float s[G];            // column steps of channels col0 + G (lane & 15) + ni
};
template <int G>
__device__ __forceinline__ void epilogue16_load_scales(EpilogueScales16<G>& sc, const float* __restrict__ row_scale,
                                                       const float* __restrict__ w_scale, int T, int O, int row0, int col0,
                                                       int lane) {
    sc.a_own[0] = row_scale[min(row0 + lane, T - 1)];                 // rows >= T are never stored
    sc.a_own[1] = row_scale[min(row0 + 64 + lane, T - 1)];
#pragma unroll
    for (int ni = 0; ni < G; ++ni) sc.s[ni] = w_scale[min(col0 + G * (lane & 15) + ni, O - 1)];
}

constexpr int kEpilogue16Stores = 32;     // buffer stores per wave and tile (8 accumulator tiles x 4 registers)

// STREAM: Y is written through to memory as a stream (sc1 nt).  It is not read again here, and the memory-side cache
// is left without hundreds of MiB of dirty lines, so the kernel that runs next reads its cold input faster (64 MiB:
// 4 us less; of the policies tried -- plain, nt, sc1, sc1 nt, sc0 nt, sc0 sc1 nt -- this one gave the shortest
// following absmax + quantize calls).  A small Y (see y_stays_cached) fits the memory-side cache next to everything
// else of its layer: plain stores then, which make the kernel itself 2-3 % faster on such layers and change nothing
// after it.  DEBUG: the raw accumulators are stored as well (predicated stores; no fixed count then).
template <int WTN, int G, bool DEBUG, bool STREAM, typename ACC>
__device__ __forceinline__ void epilogue16_store(ACC (&acc)[8][G], float* a_lds, const EpilogueScales16<G>& sc,
                                                 uint16_t* __restrict__ Y, int64_t ldy, int32_t* __restrict__ acc_debug,
                                                 int T, int O, int row0, int col0, int lane) {
    static_assert(G == 2 || G == 4, "two or four channels per lane");
    static_assert(WTN == 16 * G, "G tiles of 16 channels");
    constexpr int kPolicy = STREAM ? 18 : 0;             // sc1 (16) | nt (2)
    const int fr = lane & 15, grp = lane >> 4;
    a_lds[lane] = sc.a_own[0];
    a_lds[64 + lane] = sc.a_own[1];
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, 0));      // wave-private: the writes above are done
    const int o_loc = G * fr;                            // first of this lane's G channels
    // the wave's 128 x WTN outputs as a buffer: rows [row0, T) and channels [col0, O) of them exist
    const int n_rows = min(128, T - row0), n_cols = min(WTN, O - col0);
    const int pitch = (int)ldy * 2;                      // bytes; 128 rows of it stay below 2^31 (checked by the launcher)
    const int bytes = (n_rows > 0 && n_cols > 0) ? (n_rows - 1) * pitch + n_cols * 2 : 0;
    const __amdgpu_buffer_rsrc_t yb =
        __builtin_amdgcn_make_buffer_rsrc(Y + (int64_t)row0 * ldy + col0, 0, bytes, 0x00020000);   // raw, 32-bit data
    // O % 8 == 0 on this path: a lane's G channels exist or not together
    const bool o_ok = o_loc < n_cols;
    const uint32_t lane_off = o_ok ? (uint32_t)(4 * grp * pitch + o_loc * 2) : 0x80000000u;
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) {
        const float4 a4 = *reinterpret_cast<const float4*>(a_lds + 16 * mi + 4 * grp);
        const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float y[G];
#pragma unroll
            for (int ni = 0; ni < G; ++ni) {
                y[ni] = (float)acc[mi][ni][r] * av[r];
                y[ni] = rounded_f32(y[ni] * sc.s[ni]);
            }
            const int off = (int)(lane_off + (uint32_t)((16 * mi + r) * pitch));
            if (G == 4) {
                typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
                __builtin_amdgcn_raw_buffer_store_b64(u32x2v{pack_half2(y[0], y[1]), pack_half2(y[G - 2], y[G - 1])}, yb, off, 0,
                                                      kPolicy);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(pack_half2(y[0], y[1]), yb, off, 0, kPolicy);
            }
            if (DEBUG) {
                const int t_loc = 16 * mi + 4 * grp + r;
                if (row0 + t_loc < T && o_ok) {
                    int32_t* d = acc_debug + (int64_t)(row0 + t_loc) * O + col0 + o_loc;
                    // (binary32 accumulators of the FP6 kernel hold exact integers)
                    if (G == 4)
                        *reinterpret_cast<int4*>(d) = make_int4((int)acc[mi][0][r], (int)acc[mi][1][r], (int)acc[mi][G - 2][r],
                                                                (int)acc[mi][G - 1][r]);
                    else
                        *reinterpret_cast<int2*>(d) = make_int2((int)acc[mi][0][r], (int)acc[mi][1][r]);
                }
            }
        }
    }
}

// ---- Pieces of the kernels with small tiles (8 waves whose contraction shares meet in LDS).
constexpr int kSplitWaves = 8;

// what requests for pieces past the contraction's end read
__device__ const uint4 g_zero_piece = {0u, 0u, 0u, 0u};

// One request: every lane's 16 bytes at src go to LDS at dst + 16 * lane (1 KiB per wave), without passing through
// registers; completion is counted by vmcnt.  Written as inline assembly rather than with the compiler's builtin: for
// the builtin the compiler makes every later LDS read wait until all such requests have landed (it cannot tell that the
// ring's slots differ), which would serialise requests made steps ahead with the reads of the current step.  The kernels
// order reads and in-flight writes themselves (slot discipline, explicit vmcnt waits, barriers).
// ONCE: the bytes are read by this block alone and not again (non-temporal).
template <bool ONCE = false>
__device__ __forceinline__ void request_1k(const void* src, const int8_t* dst) {
    const uint32_t lds_off = (uint32_t)(uintptr_t)((lptr_t)dst);     // wave-uniform
    if (ONCE) asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(src), "s"(lds_off) : "m0");
    else asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off sc0" : : "v"(src), "s"(lds_off) : "m0");
}

// 4 bytes per lane from src to LDS at dst + 4 lane
__device__ __forceinline__ void request_words(const float* src, const int8_t* dst) {
    const uint32_t lds_off = (uint32_t)(uintptr_t)((lptr_t)dst);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" : : "v"(src), "s"(lds_off) : "m0");
}

// The step barrier of those kernels: bare, since __syncthreads would wait for all requests in flight.  The barrier
// builtin orders no memory for the compiler, which sees neither the requests' writes to LDS nor a reason to keep a
// step's LDS reads behind the barrier: the empty asm says that memory may have changed (it adds no instruction).
__device__ __forceinline__ void step_barrier() {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The end of a tile.  The rows of a wave tile are dealt to the WK waves that share it: unit (mi, h) is the two tokens of
// accumulator registers 2 h, 2 h + 1 of the tiles (mi, 0 .. NT - 1), and wave wk ends up with the units [wk U, wk U + U)
// (with more waves than units the first ones have one each).  A wave keeps its own units' partial sums in registers and hands
// those of the others over in LDS.  Weight tile ni of a wave holds the channels NT fr + ni (fr = lane & 15) of the wave's 16 NT;
// lane l holds channel l & 15 of a weight tile and, in register r, token 4 (l >> 4) + r.
// What it costs beside the LDS traffic is latency, so the scales are requested at the tile's start (tile_scales).  Against all
// partial sums through LDS and the scales after that: 512 x 4096 x 4096 15.3 -> 14.3 us, 1024 x 4096 x 4096 22.0 -> 20.0, FP6 512
// x 4096 x 4096 14.0 -> 13.2, 1024 x 4096 x 4096 19.8 -> 17.0, 32 x 5120 x 20480 16.2 -> 15.5; a 16 x 512 x 1024 FP6 launch 6.0 -> 6.1.
template <int MT, int WK>
constexpr int kUnitsPerWave = 2 * MT >= WK ? 2 * MT / WK : 1;

// The scales a lane needs for its wave's units.
template <int MT, int NT, int WK>
struct TileScales {
    float s[NT];                            // steps of its NT channels
    float a[kUnitsPerWave<MT, WK>][2];      // factors of its tokens
};
template <int MT, int NT, int WN, int WK>
__device__ __forceinline__ void tile_scales(TileScales<MT, NT, WK>& sc, const float* __restrict__ row_scale,
                                            const float* __restrict__ w_scale, int T, int O, int m0, int n0, int w, int wk, int lane) {
    constexpr int U = kUnitsPerWave<MT, WK>;
    const int col = n0 + ((w % WN) * 16 + (lane & 15)) * NT, row = m0 + (w / WN) * 16 * MT + 4 * (lane >> 4);
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) sc.s[ni] = w_scale[min(col + ni, O - 1)];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int u = min(wk * U + i, 2 * MT - 1);
#pragma unroll
        for (int r = 0; r < 2; ++r) sc.a[i][r] = row_scale[min(row + 16 * (u >> 1) + 2 * (u & 1) + r, T - 1)];
    }
}

// LDS bytes of the partial sums that change hands
template <int MT, int NT, int WM, int WN, int WK>
constexpr int kPartsBytes = WM * WN * 2 * MT * (WK - 1) * NT * 64 * 8;

// vec_out: every lane's NT channels exist or not together and their 2 NT bytes of Y are aligned.
// V: four int32 or four binary32 values (sums of the FP6 products are integers below 2^24, exact in any order).
// Y leaves with plain stores whatever its size.  Outputs beyond 64 MiB come here only off the ring's layout: 4096 x 4112 x 20480
// (160 MiB) takes 582 us, and 686 with the absmax of a cold 4096 x 8192 matrix behind each (14.5 on its own), where the ring
// takes 254 and 264 for 4096 x 4096 x 20480.
template <int MT, int NT, int WM, int WN, int WK, typename V>
__device__ __forceinline__ void sum_and_store(const V (&acc)[MT][NT], int8_t* lds, const TileScales<MT, NT, WK>& sc, int w, int wk,
                                              int lane, int T, int O, uint16_t* __restrict__ Y, int64_t ldy,
                                              int32_t* __restrict__ acc_debug, int m0, int n0, bool vec_out) {
    constexpr int U = kUnitsPerWave<MT, WK>, kUnits = 2 * MT;
    typedef decltype(acc[0][0][0] + acc[0][0][0]) elem;
    typedef elem pair __attribute__((ext_vector_type(2)));
    // [w][unit][share of one of the other WK - 1 waves][ni][lane]
    pair* parts = reinterpret_cast<pair*>(lds) + w * (kUnits * (WK - 1) * NT * 64) + lane;
    pair own[U][NT];
#pragma unroll
    for (int k = 0; k < WK; ++k) {                           // (wave-uniform: registers cannot be indexed by wk)
        if (wk != k) continue;
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int owner = u / U;
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                const V& v = acc[u >> 1][ni];
                const pair p = {v[2 * (u & 1)], v[2 * (u & 1) + 1]};
                if (owner == k) own[u % U][ni] = p;
                else parts[((u * (WK - 1) + (k < owner ? k : k - 1)) * NT + ni) * 64] = p;
            }
        }
    }
    __syncthreads();
    if (wk * U >= kUnits) return;                            // more waves than units (scalar)
    const int col = n0 + ((w % WN) * 16 + (lane & 15)) * NT;
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int u = wk * U + i;
        const int row = m0 + (w / WN) * 16 * MT + 16 * (u >> 1) + 4 * (lane >> 4) + 2 * (u & 1);
        pair sum[NT];
#pragma unroll
        for (int ni = 0; ni < NT; ++ni) sum[ni] = own[i][ni];
#pragma unroll
        for (int p = 0; p < WK - 1; ++p)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) sum[ni] += parts[((u * (WK - 1) + p) * NT + ni) * 64];
        if (col >= O) continue;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (row + r >= T) break;
            float y[NT];
#pragma unroll
            for (int ni = 0; ni < NT; ++ni) {
                y[ni] = (float)sum[ni][r] * sc.a[i][r];
                y[ni] = rounded_f32(y[ni] * sc.s[ni]);
            }
            uint16_t* dst = Y + (int64_t)(row + r) * ldy + col;
            if (NT == 4 && vec_out) {
                *reinterpret_cast<uint2*>(dst) = make_uint2(pack_half2(y[0], y[1]), pack_half2(y[NT - 2], y[NT - 1]));
            } else if (NT == 2 && vec_out) {
                *reinterpret_cast<uint32_t*>(dst) = pack_half2(y[0], y[NT - 1]);
            } else {
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    if (col + ni < O) dst[ni] = (uint16_t)f2h(y[ni]);
            }
            if (acc_debug) {
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
                    if (col + ni < O) acc_debug[(int64_t)(row + r) * O + col + ni] = (int)sum[ni][r];
            }
        }
    }
}

}  // namespace
}  // namespace cq
