// Per-output-channel weight quantization (Eq. 2) with an optional per-input-channel fold
// factor, written transposed ([O][I], contraction axis contiguous) for the integer GEMM.
// Weight preparation: done once per weight (or once per calibrated column scale).
//   W'_jk = fl32(f_j * W_jk);  s_k = fl32(max_j |W'_jk| / q_max);  qw_kj = clamp(rne(fl32(W'_jk / s_k)))
#include "cq_device.h"

namespace cq {
namespace {

__global__ void zero_u32_kernel(uint32_t* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

constexpr int64_t kCachedWeight = (int64_t)128 << 20;        // bytes of W up to which reads leave copies in the caches

// The step of a channel is fl32(max / q_max).  Rounded division by a constant does not change an order, so the largest
// rounded quotient is the rounded quotient of the largest value: steps can be formed before they are combined, and no
// pass over them has to follow.

// Steps where a launch has enough channels: a block owns 64 channels (128 bytes of a row) and reads all their rows, 128
// at a time; nothing has to be cleared first and nothing combined afterwards.
template <bool VEC>
__global__ void __launch_bounds__(1024)
weight_step_kernel(const uint16_t* __restrict__ W, int I, int O, const float* __restrict__ fold, float qmax,
                   float* __restrict__ s) {
    __shared__ float lds[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c8 = lane & 7, jr = threadIdx.x >> 3;
    const int k0 = blockIdx.x * 64 + c8 * 8;
    float m[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] = 0.0f;
    constexpr int U = 8;                                      // rows in flight per thread
    for (int j0 = jr; j0 < I; j0 += 128 * U) {
        uint4 v[U];
        float f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(j0 + 128 * u, I - 1);           // (the last row again: changes no maximum)
            v[u] = load8<VEC>(W + (int64_t)j * O, k0, O);
            f[u] = fold ? fold[j] : 1.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t w32[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float w = h2f((w32[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
                m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(f[u] * w));
            }
        }
    }
#pragma unroll
    for (int off = 8; off <= 32; off <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __shfl_xor(m[e], off, 64));
    if (lane < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds[wave][c8 * 8 + e] = m[e];
    }
    __syncthreads();
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && k < O) {
        float mm = 0.0f;
#pragma unroll
        for (int w = 0; w < 16; ++w) mm = __builtin_fmaxf(mm, lds[w][threadIdx.x]);
        s[k] = mm / qmax;
    }
}

// The same with the rows shared out over blocks, for too few channels to fill the chip that way: partial steps
// accumulated (as bit patterns of values >= 0) into s, which a kernel of its own has cleared.
// Block: 256 threads = 4 waves sharing 512 columns; each wave takes RPW consecutive rows.
template <int RPW, bool VEC>
__global__ void __launch_bounds__(256)
weight_colmax_kernel(const uint16_t* __restrict__ W, int I, int O, const float* __restrict__ fold, float qmax,
                     uint32_t* __restrict__ s_bits, int n_col_chunks) {
    __shared__ float lds[4][8][kLanes];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col_chunk = blockIdx.x % n_col_chunks, row_chunk = blockIdx.x / n_col_chunks;
    const int k0 = col_chunk * 512 + lane * 8;
    const int j_begin = row_chunk * (4 * RPW) + wave * RPW;
    float m[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] = 0.0f;
    // batches of 8 rows: all eight loads are issued before the first value is used
    for (int jb = 0; jb < RPW; jb += 8) {
        const int j8 = j_begin + jb;
        if (j8 >= I) break;                              // wave-uniform
        uint4 v[8];
        float f[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int j = min(j8 + r, I - 1);
            v[r] = load8<VEC>(W + (int64_t)j * O, k0, O);
            f[r] = fold ? fold[j] : 1.0f;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint32_t w32[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float w = h2f((w32[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
                m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(f[r] * w));
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) lds[wave][e][lane] = m[e];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 8 * kLanes; idx += 256) {
        const int e = idx / kLanes, ln = idx % kLanes;
        const float v = __builtin_fmaxf(__builtin_fmaxf(lds[0][e][ln], lds[1][e][ln]), __builtin_fmaxf(lds[2][e][ln], lds[3][e][ln]));
        const int k = col_chunk * 512 + ln * 8 + e;
        const uint32_t bits = __float_as_uint(v / qmax);
        if (k < O && bits) atomicMax(&s_bits[k], bits);
    }
}

// Codes of one 128 SWEEPS (input channels j) x 64 (output channels k) tile, with given steps (GROUPED false) or with the
// steps of its own groups of g input channels (32, 64, 128 or 256; g divides 128 SWEEPS): the tile is read once and held
// in registers.  A thread works on 8 channels of 4 consecutive rows, so that its codes leave for LDS four at a time (a
// byte at a time, as before, this transposition was the larger part of the kernel's instructions); rows of the
// transposed tile are 33 (65) words apart, which puts the 64 words a wave writes at a time on 64 distinct banks.
// The correctly rounded division is taken only where it can matter (as in the activation quantizer): w * (1/s) is
// rounded to an integer by one fma against 1.5 * 2^23 (the sum's ulp is 1), a second fma gives the distance from it, and
// a wave in which any lane is within the approximation's error of a rounding tie (or has a step so small that its
// reciprocal leaves the normal range) redoes its eight elements with the division.
// Bound by the memory: 4096 x 11008 per channel (steps + codes) 65 -> 42 us, 5120 x 20480 in groups of 128 with the
// dequantized weights 156 -> 106 us = 4.9 TB/s (the group was read twice before).  Outputs leave with non-temporal stores
// (118.6 us for the latter with plain ones, 119.5 written through): they do not push the weights out of the caches.
template <int SWEEPS, bool GROUPED, bool VEC, bool ONCE = false>
__global__ void __launch_bounds__(256)
weight_tile_kernel(const uint16_t* __restrict__ W, int I, int O, const float* __restrict__ fold, int g, float qmax,
                   int8_t* __restrict__ qw, float* __restrict__ s, uint16_t* __restrict__ wdq, int n_k_tiles, bool qw_vec,
                   bool dq_vec, int strip) {
    constexpr int kJ = 128 * SWEEPS, kPitch = kJ / 4 + 1;          // words
    __shared__ uint32_t tile[64 * kPitch];
    __shared__ float lmax[GROUPED ? 4 * SWEEPS : 1][64];
    __shared__ float lstep[GROUPED ? 4 * SWEEPS : 1][64];
    // Walk: with given steps, down the rows of one set of channels, the last channels first -- what the pass over the steps
    // read last is still in the memory-side cache (8192 x 28672, plain loads: 222 us for the call against 259 along them; equal
    // for weights that fit the cache); else along the channels (4096 x 11008, g = 128: 43.5 us against 51), `strip` row tiles
    // at a time.
    const int n_j_tiles = gridDim.x / n_k_tiles;
    int kt, jt;
    if (GROUPED) {
        const int first = (int)blockIdx.x / (n_k_tiles * strip) * strip, height = min(strip, n_j_tiles - first);
        const int at = (int)blockIdx.x - first * n_k_tiles;
        kt = at / height;
        jt = first + at - kt * height;
    } else {
        kt = n_k_tiles - 1 - blockIdx.x / n_j_tiles;
        jt = blockIdx.x % n_j_tiles;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c8 = lane & 7, jq = threadIdx.x >> 3;
    const int k0 = kt * 64 + c8 * 8, j_base = jt * kJ;
    constexpr float kRound = 12582912.0f;             // 1.5 * 2^23
    constexpr float kTol = 1.9073486328125e-06f;      // 2^-19; the approximation is within 2^-22

    uint4 v[SWEEPS][4];
    float f[SWEEPS][4];
#pragma unroll
    for (int sw = 0; sw < SWEEPS; ++sw)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = j_base + sw * 128 + jq * 4 + r;
            const uint16_t* row = W + (int64_t)j * O;
            v[sw][r] = make_uint4(0u, 0u, 0u, 0u);
            if (VEC && ONCE) {                                // the last read of W, and no cache keeps it for the next call
                if (j < I && k0 < O) v[sw][r] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + k0)));
            } else if (j < I) {
                v[sw][r] = load8<VEC>(row, k0, O);
            }
            f[sw][r] = (fold && j < I) ? fold[j] : 1.0f;
        }
    auto weights_of = [&](int sw, int r, float (&w)[8]) {
        const uint32_t w32[4] = {v[sw][r].x, v[sw][r].y, v[sw][r].z, v[sw][r].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = f[sw][r] * h2f((w32[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
    };

    if (GROUPED) {
        // the 32 rows of a wave and sweep, then the g / 32 of those that make a group
#pragma unroll
        for (int sw = 0; sw < SWEEPS; ++sw) {
            float m[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) m[e] = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float w[8];
                weights_of(sw, r, w);
#pragma unroll
                for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(w[e]));
            }
#pragma unroll
            for (int off = 8; off <= 32; off <<= 1)
#pragma unroll
                for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __shfl_xor(m[e], off, 64));
            if (lane < 8) {
#pragma unroll
                for (int e = 0; e < 8; ++e) lmax[sw * 4 + wave][c8 * 8 + e] = m[e];
            }
        }
        __syncthreads();
        const int per = g / 32, ng = I / g;
        for (int idx = threadIdx.x; idx < 4 * SWEEPS / per * 64; idx += 256) {
            const int G = idx >> 6, kl = idx & 63;
            float mm = 0.0f;
            for (int p = 0; p < per; ++p) mm = __builtin_fmaxf(mm, lmax[G * per + p][kl]);
            const float step = mm / qmax;
            for (int p = 0; p < per; ++p) lstep[G * per + p][kl] = step;
            const int k = kt * 64 + kl, group = j_base / g + G;
            if (k < O && group < ng) s[(int64_t)k * ng + group] = step;
        }
        __syncthreads();
    }

    float sk[8], rs[8];
    bool odd_step = false;
#pragma unroll
    for (int sw = 0; sw < SWEEPS; ++sw) {
        if (GROUPED || sw == 0) {
            odd_step = false;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sk[e] = GROUPED ? lstep[sw * 4 + wave][c8 * 8 + e] : ((k0 + e < O) ? s[k0 + e] : 0.0f);
                rs[e] = (sk[e] == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(sk[e]);
                odd_step |= sk[e] != 0.0f && !(sk[e] >= 7.888609052210118e-31f);     // 2^-100, also catches NaN
            }
        }
        uint32_t packed[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) packed[e] = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float w[8], m[8], q[8];
            weights_of(sw, r, w);
            float score = 0.0f, big = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                m[e] = __builtin_fmaf(w[e], rs[e], kRound);
                q[e] = m[e] - kRound;
                const float d = __builtin_fmaf(w[e], rs[e], -q[e]);
                score = __builtin_fmaxf(score, __builtin_fmaf(__builtin_fabsf(q[e]), kTol, __builtin_fabsf(d)));
                big = __builtin_fmaxf(big, __builtin_fabsf(q[e]));
            }
            if (__any(score >= 0.5f - kTol || !(big <= qmax) || odd_step)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float d = (sk[e] == 0.0f) ? 0.0f : w[e] / sk[e];
                    d = __builtin_rintf(d);
                    q[e] = __builtin_fminf(__builtin_fmaxf(d, -qmax), qmax) + 0.0f;      // -0 (from rounding e.g. -0.3) -> +0
                    m[e] = q[e] + kRound;
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)                                     // byte r <- the code, the low byte of m
                packed[e] = __builtin_amdgcn_perm(__float_as_uint(m[e]), packed[e],
                                                  r == 0 ? 0x03020104u : (r == 1 ? 0x03020400u : (r == 2 ? 0x03040100u : 0x04020100u)));
            const int j = j_base + sw * 128 + jq * 4 + r;
            if (wdq && j < I) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = rounded_f32(q[e] * sk[e]);
                uint16_t* dst = wdq + (int64_t)j * O + k0;
                if (dq_vec) {
                    if (k0 < O)
                        __builtin_nontemporal_store(u32x4{pack_half2(y[0], y[1]), pack_half2(y[2], y[3]), pack_half2(y[4], y[5]),
                                                          pack_half2(y[6], y[7])},
                                                    reinterpret_cast<u32x4*>(dst));
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (k0 + e < O) dst[e] = (uint16_t)f2h(y[e]);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[(c8 * 8 + e) * kPitch + sw * 32 + jq] = packed[e];
    }
    __syncthreads();
    // 64 rows (k) of 128 SWEEPS bytes (j): 8 SWEEPS threads a row, 16 bytes each
    constexpr int kPieces = 8 * SWEEPS;
#pragma unroll
    for (int i = 0; i < 64 * kPieces / 256; ++i) {
        const int idx = i * 256 + threadIdx.x, kl = idx / kPieces, piece = idx % kPieces;
        const int k = kt * 64 + kl, j = j_base + piece * 16;
        if (k >= O || j >= I) continue;
        const uint32_t* src = &tile[kl * kPitch + piece * 4];
        const u32x4 w4 = {src[0], src[1], src[2], src[3]};
        int8_t* dst = qw + (int64_t)k * I + j;
        if (qw_vec && j + 16 <= I) {
            __builtin_nontemporal_store(w4, reinterpret_cast<u32x4*>(dst));
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (j + e < I) dst[e] = (int8_t)((w4[e >> 2] >> (8 * (e & 3))) & 0xFFu);
        }
    }
}

// Group-wise variant: every output channel is cut into groups of g consecutive input channels,
// each with its own step (Background section's group-wise quantization).  One block handles one
// group of one 64-channel tile: pass 1 finds the 64 group maxima, pass 2 quantizes, transposes
// through LDS 32 input channels at a time, and optionally writes the dequantized weights.
__global__ void __launch_bounds__(256)
weight_group_kernel(const uint16_t* __restrict__ W, int I, int O, const float* __restrict__ fold, int g,
                    float qmax, int8_t* __restrict__ qw, float* __restrict__ s, uint16_t* __restrict__ wdq,
                    int n_k_tiles, bool in_vec, bool out_vec) {
    __shared__ float lmax[32][64 + 1];
    __shared__ float lstep[64];
    __shared__ __align__(16) int8_t tile[64][128 + 16];        // [k][j within the 128-row chunk]
    const int kt = blockIdx.x % n_k_tiles, G = blockIdx.x / n_k_tiles;
    const int ng = I / g;
    const int c8 = threadIdx.x & 7, jr = threadIdx.x >> 3;
    const int k0 = kt * 64 + c8 * 8;
    const int j_begin = G * g, j_end = j_begin + g;

    auto load_row = [&](int j, float (&w)[8]) {
        uint32_t h[8];
        const uint16_t* row = W + (int64_t)j * O;
        if (in_vec && k0 + 8 <= O) {
            const uint4 v = *reinterpret_cast<const uint4*>(row + k0);
            h[0] = v.x & 0xFFFFu; h[1] = v.x >> 16; h[2] = v.y & 0xFFFFu; h[3] = v.y >> 16;
            h[4] = v.z & 0xFFFFu; h[5] = v.z >> 16; h[6] = v.w & 0xFFFFu; h[7] = v.w >> 16;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = (k0 + e < O) ? row[k0 + e] : 0u;
        }
        const float f = fold ? fold[j] : 1.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            w[e] = h2f(h[e]);
            if (fold) w[e] = f * w[e];
        }
    };

    float m[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] = 0.0f;
    for (int j = j_begin + jr; j < j_end; j += 32) {
        float w[8];
        load_row(j, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(w[e]));
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) lmax[jr][c8 * 8 + e] = m[e];
    __syncthreads();
    if (threadIdx.x < 64) {
        float mm = 0.0f;
        for (int r = 0; r < 32; ++r) mm = __builtin_fmaxf(mm, lmax[r][threadIdx.x]);
        const float step = mm / qmax;
        lstep[threadIdx.x] = step;
        const int k = kt * 64 + threadIdx.x;
        if (k < O) s[(int64_t)k * ng + G] = step;
    }
    __syncthreads();
    // the division is taken only near a rounding tie, as in weight_tile_kernel
    constexpr float kRound = 12582912.0f;             // 1.5 * 2^23
    constexpr float kTol = 1.9073486328125e-06f;      // 2^-19
    float sk[8], rs[8];
    bool odd_step = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        sk[e] = lstep[c8 * 8 + e];
        rs[e] = (sk[e] == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(sk[e]);
        odd_step |= sk[e] != 0.0f && !(sk[e] >= 7.888609052210118e-31f);     // 2^-100, also catches NaN
    }

    // up to 128 input channels of the group at a time (4 passes of 32 rows), so that the codes leave
    // in whole 128-byte row pieces where the group is that long
    for (int jc = j_begin; jc < j_end; jc += 128) {
        const int jc_end = min(jc + 128, j_end);
#pragma unroll
        for (int sub = 0; sub < 4; ++sub) {
            const int j = jc + sub * 32 + jr;
            const bool live = j < jc_end;
            float w[8], q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = 0.0f;
            if (live) load_row(j, w);
            float score = 0.0f, big = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float mm = __builtin_fmaf(w[e], rs[e], kRound);
                q[e] = mm - kRound;
                const float d = __builtin_fmaf(w[e], rs[e], -q[e]);
                score = __builtin_fmaxf(score, __builtin_fmaf(__builtin_fabsf(q[e]), kTol, __builtin_fabsf(d)));
                big = __builtin_fmaxf(big, __builtin_fabsf(q[e]));
            }
            if (__any(score >= 0.5f - kTol || !(big <= qmax) || odd_step)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float r = (sk[e] == 0.0f) ? 0.0f : w[e] / sk[e];
                    r = __builtin_rintf(r);
                    q[e] = __builtin_amdgcn_fmed3f(r, -qmax, qmax) + 0.0f;      // -0 (from rounding e.g. -0.3) -> +0
                }
            }
            if (live) {
                uint32_t hq[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    tile[c8 * 8 + e][sub * 32 + jr] = (int8_t)(int)q[e];
                    hq[e] = f2h(rounded_f32(q[e] * sk[e]));
                }
                if (wdq) {
                    uint16_t* dst = wdq + (int64_t)j * O + k0;
                    if (in_vec && k0 + 8 <= O && (reinterpret_cast<uintptr_t>(wdq) % 16 == 0)) {
                        *reinterpret_cast<uint4*>(dst) = make_uint4(hq[0] | (hq[1] << 16), hq[2] | (hq[3] << 16),
                                                                    hq[4] | (hq[5] << 16), hq[6] | (hq[7] << 16));
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (k0 + e < O) dst[e] = (uint16_t)hq[e];
                    }
                }
            }
        }
        __syncthreads();
        {   // 64 rows (k) of up to 128 bytes (j): thread -> (k local, 32-byte piece) = two 16-byte stores
            const int kl = threadIdx.x >> 2, piece = threadIdx.x & 3;
            const int k = kt * 64 + kl;
            if (k < O) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int jl = piece * 32 + half * 16;
                    const int jo = jc + jl;
                    int8_t* dst = qw + (int64_t)k * I + jo;
                    if (out_vec && jo + 16 <= jc_end) {
                        *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(&tile[kl][jl]);
                    } else {
                        for (int e = 0; e < 16; ++e)
                            if (jo + e < jc_end) dst[e] = tile[kl][jl + e];
                    }
                }
            }
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_weight_quantize(const uint16_t* W, int I, int O, const float* fold, int qmax, int8_t* qw,
                                  float* w_scale, hipStream_t stream) {
    constexpr int RPW = 32;
    const int nkt = (O + 63) / 64;
    if (!grid_fits((int64_t)nkt * ((I + 127) / 128), 256)) return hipErrorInvalidValue;   // the largest of the grids
    const bool vec = (reinterpret_cast<uintptr_t>(W) % 16 == 0) && (O % 8 == 0);
    const bool qw_vec = (reinterpret_cast<uintptr_t>(qw) % 16 == 0) && (I % 16 == 0);
    const float qm = (float)qmax;
    // One block per 64 channels wherever that is not behind the shared-out form, whose clearing kernel and gap cost about 5 us.
    // A block reads a row piece at 62 GB/s, so the time of few blocks grows with their rows; beyond 8192 rows the shared-out
    // form is ahead until the weight is wide.  Block per 64 channels : shared out, us for the call: 1024 x 512 8.6 : 12.2, 4096 x
    // 512 15.3 : 16.2, 6144 x 2048 24.8 : 24.0, 8192 x 2048 30.8 : 29.0, 28672 x 2048 140 : 85; 4096 x 4096 22.9 : 25.5, 8192 x 4096
    // 39.0 : 42.5, 9216 x 4096 42.9 : 42.6, 28672 x 4096 172 : 114, 9216 x 5120 60.3 : 48.9, 28672 x 8192 247 : 224; 4096 x 11008
    // 41.9 : 46.5, 12288 x 11008 121 : 122, 28672 x 16384 434 : 442.
    if (I <= 4096 || (O >= 4096 && (I <= 8192 || O >= 10240))) {
        if (vec) weight_step_kernel<true><<<dim3((unsigned)nkt), dim3(1024), 0, stream>>>(W, I, O, fold, qm, w_scale);
        else weight_step_kernel<false><<<dim3((unsigned)nkt), dim3(1024), 0, stream>>>(W, I, O, fold, qm, w_scale);
    } else {
        uint32_t* bits = reinterpret_cast<uint32_t*>(w_scale);
        zero_u32_kernel<<<dim3((O + 255) / 256), dim3(256), 0, stream>>>(bits, O);
        const int ncc = (O + 511) / 512, nrc = (I + 4 * RPW - 1) / (4 * RPW);
        const dim3 grid((unsigned)(ncc * nrc));
        if (vec) weight_colmax_kernel<RPW, true><<<grid, dim3(256), 0, stream>>>(W, I, O, fold, qm, bits, ncc);
        else weight_colmax_kernel<RPW, false><<<grid, dim3(256), 0, stream>>>(W, I, O, fold, qm, bits, ncc);
    }
    const dim3 grid((unsigned)(nkt * ((I + 127) / 128)));       // (tiles of 256 rows measured 0 to 2 us slower)
    // This is the last read of W.  Up to 128 MiB the next call still finds part of it in the memory-side cache if the reads
    // are plain (4096 x 11008: 42.8 us against 44.6; 8192 x 8192, 128 MiB: 70.2 : 69.9); beyond, non-temporal reads leave
    // that cache to what the step pass brought in (4096 x 22016: 95.0 -> 87.7, 8192 x 28672 221 -> 213).
    // The same in the step pass, for the channels that the cache will have lost by then, gained 1 % at 8192 x 28672 and lost
    // 3 % at 28672 x 8192.
    if (vec && (int64_t)I * O * 2 > kCachedWeight)
        weight_tile_kernel<1, false, true, true><<<grid, dim3(256), 0, stream>>>(W, I, O, fold, 0, qm, qw, w_scale, nullptr, nkt, qw_vec, false, 1);
    else if (vec)
        weight_tile_kernel<1, false, true><<<grid, dim3(256), 0, stream>>>(W, I, O, fold, 0, qm, qw, w_scale, nullptr, nkt, qw_vec, false, 1);
    else
        weight_tile_kernel<1, false, false><<<grid, dim3(256), 0, stream>>>(W, I, O, fold, 0, qm, qw, w_scale, nullptr, nkt, qw_vec, false, 1);
    return hipGetLastError();
}

hipError_t launch_weight_quantize_grouped(const uint16_t* W, int I, int O, const float* fold, int group, int qmax,
                                          int8_t* qw, float* w_scale, uint16_t* wdq, hipStream_t stream) {
    const int nkt = (O + 63) / 64, ng = I / group;
    if (!grid_fits((int64_t)nkt * ng, 256)) return hipErrorInvalidValue;
    const bool in_vec = (reinterpret_cast<uintptr_t>(W) % 16 == 0) && (O % 8 == 0);
    const float qm = (float)qmax;
    // groups that a tile held in registers has whole; the others are read twice
    const bool held = group == 32 || group == 64 || group == 128 || group == 256;
    if (held) {
        const bool qw_vec = (reinterpret_cast<uintptr_t>(qw) % 16 == 0) && (I % 16 == 0);
        const bool dq_vec = O % 8 == 0 && reinterpret_cast<uintptr_t>(wdq) % 16 == 0;
        const int rows = group == 256 ? 256 : 128;
        const dim3 grid((unsigned)(nkt * ((I + rows - 1) / rows)));
        // One row of tiles after another leaves a channel's codes as single 128-byte lines, a row of the codes apart.  Where the
        // memory takes them rather than a cache, the tiles go in strips of at most 13 rows of tiles, of equal height but for the
        // last: the lines of a channel follow each other, and neighbouring channels (whose weights share DRAM pages) are still
        // only a few tiles apart.  By rows : in strips, us: with the dequantized weights 5120 x 20480 111 : 106, 8192 x 28672 267 :
        // 237, 28672 x 8192 253 : 233, 10240 x 16384 174 : 173, 4096 x 22016 101 : 97; codes alone 68 : 66, 179 : 135, 164 : 151,
        // 104 : 104, 68 : 60.  Over 23 shapes of 128 to 512 MiB heights of 9 to 14 are within 2 % of each other on average and
        // this limit is the one that loses nowhere (8192 x 8256, 129 MiB, 63.9 : 64.9 with the dequantized weights, 43.6 : 41.6
        // without); heights of 8, 16, 20 and 23 cost 6 to 9 % against rows on some shape, whole columns 33 %.  Weights that a
        // cache keeps lose: 4096 x 11008 46.1 : 46.4 and 29.2 : 31.6.
        const bool big = (int64_t)I * O * 2 > kCachedWeight;
        const int row_tiles = (I + rows - 1) / rows, n_strips = (row_tiles + 12) / 13;
        const int strip = rows == 128 && big ? (row_tiles + n_strips - 1) / n_strips : 1;
        auto run = [&](auto kernel) {
            kernel<<<grid, dim3(256), 0, stream>>>(W, I, O, fold, group, qm, qw, w_scale, wdq, nkt, qw_vec, dq_vec,
                                                   strip);
        };
        // W is read once; one that no cache keeps is read non-temporally (5120 x 20480: 112.3 -> 109.9 us)
        const bool once = in_vec && big;
        if (rows == 256) {
            if (once) run(&weight_tile_kernel<2, true, true, true>);
            else if (in_vec) run(&weight_tile_kernel<2, true, true>);
            else run(&weight_tile_kernel<2, true, false>);
        } else {
            if (once) run(&weight_tile_kernel<1, true, true, true>);
            else if (in_vec) run(&weight_tile_kernel<1, true, true>);
            else run(&weight_tile_kernel<1, true, false>);
        }
        return hipGetLastError();
    }
    const bool out_vec = (reinterpret_cast<uintptr_t>(qw) % 16 == 0) && (I % 16 == 0) && (group % 16 == 0);
    weight_group_kernel<<<dim3((unsigned)(nkt * ng)), dim3(256), 0, stream>>>(W, I, O, fold, group, qm, qw, w_scale, wdq, nkt,
                                                                             in_vec, out_vec);
    return hipGetLastError();
}

}  // namespace cq
