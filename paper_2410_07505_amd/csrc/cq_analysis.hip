// Quantization-kernel analysis (Definition 1; Table 1; the "Remove Kernel" experiment of the
// zero-shot accuracy figures): one pass over X that writes X with its kernel elements zeroed and
// counts the kernel size and the two indicators of the kernel-size analysis,
//   case II:  c_j >= t_i          and          B~_ij < B_ij  (zero bound of CrossQuant below per-token's).
// Only "is the code zero" is needed, and q = rne(fl32(x / fl32(a b))) is 0 exactly when the quotient
// is at most 1/2, so the sign of one fma, |x| (1/b) - a/2, decides; a wave in which any lane has
// the two sides within 2^-20 of each other (the approximation is within 2^-22) takes the correctly
// rounded division for its row piece instead.  The three counts are kept per lane (one compare and
// one add of its carry each) and summed once per wave at the end.
// Bound by the memory now (4096 x 5120: 84 MB in 15.7 us = 5.35 TB/s): with the counts left to the compiler, which
// counted the bits of compare masks, one register set and plain bounds handling the kernel took 26 us there, and
// 32.4 against 21.8 us on 4096 x 8192.
#include "cq_device.h"

namespace cq {
namespace {

constexpr int kWaves = 8;
constexpr int kU = 4;

__global__ void zero_counters_kernel(unsigned long long* __restrict__ counters) {
    if (threadIdx.x < 3) counters[threadIdx.x] = 0ull;
}

// Block: 8 waves share 512 columns; each wave takes nb batches of 4 consecutive rows, last batch first, two register sets
// alternating as in the quantize kernel (rows as raw buffers with BUF, the layout every real activation has; unaligned
// loads and stores otherwise; rows past the last one are read as copies of it and not worked on).
// OWN_FACTORS: a_vec / b_vec are not given; the block forms the factors of its rows and columns itself
// (as the quantize kernel does) and keeps them in LDS.
template <bool BUF, bool OWN_FACTORS>
__global__ void __launch_bounds__(kWaves * kLanes)
analysis_kernel(const uint16_t* __restrict__ X, int T, int I, int64_t ldx, const float* __restrict__ t_vec,
                const float* __restrict__ c_vec, const float* __restrict__ a_vec, const float* __restrict__ b_vec,
                double alpha, int qmax_i, uint16_t* __restrict__ xrk, unsigned long long* __restrict__ counters,
                int n_col_chunks, int nb) {
    __shared__ uint32_t lds_cnt[kWaves][3];
    __shared__ float lds_a[OWN_FACTORS ? kWaves * kLanes : 1];
    __shared__ float lds_b[OWN_FACTORS ? kColsPerWave : 1];
    const float qmax = (float)qmax_i;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int col_chunk = blockIdx.x % n_col_chunks;
    const int row_chunk = blockIdx.x / n_col_chunks;
    const int col0 = col_chunk * kColsPerWave, j0 = col0 + lane * 8;
    const int cols_here = min(kColsPerWave, I - col0);      // a multiple of 8 with BUF
    const int rows_per_wave = nb * kU;
    const int row0 = row_chunk * (kWaves * rows_per_wave) + wave * rows_per_wave;

    auto load_batch = [&](uint4 (&dst)[kU], int bi) {
        if (bi >= nb) return;                                // scalar condition
        const int rbase = row0 + (nb - 1 - bi) * kU;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint16_t* row = X + (int64_t)min(rbase + u, T - 1) * ldx;
            dst[u] = BUF ? buffer_load16(row_buffer(row + col0, cols_here * 2), lane * 16) : load8<false>(row, j0, I);
        }
    };
    uint4 va[kU], vb[kU];
    load_batch(va, 0);
    load_batch(vb, 1);

    if (OWN_FACTORS) {
        block_scale_factors(t_vec, c_vec, alpha, qmax_i, T, I, col0, row_chunk * (kWaves * rows_per_wave),
                            kWaves * rows_per_wave, lds_a, lds_b, nullptr, nullptr);
        __syncthreads();
    }

    // Columns past the end: x reads as 0 there and their step is infinite, so the code is 0 (not counted as non-zero) and
    // the step (NaN for a_i = 0) is never below the per-token step; c = -1 is never >= t_i.
    float b[8], rb[8], c[8];
    bool odd = false;
    if (BUF) {                                              // all eight exist or none: two loads each, none past the end
        const int j = min(j0, I - 8);
        __builtin_memcpy(c, c_vec + j, 32);
        if (OWN_FACTORS) __builtin_memcpy(b, lds_b + lane * 8, 32);
        else __builtin_memcpy(b, b_vec + j, 32);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = min(j0 + e, I - 1);
            c[e] = c_vec[j];
            b[e] = OWN_FACTORS ? lds_b[lane * 8 + e] : b_vec[j];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (j0 + e >= I) {
            b[e] = __builtin_inff();
            c[e] = -1.0f;
        }
        rb[e] = safe_rcp(b[e]);
        odd |= tiny_factor(b[e]);
    }
    // per row: a_i, t_i and the per-token step fl32(t_i / q_max), one row per lane
    const bool has_row = lane < rows_per_wave && row0 + lane < T;
    const float a_lane = has_row ? (OWN_FACTORS ? lds_a[wave * rows_per_wave + lane] : a_vec[row0 + lane]) : 0.0f;
    const float t_lane = has_row ? t_vec[row0 + lane] : 0.0f;
    const float pt_lane = (float)((double)t_lane / (double)qmax);

    uint32_t nz_lane = 0, ge_lane = 0, sm_lane = 0;         // this lane's counts: codes != 0, c_j >= t_i, B~ < B
    int rows_done = 0;
    auto work = [&](const uint4 (&v)[kU], int bi) {
        const int rbase = row0 + (nb - 1 - bi) * kU;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = rbase + u;
            if (r >= T) break;                              // scalar
            ++rows_done;
            const int ri = (nb - 1 - bi) * kU + u;
            const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a_lane), ri));
            const float ti = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, t_lane), ri));
            const float pt = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pt_lane), ri));
            const float ha = 0.5f * a, tol = ha * kTieTol;
            const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            _Float16 h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = __builtin_bit_cast(_Float16, (unsigned short)(w[e >> 1] >> (16 * (e & 1))));
            // The X-independent counts.  Compares and adds of their carry are written out: from "n += x ? 1 : 0" the
            // compiler builds a bit mask of the eight compares and counts its bits, three times the work.
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float D = a * b[e];                                // 0.5 * D < 0.5 * pt, exactly
                asm("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(ge_lane) : "v"(ti), "v"(c[e]) : "vcc");
                asm("v_cmp_gt_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(sm_lane) : "v"(pt), "v"(D) : "vcc");
            }
            uint16_t* dst = xrk + (int64_t)r * I + col0;
            auto emit = [&](const uint32_t (&kept)[8]) {    // kept[e]: element e's word, or 0 where its code is 0
                if (!xrk) return;
                u32x4 o;
#pragma unroll
                for (int p = 0; p < 4; ++p) o[p] = (kept[2 * p] & 0xFFFFu) | (kept[2 * p + 1] & 0xFFFF0000u);
                if (BUF) __builtin_amdgcn_raw_buffer_store_b128(o, row_buffer(dst, cols_here * 2), lane * 16, 0, kWriteThrough);
                else store_piece<16, uint16_t>(o, dst + lane * 8, 2 * max(0, min(8, cols_here - lane * 8)));
            };
            uint32_t kept[8], nz = 0u;
            float nearest = __builtin_inff();               // min over the 8 elements of | |x|/b - a/2 |
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = __builtin_fmaf(__builtin_fabsf((float)h[e]), rb[e], -ha);
                asm("v_cmp_lt_f32 vcc, 0, %3\n\tv_cndmask_b32 %1, 0, %2, vcc\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc"
                    : "+v"(nz), "=&v"(kept[e])
                    : "v"(w[e >> 1]), "v"(d)
                    : "vcc");
                nearest = __builtin_fminf(nearest, __builtin_fabsf(d));
            }
            // a == 0: D = 0 and every code of the row is 0 by definition (left to the exact path, which packs and stores
            // for itself: values from either path would need register copies where the paths join)
            if (__builtin_expect(__any(nearest <= tol || odd || tiny_factor(a) || a == 0.0f), 0)) {
                nz = 0u;
                uint32_t kx[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float D = a * b[e];
                    float q = (D == 0.0f) ? 0.0f : __builtin_rintf((float)h[e] / D);
                    q = __builtin_amdgcn_fmed3f(q, -qmax, qmax);
                    const bool nonzero = __builtin_fabsf(q) > 0.0f && j0 + e < I;
                    nz += nonzero ? 1u : 0u;
                    kx[e] = nonzero ? w[e >> 1] : 0u;
                }
                emit(kx);
            } else {
                emit(kept);
            }
            nz_lane += nz;
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int bi = 0; bi < nb; bi += 2) {
        work(va, bi);
        load_batch(va, bi + 2);
        if (bi + 1 < nb) {
            work(vb, bi + 1);
            load_batch(vb, bi + 3);
        }
    }

    // wave totals
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        nz_lane += (uint32_t)__shfl_xor((int)nz_lane, off, kLanes);
        ge_lane += (uint32_t)__shfl_xor((int)ge_lane, off, kLanes);
        sm_lane += (uint32_t)__shfl_xor((int)sm_lane, off, kLanes);
    }
    if (lane == 0) {
        lds_cnt[wave][0] = (uint32_t)(rows_done * cols_here) - nz_lane;
        lds_cnt[wave][1] = ge_lane;
        lds_cnt[wave][2] = sm_lane;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t s = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += lds_cnt[w][threadIdx.x];
        if (s) atomicAdd(&counters[threadIdx.x], (unsigned long long)s);
    }
}

}  // namespace

// a, b null: the kernel forms the factors itself (counters cleared by a kernel of their own first);
// otherwise a, b are work vectors that a scale-finalize kernel fills first (it also clears the counters).
hipError_t launch_kernel_analysis(const uint16_t* X, int T, int I, int64_t ldx, const float* t, const float* c,
                                  float* a, float* b, float alpha, int qmax, uint16_t* xrk,
                                  unsigned long long* counters, hipStream_t stream) {
    const int ncc = (I + 511) / 512;
    const int nb = quantize_batches_per_wave(ncc, T);                      // rows per block = 32 * nb
    const int nrc = (T + 32 * nb - 1) / (32 * nb);
    if (!grid_fits((int64_t)ncc * nrc, kWaves * kLanes)) return hipErrorInvalidValue;     // before anything is enqueued
    const dim3 grid((unsigned)(ncc * nrc)), block(kWaves * kLanes);
    const bool buf = (reinterpret_cast<uintptr_t>(X) % 16 == 0) && (ldx % 8 == 0) && (I % 8 == 0) &&
                     (reinterpret_cast<uintptr_t>(xrk) % 16 == 0);
    const double al = (double)alpha;
    if (a && b) {
        const hipError_t e = launch_scale_finalize(t, c, T, I, alpha, qmax, a, b, counters, 3, stream);
        if (e != hipSuccess) return e;
        const auto kernel = buf ? &analysis_kernel<true, false> : &analysis_kernel<false, false>;
        kernel<<<grid, block, 0, stream>>>(X, T, I, ldx, t, c, a, b, al, qmax, xrk, counters, ncc, nb);
    } else {
        zero_counters_kernel<<<dim3(1), dim3(64), 0, stream>>>(counters);
        const auto kernel = buf ? &analysis_kernel<true, true> : &analysis_kernel<false, true>;
        kernel<<<grid, block, 0, stream>>>(X, T, I, ldx, t, c, nullptr, nullptr, al, qmax, xrk, counters, ncc, nb);
    }
    return hipGetLastError();
}

}  // namespace cq
