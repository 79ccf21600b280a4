// Quantization-kernel analysis (Definition 1; Table 1; the "Remove Kernel" experiment of the
// zero-shot accuracy figures): one pass over X that writes X with its kernel elements zeroed and
// counts the kernel size and the two indicators of the kernel-size analysis,
//   case II:  c_j >= t_i          and          B~_ij < B_ij  (zero bound of CrossQuant below per-token's).
// Only "is the code zero" is needed, and q = rne(fl32(x / fl32(a b))) is 0 exactly when the quotient
// is at most 1/2, so the sign of one fma, |x| (1/b) - a/2, decides; a wave in which any lane has
// the two sides within 2^-20 of each other (the approximation is within 2^-22) takes the correctly
// rounded division for its row piece instead.  The three counts are kept per lane (one compare and
// one add of its carry each) and summed once per wave at the end.
// Bound by the memory (4096 x 5120: 84 MB in 15.9 us = 5.3 TB/s, factors and counters included): with the counts left to the compiler, which
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

// The three counts' accumulators for each stream slot, zero between launches (launch_sum): nothing has to be cleared before.
__device__ unsigned long long g_analysis_state[kStateSlots][3][kCountWords];

// Block: 8 waves share 512 columns; each wave takes nb batches of 4 consecutive rows, last batch first, two register sets
// alternating as in the quantize kernel (rows as raw buffers with BUF, the layout every real activation has; unaligned
// loads and stores otherwise; rows past the last one are read as copies of it and not worked on).
// The block forms the factors of its rows and columns itself, while its first rows are on their way; the blocks of column
// chunk 0 / row chunk 0 write them to a_out / b_out if given.  (A kernel in front of this one
// formed them and cleared the counters, 2.5 us of a call: 4096 x 4096 16.2 -> 12.4 us, 4096 x 5120 18.4 -> 16.0, 512 x 4096 8.6 -> 6.9,
// 64 x 1024 7.2 -> 5.9.  Part of it is the counts, which were 1536 adds to one line of the caller.)
template <bool BUF>
__global__ void __launch_bounds__(kWaves * kLanes)
analysis_kernel(const uint16_t* __restrict__ X, int T, int I, int64_t ldx, const float* __restrict__ t_vec,
                const float* __restrict__ c_vec, double alpha, int qmax_i, float* __restrict__ a_out,
                float* __restrict__ b_out, uint16_t* __restrict__ xrk, unsigned long long* __restrict__ counters, int slot,
                int n_col_chunks, int nb) {
    __shared__ uint32_t lds_cnt[kWaves][3];
    __shared__ float lds_a[kWaves * kLanes], lds_t[kWaves * kLanes];
    __shared__ float lds_b[kColsPerWave], lds_c[kColsPerWave];
    const float qmax = (float)qmax_i;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int col_chunk = blockIdx.x % n_col_chunks;
    const int row_chunk = blockIdx.x / n_col_chunks;
    const int col0 = col_chunk * kColsPerWave, j0 = col0 + lane * 8;
    const int cols_here = min(kColsPerWave, I - col0);      // a multiple of 8 with BUF
    const int rows_per_wave = nb * kU, rows_per_block = kWaves * rows_per_wave;
    const int block_row0 = row_chunk * rows_per_block, row0 = block_row0 + wave * rows_per_wave;

    auto load_batch = [&](uint4 (&dst)[kU], int bi) {
        if (bi >= nb) return;                                // scalar condition
        const int rbase = row0 + (nb - 1 - bi) * kU;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint16_t* row = X + (int64_t)min(rbase + u, T - 1) * ldx;
            dst[u] = BUF ? buffer_load16(row_buffer(row + col0, cols_here * 2), lane * 16) : load8<false>(row, j0, I);
        }
    };
    // the maxima that become factors before the rows, as in the quantize kernel: 2 kU requests follow the two
    const int k = (int)threadIdx.x;
    float c_in, t_in;
    if (!BUF) {
        c_in = c_vec[min(col0 + k, I - 1)];
        t_in = t_vec[min(block_row0 + k, T - 1)];
    } else {
        const float* cp = c_vec + min(col0 + k, I - 1);
        const float* tp = t_vec + min(block_row0 + k, T - 1);
        asm volatile("global_load_dword %0, %2, off\n\tglobal_load_dword %1, %3, off"
                     : "=&v"(c_in), "=&v"(t_in)
                     : "v"(cp), "v"(tp)
                     : "memory");
    }
    uint4 va[kU], vb[kU];
    load_batch(va, 0);
    if (nb >= 2) load_batch(vb, 1);
    else if (BUF) load_batch(vb, 0);                        // a wave with one batch requests it twice: always 2 kU requests
    static_assert(kU == 4, "the wait below counts the row requests of two batches");
    if (BUF) asm volatile("s_waitcnt vmcnt(8)" : "+v"(c_in), "+v"(t_in)::"memory");

    // Columns past the end: x reads as 0 there and their step is infinite, so the code is 0 (not counted as non-zero) and
    // the step (NaN for a_i = 0) is never below the per-token step; c = -1 is never >= t_i.
    {
        const int j = col0 + k, r = block_row0 + k;
        float bj = __builtin_inff();
        if (j < I) {
            bj = col_factor(c_in, alpha);
            if (row_chunk == 0 && b_out) b_out[j] = bj;
        }
        lds_b[k] = bj;
        lds_c[k] = j < I ? c_in : -1.0f;
        float ar = 0.0f;
        if (k < rows_per_block && r < T) {
            ar = row_factor(t_in, alpha, qmax_i);
            if (col_chunk == 0 && a_out) a_out[r] = ar;
        }
        lds_a[k] = ar;
        lds_t[k] = r < T ? t_in : 0.0f;
    }
    __syncthreads();
    float b[8], rb[8], c[8];
    bool odd = false;
    __builtin_memcpy(c, lds_c + lane * 8, 32);
    __builtin_memcpy(b, lds_b + lane * 8, 32);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        rb[e] = safe_rcp(b[e]);
        odd |= tiny_factor(b[e]);
    }
    // per row: a_i, t_i and the per-token step fl32(t_i / q_max), one row per lane
    const int row_of_lane = wave * rows_per_wave + (lane < rows_per_wave ? lane : 0);
    const float a_lane = lds_a[row_of_lane], t_lane = lds_t[row_of_lane];
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
    if (threadIdx.x < 3) {                                  // a thread per count
        unsigned long long s = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += lds_cnt[w][threadIdx.x];
        if (slot < 0) {                                     // no state: the caller's counters, cleared before
            if (s) atomicAdd(&counters[threadIdx.x], s);
        } else if (launch_sum(g_analysis_state[slot][threadIdx.x], s, gridDim.x > 4 * kCountGroups)) {
            counters[threadIdx.x] = s;                      // every other block has added
        }
    }
}

}  // namespace

// a, b (both or neither): receive the scale factors.
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
    // (a captured call clears the caller's counters and adds to them: graphs with counters of their own are independent)
    const int slot = uncaptured_stream_slot(stream, kAnalysisTable);
    if (slot < 0) zero_counters_kernel<<<dim3(1), dim3(64), 0, stream>>>(counters);
    const auto kernel = buf ? &analysis_kernel<true> : &analysis_kernel<false>;
    kernel<<<grid, block, 0, stream>>>(X, T, I, ldx, t, c, al, qmax, a, b, xrk, counters, slot, ncc, nb);
    return hipGetLastError();
}

}  // namespace cq
