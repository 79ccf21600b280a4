// Device-side building blocks shared by the streaming kernels (absmax, quantize, fused).
#pragma once
#include "cq_kernels.h"

namespace cq {

constexpr int kLanes = 64;
constexpr int kColsPerWave = kLanes * 8;          // a wave owns 512 columns: 8 halfs (16 bytes) per lane
constexpr float kMagic = 12582912.0f;             // 1.5 * 2^23: adding it rounds to nearest-even integer
constexpr float kTieTol = 1.9073486328125e-06f;   // 2^-19

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// packed maximum of two pairs of 16-bit patterns (|x| of binary16 orders like an unsigned integer)
__device__ __forceinline__ uint32_t pkmax(uint32_t a, uint32_t b) {
    us2 r = __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b));
    return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ uint32_t half_bits_to_float_bits(uint32_t h) { return __float_as_uint(h2f(h)); }

__device__ __forceinline__ uint32_t shx(uint32_t v, int off) { return (uint32_t)__shfl_xor((int)v, off, kLanes); }

// 8 halfs starting at column j of a row; columns >= I read as zero, and nothing outside the row is read.
// VEC: I % 8 == 0 and the row starts on 16 bytes.  Otherwise one 16-byte load without alignment; the lane that holds the
// row's last columns loads the 8 that end the row and shifts (rows shorter than that: element by element).
template <bool VEC>
__device__ __forceinline__ uint4 load8(const uint16_t* __restrict__ row, int j, int I) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (VEC) {
        if (j + 8 <= I) v = *reinterpret_cast<const uint4*>(row + j);
    } else if (I >= 8) {                                     // uniform
        const int at = min(j, I - 8), sh = j - at;           // columns to shift out: 0 but for the row's end
        __builtin_memcpy(&v, row + at, 16);
        if (sh > 0) {
            unsigned __int128 w = __builtin_bit_cast(unsigned __int128, v);
            w = sh >= 8 ? 0 : w >> (16 * (sh & 7));
            v = __builtin_bit_cast(uint4, w);
        }
    } else {                                                 // unconditional, so that the loads of several rows overlap
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = row[min(j + e, I - 1)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (j + e >= I) h[e] = 0u;
        v = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    }
    return v;
}

// Per-lane maximum |x| of a 16-byte piece (a 16-bit pattern), also folded into four packed
// running column maxima.
__device__ __forceinline__ uint32_t absmax8(const uint4& v, uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3) {
    const uint32_t x0 = v.x & 0x7FFF7FFFu, x1 = v.y & 0x7FFF7FFFu;
    const uint32_t x2 = v.z & 0x7FFF7FFFu, x3 = v.w & 0x7FFF7FFFu;
    c0 = pkmax(c0, x0);
    c1 = pkmax(c1, x1);
    c2 = pkmax(c2, x2);
    c3 = pkmax(c3, x3);
    const uint32_t m = pkmax(pkmax(x0, x1), pkmax(x2, x3));
    return max(m & 0xFFFFu, m >> 16);
}

// rm[g] = this lane's maximum over its 8 columns of row g (a 16-bit pattern).  Returns, in lane
// l with (l & 7) == 0, the maximum over all 64 lanes of row (l >> 3).  A transposed butterfly:
// every exchange step halves the number of rows a lane still carries (7 shuffles for 8 rows).
__device__ __forceinline__ uint32_t rows8_reduce(const uint32_t* rm, int lane) {
    const uint32_t p0 = rm[0] | (rm[1] << 16), p1 = rm[2] | (rm[3] << 16);
    const uint32_t p2 = rm[4] | (rm[5] << 16), p3 = rm[6] | (rm[7] << 16);
    const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
    // lanes with bit 5 clear keep rows 0-3 and hand rows 4-7 to their partner, and vice versa
    const uint32_t q0 = pkmax(b5 ? p2 : p0, shx(b5 ? p0 : p2, 32));
    const uint32_t q1 = pkmax(b5 ? p3 : p1, shx(b5 ? p1 : p3, 32));
    const uint32_t r = pkmax(b4 ? q1 : q0, shx(b4 ? q0 : q1, 16));
    const uint32_t keep = b3 ? (r >> 16) : (r & 0xFFFFu);
    const uint32_t send = b3 ? (r & 0xFFFFu) : (r >> 16);
    uint32_t m = max(keep, shx(send, 8));
    m = max(m, shx(m, 4));
    m = max(m, shx(m, 2));
    m = max(m, shx(m, 1));
    return m;
}

// ---- scale factors of the CrossQuant step: x^y (divided by q_max for a row) in binary64, rounded once to binary32.
// The library's pow is good to an ulp of binary64 and takes as long as the rest of a small call (a 64 x 256 quantize call
// is two of them one after the other); a binary32 result needs far less.  x^y = 2^(y (k + log2 m)), x = 2^k m with m in
// [sqrt(1/2), sqrt(2)): log2 m is the atanh series in s = (m - 1) / (m + 1), |s| < 0.172, to s^19, and 2^f, |f| <= 1/2, its
// Taylor series to f^12; their truncation is below 2^-51 and the binary64 roundings (of y log2 x above all, |log2 x| < 128)
// leave less than 2^-46 relative (2^-46.5 measured over all binary32 x, 2^-48.7 over binary16 ones).  Where the value moved
// by 2^-42 either way rounds to one binary32 number, every more accurate value does too, pow's included; otherwise (once
// in 2^17) and for x that is zero, subnormal or not finite pow decides.  The result is pow's, bit for bit.
// Exponents 0 and 1 (per-column and per-token steps) are written out: exact in any correct pow.
__device__ __forceinline__ double short_pow(float x, double y) {
    const uint32_t u = __float_as_uint(x);
    double m = (double)__uint_as_float((u & 0x7FFFFFu) | 0x3F800000u);
    int k = (int)(u >> 23) - 127;
    if (m > 1.4142135623730951) {
        m *= 0.5;
        ++k;
    }
    const double den = m + 1.0;
    double r = __builtin_amdgcn_rcp(den);                   // two Newton steps: full precision
    r = __builtin_fma(__builtin_fma(-den, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-den, r, 1.0), r, r);
    const double s = (m - 1.0) * r, z = s * s;
    // 2 / ((2 n + 1) ln 2)
    double p = 0.15186263588304877;
    p = __builtin_fma(p, z, 0.16972882833987804);
    p = __builtin_fma(p, z, 0.19235933878519512);
    p = __builtin_fma(p, z, 0.2219530832136867);
    p = __builtin_fma(p, z, 0.2623081892525388);
    p = __builtin_fma(p, z, 0.3205988979753252);
    p = __builtin_fma(p, z, 0.41219858311113244);
    p = __builtin_fma(p, z, 0.5770780163555853);
    p = __builtin_fma(p, z, 0.9617966939259757);
    p = __builtin_fma(p, z, 2.8853900817779268);
    const double t = y * __builtin_fma(s, p, (double)k);
    const double n = __builtin_rint(t), f = t - n;
    // ln2^n / n!
    double e = 2.5678435993488196e-11;
    e = __builtin_fma(e, f, 4.44553827187081e-10);
    e = __builtin_fma(e, f, 7.054911620801121e-09);
    e = __builtin_fma(e, f, 1.0178086009239696e-07);
    e = __builtin_fma(e, f, 1.3215486790144305e-06);
    e = __builtin_fma(e, f, 1.5252733804059838e-05);
    e = __builtin_fma(e, f, 0.00015403530393381606);
    e = __builtin_fma(e, f, 0.0013333558146428441);
    e = __builtin_fma(e, f, 0.009618129107628477);
    e = __builtin_fma(e, f, 0.055504108664821576);
    e = __builtin_fma(e, f, 0.2402265069591007);
    e = __builtin_fma(e, f, 0.6931471805599453);
    e = __builtin_fma(e, f, 1.0);
    return __builtin_ldexp(e, (int)n);
}
// fl32(x^y / q); inv_q = 1 / q in binary64
__device__ __forceinline__ float power_over(float x, double y, double q, double inv_q) {
    if (y == 0.0) return (float)(1.0 / q);
    if (y == 1.0) return (float)((double)x / q);
    if (x >= 1.1754943508222875e-38f && x <= 3.4028234663852886e+38f) {
        const double v = short_pow(x, y) * inv_q;
        constexpr double kMargin = 2.2737367544323206e-13;   // 2^-42
        const float lo = (float)__builtin_fma(v, -kMargin, v), hi = (float)__builtin_fma(v, kMargin, v);
        if (lo == hi) return lo;
    }
    return (float)(pow((double)x, y) / q);
}
__device__ __forceinline__ float row_factor(float t, double al, int qmax) {
    return power_over(t, al, (double)qmax, qmax == 127 ? 1.0 / 127.0 : 1.0 / 7.0);
}
__device__ __forceinline__ float col_factor(float c, double al) { return power_over(c, 1.0 - al, 1.0, 1.0); }

__device__ __forceinline__ float safe_rcp(float v) { return (v == 0.0f) ? 0.0f : __builtin_amdgcn_rcpf(v); }

__device__ __forceinline__ float half_lo(uint32_t w) { return h2f(w & 0xFFFFu); }
__device__ __forceinline__ float half_hi(uint32_t w) { return h2f(w >> 16); }

// Output stores of the streaming kernels: written through to memory at device scope (sc1) instead
// of being left dirty in the caches.  Measured on the 4096 x 8192 layer against plain and
// non-temporal stores: the quantize kernel itself is 3 us (8 %) faster, and the matrix kernel that
// reads the codes next 5 us.  The compiler offers no way to ask for this policy, hence the
// assembly; it cannot see a store in it, so the two wait states the hardware needs before the data
// registers of a wide store may be overwritten are added by hand.
__device__ __forceinline__ void store_through(uint32_t v, uint32_t* dst) {
    asm volatile("global_store_dword %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through(u32x2 v, u32x2* dst) {
    asm volatile("global_store_dwordx2 %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through(u32x4 v, u32x4* dst) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
}

// bytes 0 of four words -> one word
__device__ __forceinline__ uint32_t pack_bytes(uint32_t u0, uint32_t u1, uint32_t u2, uint32_t u3) {
    const uint32_t p01 = __builtin_amdgcn_perm(u1, u0, 0x0c0c0400u);
    const uint32_t p23 = __builtin_amdgcn_perm(u3, u2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(p23, p01, 0x05040100u);
}

// ---- one lane's 8 elements of one row.  On return q[e] = q_e and m[e] = kMagic + q_e with
// q_e = clamp(rne(fl32(x_e / fl32(a * b[e]))), +-qmax), identical to dividing every element.
// The quotient is first approximated as x * (1/a) * (1/b) (ra, rb: reciprocals within 1 ulp, 0
// where the factor is 0), which lies within 2^-21 relative of the correctly rounded quotient
// (two reciprocals at 2^-23, the rounding of their product and of a * b at 2^-24, and the
// quotient's own; 2^-20.7 even if each reciprocal were a further half ulp off).  The product is
// never formed on its own: fma(x, k, 1.5 * 2^23) rounds it straight to the nearest-even integer
// (the sum's ulp is 1), q = that - 1.5 * 2^23 is the code, and a second fma, x * k - q, gives the
// distance from it.  The integer can differ from the exact one only if the approximation lies
// within the bound of a rounding tie k + 1/2: lanes test |x k - q| + (|q| + 1) * 2^-19 >= 1/2
// (a 3x to 4x margin) and also |q| > qmax (a code that needs clamping: only with caller-supplied
// maxima below the data's), and a wave in which any lane trips recomputes its eight elements with
// the exact division and the clamp.  Both fmas read the binary16 value directly (v_fma_mix_f32).
// The bound needs ra * rb and a * b to be normal numbers: `tiny` (any factor of this lane's piece
// below kTinyFactor, possible only with caller-supplied maxima far below anything binary16 data
// can produce) sends the piece to the exact division as well.
constexpr float kTinyFactor = 8.673617379884035e-19f;   // 2^-60: both products stay within 2^+-120

__device__ __forceinline__ bool tiny_factor(float f) { return f != 0.0f && f < kTinyFactor; }

// max(|a|, |b|, |c|), NaN where one of them is (written out: the compiler makes two-operand steps of some of a chain of these)
__device__ __forceinline__ float ordered_max3(float a, float b, float c) {
    float r;
    asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The fast part: m, q from the reciprocals; returns whether this wave's row piece has to be redone exactly
// (wave-uniform).  An element that is no number (outside the contract) does not ask for that, its code is the low bits of m, 0;
// ORDERED: it does too.
template <bool ORDERED = false>
__device__ __forceinline__ bool quantize8_fast(const uint4& v, float ra, const float (&rb)[8], float qmax,
                                               float (&m)[8], float (&q)[8], bool tiny) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    _Float16 h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = __builtin_bit_cast(_Float16, (unsigned short)(w[e >> 1] >> (16 * (e & 1))));
    float score = 0.0f;                                 // max over the 8 elements of |x k - q| + |q| * tol
    float big = 0.0f;                                   // max over the 8 elements of |q|
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float k = ra * rb[e];
        m[e] = __builtin_fmaf((float)h[e], k, kMagic);
        q[e] = m[e] - kMagic;
        const float f = __builtin_fmaf((float)h[e], k, -q[e]);
        score = __builtin_fmaxf(score, __builtin_fmaf(__builtin_fabsf(q[e]), kTieTol, __builtin_fabsf(f)));
        if (!ORDERED) big = __builtin_fmaxf(big, __builtin_fabsf(q[e]));
        else if (e & 1) big = ordered_max3(e == 1 ? q[1] : big, q[e - 1], q[e]);
    }
    return __any(score >= 0.5f - kTieTol || !(big <= qmax) || tiny);
}
// The exact part: the correctly rounded division and the clamp, for all 8 elements.
__device__ __forceinline__ void quantize8_exact(const uint4& v, float a, const float (&b)[8], float qmax,
                                                float (&m)[8], float (&q)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float x = (float)__builtin_bit_cast(_Float16, (unsigned short)(w[e >> 1] >> (16 * (e & 1))));
        const float D = a * b[e];
        float rt = (D == 0.0f) ? 0.0f : x / D;
        rt = __builtin_amdgcn_fmed3f(rt, -qmax, qmax);
        m[e] = rt + kMagic;
        q[e] = m[e] - kMagic;
    }
}
__device__ __forceinline__ void quantize8(const uint4& v, float a, float ra, const float (&b)[8],
                                          const float (&rb)[8], float qmax, float (&m)[8], float (&q)[8],
                                          bool tiny) {
    if (quantize8_fast(v, ra, rb, qmax, m, q, tiny)) quantize8_exact(v, a, b, qmax, m, q);   // rare
}

// Count-only form of quantize8: every lane returns how many of its own 8 elements have a non-zero code, and
// the kernel adds the lanes up once at its end.
// q = rne(fl32(x / fl32(a b))) is 0 exactly when the quotient is at most 1/2 (a tie rounds to the even
// 0), so the sign of d = fma(|x|, 1/b, -a/2) decides, unless the two sides are within 2^-20 of each
// other: |x| / b differs from (x / fl32(a b)) a by at most 2^-22 relative (reciprocal, rounding of
// a b, the quotient's own rounding; the fma's single rounding never changes its sign).  A wave in
// which any lane comes that close, or has a factor so small that products leave the normal range,
// recounts the row piece with the exact division.  ha = a / 2 (exact), tol = ha * 2^-19.
// A compare and an add-with-carry per element and one running minimum of |d| for the closeness test, all vector
// instructions: handing every compare mask to the scalar unit (population count, add, or), which the four SIMDs of a
// CU share, was 1.6 scalar instructions per vector instruction.
__device__ __forceinline__ uint32_t count_row8_lane(const uint4& v, float a, float ha, float tol, const float (&b)[8],
                                                    const float (&rb)[8], float qmax, bool tiny) {
    float x[8];
    x[0] = half_lo(v.x); x[1] = half_hi(v.x);
    x[2] = half_lo(v.y); x[3] = half_hi(v.y);
    x[4] = half_lo(v.z); x[5] = half_hi(v.z);
    x[6] = half_lo(v.w); x[7] = half_hi(v.w);
    uint32_t nz = 0u;
    float nearest = __builtin_inff();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float d = __builtin_fmaf(__builtin_fabsf(x[e]), rb[e], -ha);
        // nz += d > 0, as a compare and an add of its carry (written out: from "nz += d > 0 ? 1 : 0" the compiler
        // builds a bit mask of the eight compares with shifts and ors and counts its bits, three times the work)
        asm("v_cmp_lt_f32 vcc, 0, %1\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(nz) : "v"(d) : "vcc");
        nearest = __builtin_fminf(nearest, __builtin_fabsf(d));
    }
    if (__any(nearest <= tol || tiny)) {                // rare: exact division for this wave's row piece
        nz = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float D = a * b[e];
            float rt = (D == 0.0f) ? 0.0f : x[e] / D;
            rt = __builtin_amdgcn_fmed3f(rt, -qmax, qmax);
            nz += (rt + kMagic != kMagic) ? 1u : 0u;
        }
    }
    return nz;
}

// Number of a lane's non-zero codes among m[0..8); the kernel adds the lanes up once at its end: a compare and an add of
// its carry per element and nothing for the scalar unit, which the four SIMDs of a CU share.
__device__ __forceinline__ uint32_t count_nonzero8_lane(const float (&m)[8]) {
    uint32_t nz = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        asm("v_cmp_neq_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(nz) : "v"(m[e]), "v"(kMagic) : "vcc");
    return nz;
}

// number of non-zero codes among m[0..8) (as a float: exact far below 2^24)
__device__ __forceinline__ float count_nonzero8(const float (&m)[8]) {
    float nz = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) nz += __builtin_fminf(__builtin_fabsf(m[e] - kMagic), 1.0f);
    return nz;
}

// ---- A count summed over the blocks of a launch without anything cleared in front of it.  A word of library-owned memory, zero
// between launches, holds the running sum in bits 0..40 (at most 2^40 elements) and the number of adds in bits 41..63 (a launch
// of 512-thread blocks has fewer than 2^23 of them).  The add that brings the second field to `adds` knows the total and
// clears the word again.
constexpr int kTicketShift = 41;
__device__ __forceinline__ bool ticketed_add(unsigned long long* word, unsigned long long& sum, unsigned adds) {
    const unsigned long long add = (1ull << kTicketShift) | sum;
    const unsigned long long old = __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((unsigned)(old >> kTicketShift) != adds - 1u) return false;
    sum = (old + add) & ((1ull << kTicketShift) - 1ull);
    __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}
// Adds to one word queue up (8.4 ns each: 512 blocks that end together wait 4.3 us), so the blocks of a larger launch add in
// kCountGroups groups first, each on a 128-byte line of its own, and the groups' last blocks to the launch's word.
constexpr int kCountGroups = 16, kCountLine = 16;            // words a line has
constexpr int kCountWords = (1 + kCountGroups) * kCountLine; // of a stream slot
__device__ __forceinline__ bool launch_sum(unsigned long long* state, unsigned long long& sum, bool groups) {
    const unsigned g = blockIdx.x % kCountGroups;
    if (!ticketed_add(groups ? state + (1 + g) * kCountLine : state, sum,
                      groups ? (gridDim.x - g + kCountGroups - 1) / kCountGroups : gridDim.x)) return false;
    return !groups || ticketed_add(state, sum, kCountGroups);
}

// ---- buffer access for the streaming kernels.  A row piece is addressed as a raw buffer: its base and its
// length in bytes sit in scalar registers, every lane adds its own byte offset, and the hardware's range check
// does the masking: a load at or past the end returns 0, a store there is dropped.  Only used where a lane's
// piece lies entirely inside or entirely outside the row (no partial pieces).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t row_buffer(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);   // raw, 32-bit data
}
constexpr int kWriteThrough = 16;     // cache policy sc1: written through to memory at device scope (see store_through)
constexpr int kStreamThrough = 18;    // sc1 nt: the same as a stream
__device__ __forceinline__ uint4 buffer_load16(rsrc_t r, int byte_offset) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, byte_offset, 0, 0));
}

// INT8 codes of 8 elements as 8 bytes (the low mantissa byte of kMagic + q is q in two's complement)
__device__ __forceinline__ u32x2 pack_codes_i8(const float (&m)[8]) {
    uint32_t u[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) u[e] = __float_as_uint(m[e]);
    return u32x2{pack_bytes(u[0], u[1], u[2], u[3]), pack_bytes(u[4], u[5], u[6], u[7])};
}
// INT4 codes of 8 elements as 4 bytes: two's-complement nibbles, even column in the low nibble
__device__ __forceinline__ uint32_t pack_codes_i4(const float (&m)[8]) {
    uint32_t u[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) u[e] = __float_as_uint(m[e]);
    uint32_t w0 = pack_bytes(u[0], u[1], u[2], u[3]) & 0x0F0F0F0Fu;
    uint32_t w1 = pack_bytes(u[4], u[5], u[6], u[7]) & 0x0F0F0F0Fu;
    w0 |= w0 >> 4;                 // bytes 0 and 2 now hold two nibbles each
    w1 |= w1 >> 4;
    return __builtin_amdgcn_perm(w1, w0, 0x06040200u);
}
// dequantized values fl16(fl32(q * fl32(a * b))) of 8 elements as 16 bytes
__device__ __forceinline__ u32x4 pack_xhat(const float (&q)[8], float a, const float (&b)[8]) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = rounded_f32(q[e] * (a * b[e]));
    return u32x4{pack_half2(y[0], y[1]), pack_half2(y[2], y[3]), pack_half2(y[4], y[5]), pack_half2(y[6], y[7])};
}

// A piece of N bytes at dst, which need not be aligned; of a piece at the end of a row only the first n bytes (whole U's).
template <int N, typename U, typename V>
__device__ __forceinline__ void store_piece(V v, void* dst, int n) {
    static_assert(sizeof(V) == N, "a whole piece");
    if (n == N) {
        __builtin_memcpy(dst, &v, N);
    } else if (n > 0) {
        U u[N / sizeof(U)];
        __builtin_memcpy(u, &v, N);
#pragma unroll
        for (int e = 0; e < (int)(N / sizeof(U)); ++e)
            if (e * (int)sizeof(U) < n) static_cast<U*>(dst)[e] = u[e];
    }
}

// INT4 codes as FP6 E2M3 fragments, the operand format of the A4W4 matrix kernel: a fragment is 32
// rows x 64 columns = 1536 bytes, fragments ordered [row / 32][column / 64]; fragment lane
// (row & 31) + 32 * ((column / 32) & 1) holds 32 consecutive columns as a 192-bit little-endian
// stream of 6-bit fields, its first 16 bytes at fragment + 16 * lane, the last 8 at fragment + 1024
// + 8 * lane.  The wave's lanes 4g .. 4g+3 hold the 32 columns of group g (8 each).
// They are written four rows at a time (rows 4 k .. 4 k + 3 of one matrix, as the streaming kernel
// works on them): a lane keeps its eight codes of each of the four rows as binary16 (exact), then the quad transposes them
// (quad-permuting selects, no LDS) so that lane 4 g + u holds the 32 codes of row u, which one instruction turns
// into the 24-byte record (E2M3 holds every code exactly), and each lane stores one 16-byte and one 8-byte piece: a quad
// writes 64 and 32 contiguous bytes.  The kernel is bound by vector instructions, 8.8 per element with this (12.5 with E2M3
// fields from table lookups and shifts and a transposition of 48-bit pieces): 4096 x 4096 9.9 -> 8.7 us, 4096 x 8192 18.3 -> 16.7.
struct Fp6Batch {
    uint32_t h[4][4];           // [pair of columns][row]: this lane's codes, two binary16 values each
};
// row u (0..3) of the batch: the lane's 8 codes
__device__ __forceinline__ void fp6_batch_row(Fp6Batch& out, const float (&q)[8], int u) {
#pragma unroll
    for (int p = 0; p < 4; ++p) out.h[p][u] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(q[2 * p], q[2 * p + 1]));
}
// One exchange step of the 4 x 4 transposition over a quad, for eight pairs of registers: the lanes of `mask` (32 bits,
// repeated) keep their own register, the others take one of their partner's:
//   o[i] = lane in mask ? keep[i] : (partner lane's) take[i]
// v_cndmask takes its second source where vcc is set and its first, here read from the partner lane, elsewhere.  (The
// compiler makes a move and a select of each.)  The two wait states are those between a vector instruction
// that writes a register and one that reads it from another lane.
#define CQ_QUAD_STEP(NAME, PERM)                                                                                             \
    template <uint32_t MASK>                                                                                                 \
    __device__ __forceinline__ void NAME(uint32_t (&o)[8], const uint32_t (&take)[8], const uint32_t (&keep)[8]) {           \
        asm("s_mov_b32 vcc_lo, %24\n\ts_mov_b32 vcc_hi, %24\n\ts_nop 1\n\t"                                                 \
            "v_cndmask_b32_dpp %0, %8, %16, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                           \
            "v_cndmask_b32_dpp %1, %9, %17, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                           \
            "v_cndmask_b32_dpp %2, %10, %18, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                          \
            "v_cndmask_b32_dpp %3, %11, %19, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                          \
            "v_cndmask_b32_dpp %4, %12, %20, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                          \
            "v_cndmask_b32_dpp %5, %13, %21, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                          \
            "v_cndmask_b32_dpp %6, %14, %22, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                          \
            "v_cndmask_b32_dpp %7, %15, %23, vcc quad_perm:" PERM " row_mask:0xf bank_mask:0xf"                               \
            : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7])          \
            : "v"(take[0]), "v"(take[1]), "v"(take[2]), "v"(take[3]), "v"(take[4]), "v"(take[5]), "v"(take[6]), "v"(take[7]), \
              "v"(keep[0]), "v"(keep[1]), "v"(keep[2]), "v"(keep[3]), "v"(keep[4]), "v"(keep[5]), "v"(keep[6]), "v"(keep[7]), \
              "i"(MASK)                                                                                                       \
            : "vcc");                                                                                                         \
    }
CQ_QUAD_STEP(quad_neighbours, "[1,0,3,2]")
CQ_QUAD_STEP(quad_pairs, "[2,3,0,1]")
#undef CQ_QUAD_STEP
// h[p][k] = this lane's value of row k  ->  r[4 k + p] = the value lane k of the quad had for row (lane & 3)
__device__ __forceinline__ void quad_transpose(const uint32_t (&h)[4][4], uint32_t (&r)[16]) {
    // neighbours exchange: an even lane ends up with rows 0 and 2 of both lanes (even[..]: the even lane's, odd[..]: the odd
    // one's), an odd lane with rows 1 and 3
    uint32_t row_e[8], row_o[8];                            // [2 p + 0]: rows 0 / 1, [2 p + 1]: rows 2 / 3
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        row_e[2 * p] = h[p][0];
        row_e[2 * p + 1] = h[p][2];
        row_o[2 * p] = h[p][1];
        row_o[2 * p + 1] = h[p][3];
    }
    uint32_t even[8], odd[8];
    quad_neighbours<0x55555555u>(even, row_o, row_e);
    quad_neighbours<0xAAAAAAAAu>(odd, row_e, row_o);
    // pairs exchange: lanes 0, 1 give away their rows 2, 3 and lanes 2, 3 their rows 0, 1
    uint32_t low[8], high[8], first[8], second[8];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        low[p] = even[2 * p];
        low[4 + p] = odd[2 * p];
        high[p] = even[2 * p + 1];
        high[4 + p] = odd[2 * p + 1];
    }
    quad_pairs<0x33333333u>(first, high, low);
    quad_pairs<0xCCCCCCCCu>(second, low, high);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        r[i] = first[i];                                    // lanes 0 and 1 of the quad
        r[8 + i] = second[i];
    }
}
// rows row4 .. row4 + 3 (row4 % 4 == 0); rows_ok: bit u set if row row4 + u exists; group_ok: the lane's columns exist.
// The four rows lie in one row of fragments, which is addressed as a raw buffer (frags_per_row * 1536 bytes).
// Must be called by the whole wave (the transposition exchanges registers between lanes).
__device__ __forceinline__ void fp6_batch_store(const Fp6Batch& out, uint8_t* packed, int row4, int first_col, int lane,
                                                int frags_per_row, uint32_t rows_ok, bool group_ok) {
    typedef _Float16 f16x32 __attribute__((ext_vector_type(32)));
    typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
    struct Regs {
        uint32_t r[16];
    } codes;
    quad_transpose(out.h, codes.r);
    const u32x6 rec = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(__builtin_bit_cast(f16x32, codes), 1.0f);
    const int u = lane & 3, g = lane >> 2;
    const int col = first_col + 32 * g;
    const int flane = ((row4 + u) & 31) + 32 * ((col >> 5) & 1);
    const bool ok = group_ok && ((rows_ok >> u) & 1u);
    const rsrc_t frow = row_buffer(packed + (int64_t)(row4 >> 5) * frags_per_row * 1536, frags_per_row * 1536);
    // a lane that must not store points past the buffer's end: the hardware's range check drops its stores
    const int off = ok ? (col >> 6) * 1536 : 0x7FFF0000;
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{rec[0], rec[1], rec[2], rec[3]}, frow, off + flane * 16, 0, kWriteThrough);
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{rec[4], rec[5]}, frow, off + 1024 + flane * 8, 0, kWriteThrough);
}

}  // namespace cq
