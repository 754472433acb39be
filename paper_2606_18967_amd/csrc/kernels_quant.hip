// kernels_quant.hip -- drafter refresh: RTN quantization of a weight matrix
// into the packed tile layout read by the drafter GEMMs (Sec. 4.1: the FFN
// and QKVO projections are re-quantized at every training step).
//
// Groups of 128 consecutive weights along K within an output row, one fp16
// scale each:
//   int4 symmetric:   s = fp16(max|w| / 7),   q = clamp(rint(w / s), -8, 7)
//   int4 asymmetric:  s = fp16((max - min) / 15), z = clamp(rint(-min / s), 0, 15),
//                     q = clamp(rint(w / s) + z, 0, 15)   (App. B.2)
//   int8 symmetric:   s = fp16(max|w| / 127), q = clamp(rint(w / s), -128, 127)
// (q = 0, z = 0 when s = 0).  fp32 division is correctly rounded and rint
// rounds half to even, so codes, scales and zero points are a deterministic
// function of the weights.
#include "common.h"
#include "kernels.h"

namespace {

// The codes of one wave's tile, by the formulas above: w(st, e) is this lane's
// weight e of k-step st, word(j, bits) takes its packed words in order.
template <int FMT, typename WT, typename WORD>
__device__ __forceinline__ void codes_general(const WT& w, float s, int z, const WORD& word)
{
    auto code = [&](float x) {   // the stored (unsigned) code
        if (s == 0.f) return FMT == QF_W4 ? 8 : (FMT == QF_W8 ? 128 : 0);
        const float r = rintf(x / s);
        if (FMT == QF_W4) return (r < -8.f ? -8 : (r > 7.f ? 7 : (int)r)) + 8;
        if (FMT == QF_W8) return (r < -128.f ? -128 : (r > 127.f ? 127 : (int)r)) + 128;
        const float rz = r + (float)z;
        return rz < 0.f ? 0 : (rz > 15.f ? 15 : (int)rz);
    };
    constexpr int EPW = FMT == QF_W8 ? 4 : 8;
#pragma unroll
    for (int j = 0; j < 64 / EPW; ++j) {
        uint32_t bits = 0;
#pragma unroll
        for (int b = 0; b < EPW; ++b) {
            const int e = j * EPW + b;
            bits |= (uint32_t)code(w(e >> 3, e & 7)) << (FMT == QF_W8 ? 8 * b : 4 * (b >> 1) + 16 * (b & 1));
        }
        word(j, bits);
    }
}

// The same for bf16 weights and a scale in [2^-14, inf) (a normal fp16), all
// weights finite: six vector instructions a weight where the correctly rounded
// division and the conversions take about 24 (they bounded the refresh: four
// layers of the 8B shape 590 -> 423 us, now 5.2 TB/s of HBM).  The quotient is a product with 1 / s
// and one correction, which is exact where w / s has few bits (ties, k + 1/2)
// and elsewhere off by less than 2^-22 of it; w has 8 significant bits and s
// has 11, so a quotient that is no tie is at least 2^-20 of itself from one (2 k + 1 <= 257),
// and both round to the same integer.  Adding 1.5 2^23 rounds to nearest even
// and leaves the integer in the low bits; the sum of the shifted bits less the
// constants is the word.  The symmetric formats need no clamp here: s is within
// 2^-11 of max|w| / 7 (127), so no quotient rounds past +-7 (127).
template <int FMT, typename WT, typename WORD>
__device__ __forceinline__ void codes_bf16(const WT& w, float s, int z, const WORD& word)
{
    constexpr int EPW = FMT == QF_W8 ? 4 : 8;
    constexpr uint32_t ONES = FMT == QF_W8 ? 0x01010101u : 0x11111111u, MAGIC = 0x4B400000u;
    const uint32_t off = (FMT == QF_W4 ? 8u : FMT == QF_W8 ? 128u : (uint32_t)z) * ONES - MAGIC * ONES;
    const float inv = 1.f / s, zl = -(float)z, zh = 15.f - (float)z;
#pragma unroll
    for (int j = 0; j < 64 / EPW; ++j) {
        uint32_t bits = off;
#pragma unroll
        for (int b = 0; b < EPW; ++b) {
            const int e = j * EPW + b;
            const float x = w(e >> 3, e & 7), q0 = x * inv;
            float q = __builtin_fmaf(__builtin_fmaf(-q0, s, x), inv, q0);
            if (FMT == QF_W4A) q = __builtin_amdgcn_fmed3f(q, zl, zh);
            bits += __float_as_uint(q + 12582912.f) << (FMT == QF_W8 ? 8 * b : 4 * (b >> 1) + 16 * (b & 1));
        }
        word(j, bits);
    }
}

constexpr int QWV = 4;              // most waves per work-group

// One wave per (32-column block nb, group g), the work-group's waves on
// consecutive groups.  Lane l takes column 32 nb + (l & 31) and k-half
// h = l >> 5: for k-step st = 0..7 the 8 weights k = 128 g + 16 st + 8 h + e.
// In the int4 formats they become its packed word st (code e in the nibble at
// bit 4 (e / 2) + 16 (e % 2)); in the int8 format its words 2 st and 2 st + 1
// (code e in byte e % 4 of word 2 st + e / 4) -- the B operand layout of the
// GEMM's MFMA k-step st (kernels_q4.hip).
template <typename T, int FMT>
__global__ void __launch_bounds__(64 * QWV) k_quant_rtn(const T* __restrict__ W, int NB, int K, uint32_t* __restrict__ Wq,
                                                        uint16_t* __restrict__ Sc, uint8_t* __restrict__ Z)
{
    constexpr bool BF = sizeof(T) == 2;
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63;
    const int G = K / 128;
    const long long t = (long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= (long long)NB * G) return;
    const int nb = (int)(t / G), g = (int)(t - (long long)nb * G);
    const int n = nb * 32 + (lane & 31), h = lane >> 5;
    const T* wr = W + (size_t)n * K + (size_t)g * 128 + 8 * h;
    constexpr int PIECES = BF ? 1 : 2;                 // 16-byte pieces of 8 weights
    u32x4 raw[8][PIECES];
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
        for (int i = 0; i < PIECES; ++i) raw[st][i] = *((const u32x4*)(wr + 16 * st) + i);
    auto w = [&](int st, int e) {
        if constexpr (BF) {
            const uint32_t p = raw[st][0][e >> 1];
            return __uint_as_float(e & 1 ? p & 0xFFFF0000u : p << 16);
        } else {
            return __uint_as_float(raw[st][e >> 2][e & 3]);
        }
    };
    float amax = 0.f, lo = INFINITY, hi = -INFINITY;
    bool odd = !BF;                                    // a weight that is no finite bf16
    if constexpr (BF) {
        // magnitudes compare as integers; NaN and infinity are 0x7F80 and above
        u16x2 m = {0, 0};
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, raw[st][0][i] & 0x7FFF7FFFu));
        const uint32_t top = m[0] > m[1] ? m[0] : m[1];
        odd = __any(top >= 0x7F80u);
        amax = __uint_as_float(top << 16);
    }
    if (odd || FMT == QF_W4A) {
        amax = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = w(st, e);
                amax = fmaxf(amax, fabsf(x));
                lo = fminf(lo, x);
                hi = fmaxf(hi, x);
            }
    }
    amax = fmaxf(amax, __shfl_xor(amax, 32, WAVE));
    lo = fminf(lo, __shfl_xor(lo, 32, WAVE));
    hi = fmaxf(hi, __shfl_xor(hi, 32, WAVE));
    const _Float16 sh = (_Float16)(FMT == QF_W4 ? amax / 7.0f : (FMT == QF_W8 ? amax / 127.0f : (hi - lo) / 15.0f));
    const float s = (float)sh;
    int z = 0;
    if (FMT == QF_W4A && s != 0.f) {
        const float zr = rintf(-lo / s);
        z = zr < 0.f ? 0 : (zr > 15.f ? 15 : (int)zr);
    }
    constexpr int NW = FMT == QF_W8 ? 16 : 8;          // words per lane
    u32x4 out[NW / 4];
    auto word = [&](int j, uint32_t bits) { out[j >> 2][j & 3] = bits; };
    if (odd || __any(!(s >= 0x1p-14f && s < INFINITY))) codes_general<FMT>(w, s, z, word);
    else codes_bf16<FMT>(w, s, z, word);
    u32x4* dst = (u32x4*)Wq + ((size_t)nb * G + g) * (16 * NW);
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) dst[64 * i + lane] = out[i];
    if (lane < 32) {
        Sc[((size_t)nb * G + g) * 32 + lane] = __builtin_bit_cast(uint16_t, sh);
        if (FMT == QF_W4A) Z[((size_t)nb * G + g) * 32 + lane] = (uint8_t)z;
    }
}

template <typename T>
void quant_t(int fmt, const T* W, int N, int K, uint32_t* Wq, uint16_t* Sc, uint8_t* Z, hipStream_t s)
{
    const long long tiles = (long long)(N / 32) * (K / 128);
    // four waves per work-group (a row's 1 KB read together), one where the chip
    // has room for a work-group per tile
    const int wv = tiles < 4096 ? 1 : QWV;
    const dim3 grid((unsigned)((tiles + wv - 1) / wv));
    if (fmt == QF_W4A) k_quant_rtn<T, QF_W4A><<<grid, 64 * wv, 0, s>>>(W, N / 32, K, Wq, Sc, Z);
    else if (fmt == QF_W8) k_quant_rtn<T, QF_W8><<<grid, 64 * wv, 0, s>>>(W, N / 32, K, Wq, Sc, Z);
    else k_quant_rtn<T, QF_W4><<<grid, 64 * wv, 0, s>>>(W, N / 32, K, Wq, Sc, Z);
}

}  // namespace

void launch_quant(int fmt, const void* W, int w_f32, int N, int K, uint32_t* Wq, uint16_t* Sc, uint8_t* Z,
                  hipStream_t s)
{
    if (w_f32) quant_t<float>(fmt, (const float*)W, N, K, Wq, Sc, Z, s);
    else quant_t<uint16_t>(fmt, (const uint16_t*)W, N, K, Wq, Sc, Z, s);
}
