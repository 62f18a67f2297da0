// tgl_timeenc.hip -- time encoding of sampled slots (Equation 3 of TGL: the
// time encoder of Section 2 maps a time difference dt to the vector
// cos(omega * dt + phi), omega and phi learnable vectors of the encoder's
// dimension).
//
// Each slot's row is dim independent elements, so the encoding is bound by the
// bytes it writes (dim * 4 or dim * 2 per slot against 4 read).  16-byte output
// words are dealt to the lanes of the grid such that a lane's columns never
// change (timeenc_word_kernel); rows of fewer elements than a word, or an
// output that is not 16-byte aligned, take a wavefront per row
// (timeenc_kernel).
//
// Accuracy: the argument is formed in turns, (omega / 2 pi) dt + phi / 2 pi, or
// quarter turns, in double precision from per-column factors omega / 2 pi and
// phi / 2 pi (each within 2^-52 relative of exact): below 2^24 turns it is
// within 5e-8 rad of the exact argument.  What it has above whole turns or
// quarters is exact, and is rounded to float only after that, for a polynomial
// of the cosine evaluated by fused multiply-adds.
//   timeenc_kernel: f = t - rint(t), and cos(2 pi f) = cos(2 pi g) for g = |f| in
//     [0, 1/2]; above 1/4 it is -cos(2 pi (1/2 - g)), so only [0, 1/4] is left: x =
//     2 pi g in [0, pi/2], where the cosine's Taylor series to x^12, in powers of
//     g^2, leaves out less than 6.4e-9.  Measured against 64 bits, 2.8e-8 (2-norm)
//     and 1.7e-7 at most;
//   timeenc_word_kernel: cos_quarters, 1.8e-8 and 9e-8, and 1.7e-8 and 3.1e-8 where
//     the argument is below 0.1.
// A plain float evaluation of the argument would be off by up to half an ulp
// of omega * dt -- 0.125 at dt = 2.7e6 s, Wikipedia's time span -- which the
// cosine passes on unchanged.  Arguments of 2^24 turns or more have a reduction
// of their own (far_quarters), or the double cosine.
//
// Padded slots (dt < 0) have no time difference: their rows are zeros.
#include <atomic>

#include "tgl_internal.hpp"

namespace tgl {
namespace {

constexpr int kRows = 16;                                          // slots per wavefront pass
constexpr double kInvTwoPi = 0.15915494309189535;                  // 1 / (2 pi), nearest double
constexpr double kTurnLimit = 0x1p24;                              // turns reduced in double below this
constexpr int kMaxPre = 1024;                                      // columns whose factors fit in LDS

// cos(2 pi g) = sum_n c_n g^(2n), c_n = (-1)^n (2 pi)^(2n) / (2n)!  (n <= 6)
constexpr float kC1 = -19.739208802178717f;
constexpr float kC2 = 64.93939402266829f;
constexpr float kC3 = -85.45681720669373f;
constexpr float kC4 = 60.24464137187666f;
constexpr float kC5 = -26.426256783374397f;
constexpr float kC6 = 7.903536371318469f;

// cos(z pi / 2) = 1 + z^2 (kE1 + ... + kE4 z^6) and sin(z pi / 2) = z (kS1 +
// ... + kS7 z^6) for |z| <= 1/2; sin(z pi / 2) = z + z (1 - z^2) (kR0 + ... + kR3
// z^6) for |z| <= 1: see cos_quarters
constexpr float kE1 = -1.2337005138397217f;
constexpr float kE2 = 0.25366851687431335f;
constexpr float kE3 = -0.0208552535623312f;
constexpr float kE4 = 0.0008935732766985893f;
constexpr float kS1 = 1.5707963705062866f;
constexpr float kS3 = -0.6459648013114929f;
constexpr float kS5 = 0.0796898826956749f;
constexpr float kS7 = -0.00462295301258564f;
constexpr float kR0 = 0.5707963109016418f;
constexpr float kR1 = -0.075167216360569f;
constexpr float kR2 = 0.0045216684229671955f;
constexpr float kR3 = -0.00015092534886207432f;

constexpr double kQuarters = 0.6366197723675814;                   // 2 / pi, nearest double, ...
constexpr double kQuartersLow = -3.935735335036497e-17;            // ... and what it leaves out
constexpr double kOnes = 0x1.8p52;                                 // doubles near it are 1 apart
constexpr double kFours = 0x1.8p54;                                // doubles near it are 4 apart

// An argument of 2^26 quarter turns or more is reduced by far_quarters, from
// 2^50 rad on by the double cosine; below kNearRad radians, |omega| dt + |phi|
// in float, none of a lane's columns has one.
constexpr double kQuarterLimit = 0x1p26;
constexpr float kNearRad = 1.0541e8f;
constexpr float kFarRad = 0x1p50f;

using i32x4 = int __attribute__((ext_vector_type(4)));

// cos(2 pi t) for an argument t in turns with |t| < kTurnLimit
__device__ __forceinline__ float cos_turns(double t) {
    const double f = t - rint(t);                                  // exact, in [-1/2, 1/2]
    const double a = fabs(f);
    const bool flip = a > 0.25;                                    // cos(2 pi a) = -cos(2 pi (1/2 - a))
    const float g = static_cast<float>(fmin(a, 0.5 - a));         // 0.5 - a is exact; flip picks it
    const float y = g * g;
    float c = __builtin_fmaf(y, kC6, kC5);
    c = __builtin_fmaf(y, c, kC4);
    c = __builtin_fmaf(y, c, kC3);
    c = __builtin_fmaf(y, c, kC2);
    c = __builtin_fmaf(y, c, kC1);
    c = __builtin_fmaf(y, c, 1.0f);
    return flip ? -c : c;
}

// cos(omega dt + phi) from wp = omega / 2 pi and pp = phi / 2 pi; omega[j] and
// phi[j] are read only for the double-precision fallback.
__device__ __forceinline__ float encode(double wp, double pp, float dt, const float *__restrict__ omega,
                                        const float *__restrict__ phi, int j) {
    const double t = fma(wp, static_cast<double>(dt), pp);        // the argument in turns
    if (!(fabs(t) < kTurnLimit))                                   // huge, infinite or NaN
        return static_cast<float>(cos(fma(static_cast<double>(omega[j]), static_cast<double>(dt),
                                          static_cast<double>(phi[j]))));
    return cos_turns(t);
}

// the per-column factors (omega / 2 pi, phi / 2 pi) of columns [0, dim), into
// LDS by the whole block (dim <= kMaxPre)
__device__ __forceinline__ void load_factors(double2 *__restrict__ f, const float *__restrict__ omega,
                                             const float *__restrict__ phi, int dim) {
    for (int j = threadIdx.x; j < dim; j += kBlock)
        f[j] = make_double2(static_cast<double>(omega[j]) * kInvTwoPi, static_cast<double>(phi[j]) * kInvTwoPi);
    __syncthreads();
}

// float -> bfloat16, round to nearest even (NaN stays a quiet NaN)
__device__ __forceinline__ uint16_t to_bf16(float v) {
    const uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((b >> 16) | 0x40u);
    return static_cast<uint16_t>((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

// Two floats as bfloat16, a in the low half (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ int pack_bf16(float a, float b) {
    using f32x2 = float __attribute__((ext_vector_type(2)));
    using bf16x2 = __bf16 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(int, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// Rows by wavefronts, kRows slots at a time: one vector load brings their
// time differences (lane u holds slot u's), each is broadcast from its lane,
// and lane l computes elements l, l + 64, ... of the row.
template <int OUT, bool PRE>
__global__ __launch_bounds__(kBlock) void timeenc_kernel(const float *__restrict__ dt, int64_t n,
                                                         const int64_t *__restrict__ count, int64_t per,
                                                         const float *__restrict__ omega,
                                                         const float *__restrict__ phi, int dim,
                                                         void *__restrict__ out) {
    __shared__ double2 fac[PRE ? kMaxPre : 1];
    if constexpr (PRE) load_factors(fac, omega, phi, dim);
    const int lane = lane_id();
    constexpr int kWaves = kBlock / kWave;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * kWaves;
    const int64_t wave = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * kWaves + threadIdx.x / kWave));
    if (count) {
        // valid prefix: min(n, count * per), without overflowing the product
        const int64_t c = *count;
        const int64_t lim = c <= 0 ? 0 : (c > n / per ? n : c * per);
        n = lim < n ? lim : n;
    }
    for (int64_t r0 = wave * kRows; r0 < n; r0 += waves * kRows) {
        const float dl = lane < kRows && r0 + lane < n ? dt[r0 + lane] : -1.0f;
#pragma unroll 1
        for (int u = 0; u < kRows; u++) {
            const int64_t row = r0 + u;
            if (row >= n) break;                                   // wavefront-uniform
            const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dl), u));
            const int64_t base = row * dim;
            if (d >= 0.0f) {                                       // wavefront-uniform
                for (int j = lane; j < dim; j += kWave) {
                    const double2 fj = PRE ? fac[j]
                                           : make_double2(static_cast<double>(omega[j]) * kInvTwoPi,
                                                          static_cast<double>(phi[j]) * kInvTwoPi);
                    const float v = encode(fj.x, fj.y, d, omega, phi, j);
                    if constexpr (OUT == TGL_OUT_F32)
                        __builtin_nontemporal_store(v, static_cast<float *>(out) + base + j);
                    else
                        __builtin_nontemporal_store(to_bf16(v), static_cast<uint16_t *>(out) + base + j);
                }
            } else {
                for (int j = lane; j < dim; j += kWave) {
                    if constexpr (OUT == TGL_OUT_F32)
                        __builtin_nontemporal_store(0.0f, static_cast<float *>(out) + base + j);
                    else
                        __builtin_nontemporal_store(static_cast<uint16_t>(0), static_cast<uint16_t *>(out) + base + j);
                }
            }
        }
    }
}

// cos(t pi / 2) for an argument t in quarter turns, |t| < 2^51.
//
// float32: t is a whole number q of quarters plus z of one, |z| <= 1/2, and the
// result plus or minus cos(z pi / 2) or sin(z pi / 2), which q decides.  Both
// polynomials (minimax fits, errors 4e-10 and 4e-9) are evaluated and one is
// taken.  Near 1 the result is 1 minus a small sum, rounded once, as a cosine
// series gives it.  One polynomial for the sine of the complement over a whole
// quarter needs 7 instructions fewer; as an odd series it adds two terms of
// the size of 1 there, with errors up to 1.3e-7 instead of 3e-8 for arguments
// below 0.1 and results above 1.
//
// bfloat16, whose rounding hides the difference and whose words, half as
// many bytes, are bound by instructions: that complement z = 1 - |r|, r in
// [-2, 2] quarters, and the correction to z of sin(z pi / 2), which vanishes at 0
// and 1 (minimax fit, error 5e-9), so that the result never exceeds 1 either:
// 8.5e-8 at most before the rounding.
template <int OUT>
__device__ __forceinline__ float cos_quarters(double t) {
    if constexpr (OUT == TGL_OUT_F32) {
        const double m = t + kOnes;
        const float z = static_cast<float>(t - (m - kOnes));
        const uint32_t q = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, m));
        const float y = z * z;
        float c = __builtin_fmaf(y, kE4, kE3);
        c = __builtin_fmaf(y, c, kE2);
        c = __builtin_fmaf(y, c, kE1);
        c = __builtin_fmaf(y, c, 1.0f);
        float s = __builtin_fmaf(y, kS7, kS5);
        s = __builtin_fmaf(y, s, kS3);
        s = __builtin_fmaf(y, s, kS1);
        s = z * s;
        const float r = (q & 1u) != 0 ? s : c;
        return __uint_as_float(__float_as_uint(r) ^ (((q + 1u) << 30) & 0x80000000u));   // q mod 4 = 1, 2
    } else {
        const double r = t - ((t + kFours) - kFours);
        const float z = static_cast<float>(1.0 - fabs(r));
        const float y = z * z;
        float p = __builtin_fmaf(y, kR3, kR2);
        p = __builtin_fmaf(y, p, kR1);
        p = __builtin_fmaf(y, p, kR0);
        return __builtin_fmaf(z * __builtin_fmaf(-z, z, 1.0f), p, z);
    }
}

// omega dt + phi in quarter turns, less a multiple of 4 of them, for arguments
// below 2^50 rad, from wq = 2 omega / pi and pq = 2 phi / pi as the kernel holds
// them: omega is wq pi / 2 rounded to float, omega dt exact in double, and its
// product with 2 / pi taken to 106 bits (2^-54 quarters of error).
__device__ __forceinline__ double far_quarters(double wq, double pq, double dt) {
    const double x = static_cast<double>(static_cast<float>(wq * (1.0 / kQuarters))) * dt;
    const double h = x * kQuarters;
    const double l = fma(x, kQuartersLow, fma(x, kQuarters, -h));
    return (h - ((h + kFours) - kFours)) + (l + pq);
}

// Words of a lane whose time differences are loaded ahead: with dt in memory
// 100 float32 of 8M slots take 818, 717 and 596 us with 1, 2 and 4.
constexpr int kAhead = 4;

// Blocks that share `words` 16-byte words: one per `lane_words` words of its
// lanes, at most `most`, and a multiple of `unit`; or a block per 256 words
// when that is no more than `unit` (one word per lane: no step is taken).
__host__ __device__ __forceinline__ uint32_t word_blocks(int64_t words, int lane_words, uint32_t most, uint32_t unit) {
    const int64_t whole = words / kBlock + (words % kBlock != 0);
    const int64_t even = whole / lane_words + (whole % lane_words != 0);
    uint32_t nb = even < most ? static_cast<uint32_t>(even) : most;
    nb = nb / unit * unit;
    nb = nb < unit ? unit : nb;
    return whole < nb ? static_cast<uint32_t>(whole) : nb;
}

// Lane l of the grid owns the 16-byte output words l, l +
// T, ... (EPW elements each: 4 float32 or 8 bfloat16; T lanes in all), so one
// store instruction writes 1 KB of contiguous output.  T * EPW is a multiple
// of dim whenever a lane has more than one word, so its columns never change:
// their factors stay in registers and its row advances by row_step.  With
// STRADDLE a row is not a whole number of words: a word's elements from
// column dim on belong to the next row, and the last word may end early.
//
// A lane loads the time differences of kAhead words before it encodes and
// stores the kAhead before them.  Loads and stores complete in order, so that a
// load after a store waits for it too, and with a load per word that is what a
// word took where dt came from memory (a step's 8M slots, half of them PAD, 100
// float32: 856 -> 597 us; dt in the cache and no PAD 566 -> 580).
//
// The argument is one double fma per element, in quarter turns; one float fma
// per word tells whether any of its arguments needs far_quarters.  What an
// element becomes depends on its own dt, omega and phi alone.  19 instructions
// per float32 element, 5 of them double.  Against the reduction to turns, fold
// and Taylor series of timeenc_kernel with the factors in LDS (same inputs,
// before -> now): 100 float32 of 8M slots 692 -> 597 us with dt in memory (5.7
// TB/s; a plain fill writes 6.9) and 824 -> 580 with dt in the cache and no PAD,
// 101 of 2M 395 -> 197, 100 bfloat16 of 8M 1027 -> 454 and 1157 -> 505; where a
// third of the slots have arguments of 2^24 turns or more, 100 float32 of 2M
// 396 -> 181, 172 bfloat16 499 -> 275.
template <int OUT, bool STRADDLE>
__global__ __launch_bounds__(kBlock) void timeenc_word_kernel(const float *__restrict__ dt, int64_t n,
                                                              const int64_t *__restrict__ count, int64_t per,
                                                              const float *__restrict__ omega,
                                                              const float *__restrict__ phi, int dim,
                                                              int lane_words, uint32_t most, uint32_t unit,
                                                              void *__restrict__ out) {
    constexpr int EPW = OUT == TGL_OUT_F32 ? 4 : 8;                 // elements per 16-byte word
    if (count) {
        const int64_t c = *count;
        const int64_t lim = c <= 0 ? 0 : (c > n / per ? n : c * per);
        n = lim < n ? lim : n;
    }
    const int64_t elems = n * dim;
    const int64_t total = (elems + EPW - 1) / EPW;                  // words
    // the blocks that the slots counted on the device need: the grid is for
    // all n, and with few of them valid its other blocks end here
    const uint32_t nb = word_blocks(total, lane_words, most, unit);
    if (blockIdx.x >= nb) return;
    const int64_t T = static_cast<int64_t>(nb) * kBlock;
    const int64_t row_step = T * EPW / dim;
    int64_t w = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (w >= total) return;
    int64_t row = w * EPW / dim;
    const int col = static_cast<int>(w * EPW - row * dim);
    double wq[EPW], pq[EPW];                                        // quarter turns
    float om = 0.0f, pm = 0.0f;                                     // the largest |omega| and |phi|
#pragma unroll
    for (int e = 0; e < EPW; e++) {
        const int j = STRADDLE && col + e >= dim ? col + e - dim : col + e;
        wq[e] = static_cast<double>(omega[j]) * kQuarters;
        pq[e] = static_cast<double>(phi[j]) * kQuarters;
        om = fmaxf(om, fabsf(omega[j]));
        pm = fmaxf(pm, fabsf(phi[j]));
    }
    // the lane's words: every lane of the launch has total / T, some one more
    const int64_t each = total / T;
    int64_t left = each + (w < total - each * T);
    i32x4 *o = static_cast<i32x4 *>(out) + w;
    const i32x4 *const o_last = static_cast<i32x4 *>(out) + (total - 1);
    // time differences of the lane's next kAhead words (STRADDLE: and of the rows
    // after theirs); past its last word, of its first row
    struct Ahead {
        float d0[kAhead], d1[kAhead];
    };
    const int64_t row0 = row;
    const auto load_ahead = [&](int64_t r0, int64_t words) {
        Ahead a;
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
            const int64_t r = u < words ? r0 + u * row_step : row0;
            a.d0[u] = dt[r];
            a.d1[u] = STRADDLE ? dt[r + 1 < n ? r + 1 : r] : a.d0[u];
        }
        return a;
    };
    Ahead now = load_ahead(row, left);
    // in registers here, so that the loop holds no wait for them
#pragma unroll
    for (int u = 0; u < kAhead; u++) asm volatile("" : "+v"(now.d0[u]), "+v"(now.d1[u]));
    for (;;) {
        row += kAhead * row_step;
        const Ahead next = load_ahead(row, left - kAhead);
        const int words = left < kAhead ? static_cast<int>(left) : kAhead;
#pragma unroll                                                      // 4% over a loop that moves now.d0 down
        for (int u = 0; u < kAhead; u++, o += T) {
            if (u >= words) break;
            const float d0 = now.d0[u], d1 = now.d1[u];
            float v[EPW];
#pragma unroll
            for (int e = 0; e < EPW; e++) v[e] = 0.0f;
            // PAD slots; a NaN time difference gives NaN, or zeros in rows that
            // are not whole words
            const bool pad0 = STRADDLE ? !(d0 >= 0.0f) : d0 < 0.0f;
            const bool pad1 = STRADDLE ? !(d1 >= 0.0f) : pad0;
            if (!pad0 || !pad1) {
                double t[EPW];
#pragma unroll
                for (int e = 0; e < EPW; e++)
                    t[e] = fma(wq[e], static_cast<double>(STRADDLE && col + e >= dim ? d1 : d0), pq[e]);
                // a bound of every |argument| of the word (a NaN or infinite one
                // gives NaN with or without the reduction)
                const float far = __builtin_fmaf(om, fmaxf(d0, d1), pm);
                if (far >= kNearRad) {
#pragma unroll
                    for (int e = 0; e < EPW; e++)
                        if (fabs(t[e]) >= kQuarterLimit)
                            t[e] = far_quarters(wq[e], pq[e], static_cast<double>(STRADDLE && col + e >= dim ? d1 : d0));
                }
#pragma unroll
                for (int e = 0; e < EPW; e++) v[e] = cos_quarters<OUT>(t[e]);
                if (far >= kFarRad) {
                    // one element after the other: nothing of the double cosine
                    // is held in registers by the path above
#pragma unroll 1
                    for (int e = 0; e < EPW; e++) {
                        const bool next = STRADDLE && col + e >= dim;
                        const int j = next ? col + e - dim : col + e;
                        const double x = fma(static_cast<double>(omega[j]), static_cast<double>(next ? d1 : d0),
                                             static_cast<double>(phi[j]));
                        if (fabs(x) < kFarRad) continue;
                        const float r = static_cast<float>(cos(x));
#pragma unroll
                        for (int i = 0; i < EPW; i++) v[i] = i == e ? r : v[i];
                    }
                }
                if constexpr (STRADDLE) {
#pragma unroll
                    for (int e = 0; e < EPW; e++)
                        if (col + e >= dim ? pad1 : pad0) v[e] = 0.0f;
                }
            }
            if (STRADDLE && o == o_last && elems % EPW != 0) {          // the last word, cut short
#pragma unroll
                for (int e = 0; e < EPW; e++) {
                    if (e >= static_cast<int>(elems % EPW)) continue;
                    if constexpr (OUT == TGL_OUT_F32) reinterpret_cast<float *>(o)[e] = v[e];
                    else reinterpret_cast<uint16_t *>(o)[e] = to_bf16(v[e]);
                }
            } else {
                i32x4 word;
                if constexpr (OUT == TGL_OUT_F32) {
                    word = i32x4{__float_as_int(v[0]), __float_as_int(v[1]), __float_as_int(v[2]), __float_as_int(v[3])};
                } else {
                    word = i32x4{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
                }
                __builtin_nontemporal_store(word, o);
            }
        }
        left -= kAhead;
        if (left <= 0) break;
        now = next;
    }
}

// timeenc_kernel strides over its rows, so a grid of the blocks the device
// holds at once does all of them and loads each block's factors once.  Found
// once per device and kernel (CUs x resident blocks per CU).
constexpr int kMaxDevices = 64;
constexpr int kVariants = 4;                                       // output x factor table
std::atomic<int> g_resident[kMaxDevices][kVariants];

template <typename K>
unsigned resident_grid(K kernel, int variant, int64_t want) {
    int dev = 0;
    int r = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
        r = g_resident[dev][variant].load(std::memory_order_relaxed);
        if (r == 0) {
            int cus = 0, per_cu = 0;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) == hipSuccess && cus > 0 &&
                per_cu > 0) {
                r = cus * per_cu;
                g_resident[dev][variant].store(r, std::memory_order_relaxed);
            }
        }
    }
    (void)hipGetLastError();
    if (r <= 0) r = 1 << 16;
    return static_cast<unsigned>(want < r ? want : r);
}

int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }

// Words per lane, which make its setup (two divisions, its columns' factors)
// small: 100 float32 of 600,000 slots take 60 us with 4 and 50 with 8; of 18,000
// slots 6 with 8 and 8 with 16.  And blocks at most, so that a call for many slots
// of which the device counts few does not wait for empty blocks (20M slots, 2,000
// of them valid: 6, 9 and 16 us on 4096, 8192 and 16384 blocks, 100 on as many as
// there are words for).  Full calls on 4096 / 8192 / 16384 / 25600 blocks: 100
// float32 of 8M slots 662 / 599 / 580 / 592 us, 172 of 2M 271 / 252 / 260 / 273,
// 128 of 2M 269 / 237 / 198 / 209; bfloat16 on 4096 / 6144 / 8192 / 25600: 100 of
// 8M 499 / 500 / 507 / 551, 128 of 2M 134 / 140 / 147 / 259, 100 of 64M 3998 / 3964
// / 3943 / 3931.
constexpr int kLaneWordsF32 = 8;
constexpr int kLaneWordsBf16 = 4;
constexpr uint32_t kMostF32 = 16384;
constexpr uint32_t kMostBf16 = 6144;

template <typename K>
void launch_words(K kernel, int epw, int unit, hipStream_t st, const float *dt, int64_t n, const int64_t *count,
                  int64_t per, const float *omega, const float *phi, int dim, void *out) {
    const int64_t words = n > INT64_MAX / dim - epw ? INT64_MAX / epw : (n * dim + epw - 1) / epw;
    const int lane_words = epw == 4 ? kLaneWordsF32 : kLaneWordsBf16;
    const uint32_t most = epw == 4 ? kMostF32 : kMostBf16;
    ScopedTimer tm(TGL_TIMER_TIMEENC, st);
    kernel<<<word_blocks(words, lane_words, most, static_cast<uint32_t>(unit)), kBlock, 0, st>>>(
        dt, n, count, per, omega, phi, dim, lane_words, most, static_cast<uint32_t>(unit), out);
}

template <typename K>
void launch_resident(K kernel, int variant, int64_t want, hipStream_t st, const float *dt, int64_t n,
                     const int64_t *count, int64_t per, const float *omega, const float *phi, int dim, void *out) {
    const unsigned nb = resident_grid(kernel, variant, want);
    ScopedTimer tm(TGL_TIMER_TIMEENC, st);
    kernel<<<nb, kBlock, 0, st>>>(dt, n, count, per, omega, phi, dim, out);
}

}  // namespace
}  // namespace tgl

using namespace tgl;

extern "C" {

tgl_status tgl_time_encode(const float *dt, int64_t n, const int64_t *count, int64_t per_count,
                           const float *omega, const float *phi, int32_t dim, int32_t out_type,
                           void *out, void *stream) {
    if (n < 0 || per_count < 1 || dim < 1 || dim > TGL_MAX_TIME_DIM) return TGL_EINVAL;
    if (out_type != TGL_OUT_F32 && out_type != TGL_OUT_BF16) return TGL_EINVAL;
    if (!omega || !phi) return TGL_EINVAL;
    if (n > 0 && (!dt || !out)) return TGL_EINVAL;
    if ((reinterpret_cast<uintptr_t>(out) & 3u) != 0) return TGL_EINVAL;
    if (n > INT64_MAX / dim) return TGL_EINVAL;
    if (n == 0) return TGL_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    const int esize = out_type == TGL_OUT_F32 ? 4 : 2;
    const bool pre = dim <= kMaxPre;                      // per-column factors staged in LDS
    const int epw = 16 / esize;
    // words by lanes with columns of their own: T * epw, T the lanes of the
    // grid, has to be a multiple of dim, i.e. the blocks one of `unit`
    const int unit = dim / gcd(dim, kBlock * epw);
    if ((reinterpret_cast<uintptr_t>(out) & 15u) == 0 && dim >= epw) {
        const bool straddle = dim % epw != 0;
        if (out_type == TGL_OUT_F32 && straddle)
            launch_words(timeenc_word_kernel<TGL_OUT_F32, true>, epw, unit, st, dt, n, count, per_count, omega, phi, dim, out);
        else if (out_type == TGL_OUT_F32)
            launch_words(timeenc_word_kernel<TGL_OUT_F32, false>, epw, unit, st, dt, n, count, per_count, omega, phi, dim, out);
        else if (straddle)
            launch_words(timeenc_word_kernel<TGL_OUT_BF16, true>, epw, unit, st, dt, n, count, per_count, omega, phi, dim, out);
        else
            launch_words(timeenc_word_kernel<TGL_OUT_BF16, false>, epw, unit, st, dt, n, count, per_count, omega, phi, dim, out);
        return launch_status();
    }
    constexpr int64_t rows_per_block = static_cast<int64_t>(kBlock / kWave) * kRows;
    const int64_t want = (n + rows_per_block - 1) / rows_per_block;
    if (out_type == TGL_OUT_F32) {
        if (pre) launch_resident(timeenc_kernel<TGL_OUT_F32, true>, 0, want, st, dt, n, count, per_count, omega, phi, dim, out);
        else launch_resident(timeenc_kernel<TGL_OUT_F32, false>, 1, want, st, dt, n, count, per_count, omega, phi, dim, out);
    } else {
        if (pre) launch_resident(timeenc_kernel<TGL_OUT_BF16, true>, 2, want, st, dt, n, count, per_count, omega, phi, dim, out);
        else launch_resident(timeenc_kernel<TGL_OUT_BF16, false>, 3, want, st, dt, n, count, per_count, omega, phi, dim, out);
    }
    return launch_status();
}

}  // extern "C"
