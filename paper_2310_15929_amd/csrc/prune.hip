// Offline pruning stage on the GPU: channel statistics (Section 3.2, eq. 1-2), pruning metric
// (eq. 3), global naive shuffle and local block shuffle (Section 3.3, Algorithm 1), n:m mask.
//
// Everything that decides an integer (a bin, a rank, an exchange, a kept position) is computed so
// that the result does not depend on the order in which threads run:
//   - histogram counts, minima and maxima are integer / ordered-integer atomics;
//   - sums of squares and column sums of |w| are accumulated EXACTLY: every term is split by its
//     binary exponent into one of a few 64-bit integer accumulators (16 exponents per accumulator),
//     which are added exactly and rounded once;
//   - the retained metric of a candidate group is summed over the output rows in a FIXED order (interleaved
//     sub-sums, see k_lbs_eval) in float64 without contraction, so repeated runs make the
//     same exchanges; eq. (5) fixes no order for that sum, and the exchanges Algorithm 1 makes do not
//     hinge on it where candidates are not tied to the last bit (the tests compare them with a plain
//     ascending-row sum);
//   - logarithms are the host's (square roots are correctly rounded anywhere); the rank of a channel mean is a count of
//     comparisons.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <thread>

#include "common.h"

// ------------------------------------------------------------------------------------------------
// exact exponent-binned accumulation
// ------------------------------------------------------------------------------------------------
// squares of 16-bit values: exponent in [-266, 255], at most 22 significant bits
#define SQ_NB 33
#define SQ_EOFF 272
#define SQ_SIG 21
// |w| = m 2^e with an integer m of at most 11 bits and e in [-133, 120]: bin b counts units of 2^(16 b - AB_OFF)
#define AB_NB 17
#define AB_OFF 144

// value = sum_b bins[b] 2^(16 b - off), bins[b] < 2^63: exact, then one round-to-nearest-even to double
template <int NB>
__device__ double exact_bins_to_double(const unsigned long long* __restrict__ bins, int off) {
  constexpr int ND = NB + 3;  // digits of 16 bits
  uint16_t d[ND];
  unsigned long long carry = 0;  // < 2^48
#pragma unroll
  for (int i = 0; i < ND; i++) {
    if (i < NB) carry += bins[i];
    d[i] = (uint16_t)carry;
    carry >>= 16;
  }
  // the highest digit that is not zero and the four below it, and whether anything is left below those
  int top = -1;
  unsigned long long w = 0;
  uint32_t w4 = 0, below = 0;
#pragma unroll
  for (int i = ND - 1; i >= 0; i--) {
    if (top < 0 && d[i]) top = i;
    const int k = top - i;
    if (top >= 0 && k < 4) w |= (unsigned long long)d[i] << (48 - 16 * k);
    else if (top >= 0 && k == 4) w4 = d[i];
    else if (top >= 0) below |= d[i];
  }
  if (top < 0) return 0.0;
  const int lz = __clzll((long long)w);  // 0 .. 15
  if (lz) w = (w << lz) | (w4 >> (16 - lz));
  below |= (w4 << lz) & 0xffffu;
  // w: the 64 highest bits, the highest at position 16 top + 15 - lz
  unsigned long long mant = w >> 11;
  const uint32_t rest = (uint32_t)w & 0x7ffu;
  if (rest > 0x400u || (rest == 0x400u && (below || (mant & 1ull)))) mant++;
  return ldexp((double)mant, 16 * top + 15 - lz - 52 - off);
}

// the same value, but nothing that is formed from it is moved ahead of this place (kept in registers through a loop whose body needs them all)
__device__ __forceinline__ int opaque(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
  return v;
}

__device__ __forceinline__ unsigned int ordered_bits(float f) {
  unsigned int u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ------------------------------------------------------------------------------------------------
// Channel statistics in two scans of the calibration features, each at memory speed.
// Both kernels: block 1024 = 32 column lanes of CPL channels (CPL = 4: 8-byte loads, needs K % 4 == 0;
// CPL = 2 otherwise) x 32 row lanes, eight rows in flight per thread; grid (ceil(K / (32 CPL)), row chunks).
//
// Scan A: per-channel min / max and the exact sum of squares.  A 16-bit value is m * 2^E with an integer m of
// at most 11 bits, so its square is the integer m * m at binary position 2 E: bin and quotient of the exponent-
// binned accumulation come from integer shifts (no float64 arithmetic, no ilogb / ldexp).
// Scan B: the histogram over [min, max].  The bin of x is floor(((x - lo) * bins) / (hi - lo)) evaluated in
// float64, clamped to bins - 1 (the definition).  A float32 estimate q of that quotient is at most 1.8e-7 bins off
// (three roundings of 2^-24 relative), the float64 quotient at most 2^-44: whenever q is farther
// than 2.1e-7 bins + 1e-6 from the nearest integer both have the same floor, so only the lanes near a bin edge (and the lanes
// where the estimate overflowed) evaluate the definition itself.  (Some lane of a wave is that near in one trip of 256 rows in twelve
// for 100 bins; with 1e-4 for any number of bins it was one in three.)
// ------------------------------------------------------------------------------------------------
// bin and quotient of the square of a 16-bit value for the exponent-binned exact accumulation, from the bits of the
// (exact) floating-point square: fp16 squares have at most 22 significant bits and fit float32, bf16 squares have 16
// and fit float64 (their exponents go beyond float32).  With t = ilogb(x^2) + SQ_EOFF the bin is t / 16 and the
// quotient x^2 / 2^(16 bin - SQ_EOFF - SQ_SIG) is the square's integer significand shifted left by t % 16 (less than
// 2^37).  Zero gives quotient 0.
template <int DT>
__device__ __forceinline__ void square_bin(float x, unsigned int* bin, unsigned long long* q) {
  if (DT == ESPARSE_F16) {
    const float xs = x * x;
    const uint32_t bits = __float_as_uint(xs);
    const uint32_t t = (bits >> 23) + (uint32_t)(SQ_EOFF - 127);
    uint32_t mant = ((bits & 0x7fffffu) | 0x800000u) >> 2;  // 24-bit significand, its two low bits are zero: SQ_SIG + 1 = 22 bits
    mant = bits ? mant : 0u;
    *bin = t >> 4;
    *q = (unsigned long long)mant << (t & 15u);
  } else {
    const double xs = (double)x * (double)x;
    const uint32_t hi = (uint32_t)(__double_as_longlong(xs) >> 32);  // the low word of the significand is zero
    const uint32_t t = (hi >> 20) + (uint32_t)(SQ_EOFF - 1023);
    uint32_t mant = (hi & 0xfffffu) | 0x100000u;  // top 21 bits of the significand
    mant = hi ? mant : 0u;
    *bin = t >> 4;
    *q = (unsigned long long)mant << ((t & 15u) + 1u);
  }
}

// the 16-bit values of ROWS rows (32 rows apart) x CPL channels of one thread; FULL: all rows exist, else rows past the
// end are replaced by the thread's first row (callers give those no weight)
template <int CPL, int ROWS, bool FULL>
__device__ __forceinline__ void load_rows(const uint16_t* __restrict__ p, long long stride32, long long rb, long long r1,
                                          uint32_t (&w)[ROWS][CPL / 2]) {
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    const uint16_t* src = (FULL || rb + 32 * u < r1) ? p + u * stride32 : p;
    if (CPL == 4) {
      const uint2 v = *reinterpret_cast<const uint2*>(src);
      w[u][0] = v.x;
      w[u][1 % (CPL / 2)] = v.y;
    } else {
      w[u][0] = *reinterpret_cast<const uint32_t*>(src);
    }
  }
}

// Exact sum of squares of one channel in a lane, fp16: a square is a multiple of 2^-48 below 2^32 and fits float32.  It is split in
// float64 at 2^-12 (adding and subtracting 1.5 2^40 rounds to a multiple of that), both parts are added up exactly: SQ_ROWS of
// them are below 2^51 and 2^43 units.  Eight instructions per value and none of them to the LDS; by exponent into LDS bins, as
// bf16 squares go, it takes about 14 and an LDS atomic.
#define SQ_ROWS 128
struct SquareSum {
  double hi, lo;
};
__device__ __forceinline__ void square_add(SquareSum& a, float x) {
  const double s = (double)(x * x), c = 0x1.8p40;
  const double h = (s + c) - c;
  a.hi = a.hi + h;
  a.lo = a.lo + (s - h);
}
// into the channel's bins: units of 2^-48 are bit 245 = 16 15 + 5, units of 2^-12 bit 281 = 16 17 + 9
__device__ __forceinline__ void square_flush(SquareSum& a, unsigned long long* bins) {
  static_assert(SQ_EOFF + SQ_SIG == 293, "the places of the two units");
  // whole numbers below 2^43 and 2^51, read out of the significand of a sum (conversions to 64-bit integers take ten times as long); the parts
  // below 2^-12 may add up to less than zero
  const long long l = __double_as_longlong(__builtin_fma(a.lo, 0x1p48, 0x1.8p52)) - __double_as_longlong(0x1.8p52);
  const unsigned long long h = (unsigned long long)(__double_as_longlong(__builtin_fma(a.hi, 0x1p12, 0x1p52)) - __double_as_longlong(0x1p52) + (l >> 36));
  atomicAdd(bins + 15, (unsigned long long)(l & 0xfffffffffll) << 5);
  atomicAdd(bins + 17, (h & 0xffffffffull) << 9);
  if (h >> 32) atomicAdd(bins + 19, (h >> 32) << 9);
  a = SquareSum{0.0, 0.0};
}

template <int DT, int CPL, int ROWS, bool FULL>
__device__ __forceinline__ void minmax_sumsq_trip(const uint16_t* __restrict__ p, long long stride32, long long rb, long long r1,
                                                  float (&lo)[CPL], float (&hi)[CPL], SquareSum (&sum)[CPL], unsigned long long* s_sq_lane, int want_sq) {
  uint32_t w[ROWS][CPL / 2];
  load_rows<CPL, ROWS, FULL>(p, stride32, rb, r1, w);
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    // a repeated row changes neither min nor max; its square is replaced by zero (no branches in this loop)
    const bool live = FULL || rb + 32 * u < r1;
#pragma unroll
    for (int j = 0; j < CPL; j++) {
      const float x = esp_to_float<DT>((uint16_t)(w[u][j / 2] >> (16 * (j & 1))));
      lo[j] = fminf(lo[j], x);
      hi[j] = fmaxf(hi[j], x);
      if (want_sq && DT == ESPARSE_F16) {
        square_add(sum[j], live ? x : 0.0f);
      } else if (want_sq) {
        unsigned int bi;
        unsigned long long q;
        square_bin<DT>(live ? x : 0.0f, &bi, &q);
        atomicAdd(s_sq_lane + j * (32 * SQ_NB) + bi, q);
      }
    }
  }
}

template <int DT, int CPL>
__global__ void __launch_bounds__(1024, 8) k_minmax_sumsq(const uint16_t* __restrict__ X, long long T, long long K,
                                                        long long rows_per_block, unsigned int* __restrict__ onmin /*~minimum*/,
                                                        unsigned int* __restrict__ omax,
                                                        unsigned long long* __restrict__ sq /*[K][SQ_NB]*/, int want_sq) {
  constexpr int CH = 32 * CPL;  // channels per block
  // LDS row of a channel = j * 32 + cl (cl: column lane, j: which of the lane's CPL channels)
  __shared__ unsigned long long s_sq[CH * SQ_NB];
  __shared__ unsigned int s_lo[CH], s_hi[CH];
  const int tid = threadIdx.x, cl = tid & 31, rl = tid >> 5;
  for (int i = tid; i < CH * SQ_NB; i += 1024) s_sq[i] = 0ull;
  if (tid < CH) {
    s_lo[tid] = 0xffffffffu;
    s_hi[tid] = 0u;
  }
  __syncthreads();
  const long long c = ((long long)blockIdx.x * 32 + cl) * CPL;
  const long long r0 = (long long)blockIdx.y * rows_per_block;
  const long long r1 = r0 + rows_per_block < T ? r0 + rows_per_block : T;
  if (c < K && r0 + rl < r1) {
    float lo[CPL], hi[CPL];
#pragma unroll
    for (int j = 0; j < CPL; j++) {
      lo[j] = INFINITY;
      hi[j] = -INFINITY;
    }
    constexpr int ROWS = 8;
    const long long stride32 = 32 * K;
    const uint16_t* p = X + (r0 + rl) * K + c;
    unsigned long long* s_sq_lane = s_sq + cl * SQ_NB;
    SquareSum sum[CPL];
#pragma unroll
    for (int j = 0; j < CPL; j++) sum[j] = SquareSum{0.0, 0.0};
    auto flush = [&]() {
      if (want_sq && DT == ESPARSE_F16)
#pragma unroll
        for (int j = 0; j < CPL; j++) square_flush(sum[j], s_sq_lane + j * (32 * SQ_NB));
    };
    long long rb = r0 + rl;
    for (int trips = 0; rb + 32 * (ROWS - 1) < r1; rb += 32 * ROWS, p += ROWS * stride32) {
      minmax_sumsq_trip<DT, CPL, ROWS, true>(p, stride32, rb, r1, lo, hi, sum, s_sq_lane, want_sq);
      if (++trips % (SQ_ROWS / ROWS) == 0) flush();
    }
    if (rb < r1) minmax_sumsq_trip<DT, CPL, ROWS, false>(p, stride32, rb, r1, lo, hi, sum, s_sq_lane, want_sq);
    flush();
#pragma unroll
    for (int j = 0; j < CPL; j++) {
      atomicMin(&s_lo[j * 32 + cl], ordered_bits(lo[j]));
      atomicMax(&s_hi[j * 32 + cl], ordered_bits(hi[j]));
    }
  }
  __syncthreads();
  const long long cbase = (long long)blockIdx.x * CH;
  if (tid < CH && r0 < r1) {
    const long long ch = cbase + (long long)(tid & 31) * CPL + (tid >> 5);  // LDS row tid = j * 32 + cl
    if (ch < K) {
      atomicMax(&onmin[ch], ~s_lo[tid]);  // so that both start from zero
      atomicMax(&omax[ch], s_hi[tid]);
    }
  }
  if (want_sq)
    for (int i = tid; i < CH * SQ_NB; i += 1024) {
      const int row = i / SQ_NB;
      const long long ch = cbase + (long long)(row & 31) * CPL + (row >> 5);
      const unsigned long long v = s_sq[i];
      if (ch < K && v) atomicAdd(&sq[ch * SQ_NB + (i % SQ_NB)], v);
    }
}

__device__ __forceinline__ float float_from_ordered_bits(unsigned int o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

__device__ __forceinline__ float fraction_of(float q) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_fractf(q);
#else
  return q - floorf(q);
#endif
}

// x - lo of a 16-bit value (one v_fma_mix_f32 for fp16: `one` is 1.0 in a register the compiler cannot see into)
template <int DT>
__device__ __forceinline__ float offset_of(uint16_t raw, float lo32, float one) {
  if (DT == ESPARSE_F16) return __builtin_fmaf(esp_to_float<DT>(raw), one, -lo32);
  return esp_to_float<DT>(raw) - lo32;
}

// An estimate q can be trusted if it is farther than `edge` from both neighbouring integers and, where it may overflow (bf16), below
// `bins`.  Else the value is looked at in float64.  These are not as rare as `edge` makes them: 16-bit values stand on bin edges
// (one in a thousand on a few of them per channel), so a wave meets some in most trips, and they are settled on the spot, between the
// others; done after all others, with the estimates of the trip formed again, they cost 470 - 397 us.
template <int DT, int CPL, int ROWS, bool FULL>
__device__ __forceinline__ void hist_trip(const uint16_t* __restrict__ p, long long stride32, long long rb, long long r1,
                                          const float (&lo32)[CPL], const float (&c32)[CPL], const double (&lo)[CPL],
                                          const double (&wd)[CPL], int bins, float one, float edge, unsigned int* s_hist_lane, int stride) {
  uint32_t w[ROWS][CPL / 2];
  load_rows<CPL, ROWS, FULL>(p, stride32, rb, r1, w);
  const float safe = 0.5f - edge, nb32 = (float)bins;
  const double nb = (double)bins;
#pragma unroll
  for (int u = 0; u < ROWS; u++) {
    const unsigned int add = (FULL || rb + 32 * u < r1) ? 1u : 0u;  // a repeated row counts nothing
#pragma unroll
    for (int j = 0; j < CPL; j++) {
      const uint16_t raw = (uint16_t)(w[u][j / 2] >> (16 * (j & 1)));
      const float q = offset_of<DT>(raw, lo32[j], one) * c32[j];
      unsigned int b = (unsigned int)(int)q;
      if (!(fabsf(fraction_of(q) - 0.5f) <= safe) || (DT != ESPARSE_F16 && !(q < nb32))) {
        const double t = ((double)esp_to_float<DT>(raw) - lo[j]) * nb;
        if (DT == ESPARSE_F16) {
          // t and multiples of the width are exact (at most 49 bits), and a quotient that is not an integer is at least 2^-41 away from
          // one: floor(t / wd) is the nearest integer e to q, or e - 1 where t < e wd
          const float e = rintf(q);
          b = (unsigned int)((int)e - (__builtin_fma(-(double)e, wd[j], t) < 0.0 ? 1 : 0));
        } else {
          b = wd[j] > 0.0 ? (unsigned int)(int)floor(t / wd[j]) : 0u;  // the definition
        }
      }
      atomicAdd(s_hist_lane + j * (32 * stride) + min(b, (unsigned int)bins - 1u), add);
    }
  }
}

template <int DT, int CPL>
__global__ void __launch_bounds__(1024, 8) k_hist(const uint16_t* __restrict__ X, long long T, long long K,
                                                long long rows_per_block, int bins, const unsigned int* __restrict__ onmin,
                                                const unsigned int* __restrict__ omax, unsigned int* __restrict__ hist /*[K][bins]*/,
                                                unsigned int* __restrict__ most /*[gridDim.x] no count of these channels is larger*/) {
  constexpr int CH = 32 * CPL;
  __shared__ unsigned int s_most;
  // [CH rows][stride]: the row of a channel is j * 32 + cl (cl: column lane, j: which of the lane's CPL channels), the stride odd, so that the column
  // lanes of one instruction start in 32 different banks.  A column lane always in its own bank ([j][bins][cl]) is no faster in the loop (T = 262144,
  // K = 4096 408 us, 100 bins; 500 us, 256 bins; this 394 and 430), and its bins go out in short pieces: T = 131072, K = 232 97 and 186 us, this 52 and 91
  extern __shared__ unsigned int s_hist[];
  const int stride = bins | 1;
  const int tid = threadIdx.x, cl = tid & 31, rl = tid >> 5;
  for (int i = tid; i < CH * stride; i += 1024) s_hist[i] = 0u;
  if (tid == 0) s_most = 0u;
  __syncthreads();
  const long long c = ((long long)blockIdx.x * 32 + cl) * CPL;
  const long long r0 = (long long)blockIdx.y * rows_per_block;
  const long long r1 = r0 + rows_per_block < T ? r0 + rows_per_block : T;
  if (c < K && r0 + rl < r1) {
    float lo32[CPL], c32[CPL];
    double lo[CPL], wd[CPL];
    const double nb = (double)bins;
#pragma unroll
    for (int j = 0; j < CPL; j++) {
      lo32[j] = float_from_ordered_bits(~onmin[c + j]);
      lo[j] = (double)lo32[j];
      wd[j] = (double)float_from_ordered_bits(omax[c + j]) - lo[j];
      // the estimate's factor; a constant channel (width 0) gets 0: every value in bin 0
      c32[j] = wd[j] > 0.0 ? (float)(nb / wd[j]) : 0.0f;
    }
    const float one = __int_as_float(opaque(0x3f800000)), edge = (float)bins * 2.1e-7f + 1e-6f;
    constexpr int ROWS = 8;
    const long long stride32 = 32 * K;
    const uint16_t* p = X + (r0 + rl) * K + c;
    unsigned int* s_hist_lane = s_hist + cl * stride;
    long long rb = r0 + rl;
    for (; rb + 32 * (ROWS - 1) < r1; rb += 32 * ROWS, p += ROWS * stride32)
      hist_trip<DT, CPL, ROWS, true>(p, stride32, rb, r1, lo32, c32, lo, wd, bins, one, edge, s_hist_lane, stride);
    if (rb < r1) hist_trip<DT, CPL, ROWS, false>(p, stride32, rb, r1, lo32, c32, lo, wd, bins, one, edge, s_hist_lane, stride);
  }
  __syncthreads();
  const long long cbase = (long long)blockIdx.x * CH;
  // a wave takes as many channels as 64 lanes hold the bins of, one at least: runs of up to 256 bytes (always one channel: 229598 tokens of 84 channels, 2 bins,
  // a call 231 us, this 120)
  unsigned int mine = 0u;
  const int each = bins < 64 ? 64 / bins : 1;
  for (int g = tid >> 6; g < (CH + each - 1) / each; g += 16)
    for (int i = tid & 63; i < each * bins; i += 64) {
      const int c_in = i / bins, ch = g * each + c_in;
      if (ch >= CH || cbase + ch >= K) break;
      const unsigned int v = s_hist[(ch % CPL * 32 + ch / CPL) * stride + (i - c_in * bins)];
      if (v) atomicAdd(&hist[(cbase + g * each) * bins + i], v);
      mine = v > mine ? v : mine;
    }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned int other = __shfl_xor(mine, d);
    mine = other > mine ? other : mine;
  }
  if ((tid & 63) == 0) atomicMax(&s_most, mine);
  __syncthreads();
  if (tid == 0) atomicAdd(&most[blockIdx.x], s_most);  // the workgroups' largest counts, added up
}

// ------------------------------------------------------------------------------------------------
// exact column sums of |W|: grid (ceil(K / 128), row chunks), block 256 = 8 row lanes x 32 lanes of four channels (8-byte
// loads, eight rows in flight).  fp16: a lane adds its rows as integers of 2^-24 (less than 2^40 each); bf16: by exponent
// into LDS.  4096 x 4096: 25 -> 12 us, fp16 (one float64 ilogb and ldexp per element and 4-byte loads before).  A NaN adds
// nothing; an infinity adds the power of two that follows the type's largest value.
// ------------------------------------------------------------------------------------------------
template <int DT>
__global__ void __launch_bounds__(256) k_abs_colsum(const uint16_t* __restrict__ W, long long N, long long K,
                                                     long long rows_per_block, unsigned long long* __restrict__ out /*[K][AB_NB]*/) {
  __shared__ unsigned long long s_acc[128 * AB_NB];  // channel j of lane cl: row j * 32 + cl
  const int tid = threadIdx.x;
  for (int i = tid; i < 128 * AB_NB; i += 256) s_acc[i] = 0ull;
  __syncthreads();
  const int cl = tid & 31, rl = tid >> 5;
  const long long c = (long long)blockIdx.x * 128 + cl * 4;
  if (c < K) {
    const long long r0 = (long long)blockIdx.y * rows_per_block;
    const long long r1 = r0 + rows_per_block < N ? r0 + rows_per_block : N;
    unsigned long long sum[4] = {0ull, 0ull, 0ull, 0ull};
    auto add = [&](uint2 v) {
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const uint32_t raw = ((j < 2 ? v.x : v.y) >> (16 * (j & 1))) & 0x7fffu;
        if (DT == ESPARSE_F16) {
          const uint32_t e = raw >> 10;
          uint32_t m = e ? (raw & 0x3ffu) | 0x400u : raw;
          m = raw > 0x7c00u ? 0u : m;
          sum[j] += (unsigned long long)m << (e ? e - 1 : 0);
        } else {
          const uint32_t e = raw >> 7;
          const uint32_t m = e ? (raw & 0x7fu) | 0x80u : raw;
          const uint32_t pos = (e ? e : 1u) + (AB_OFF - 134);
          if (m && raw <= 0x7f80u) atomicAdd(&s_acc[(j * 32 + cl) * AB_NB + (pos >> 4)], (unsigned long long)m << (pos & 15u));
        }
      }
    };
    const uint16_t* p = W + (r0 + rl) * K + c;
    long long r = r0 + rl;
    for (; r + 56 < r1; r += 64, p += 64 * K) {
      uint2 v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = *reinterpret_cast<const uint2*>(p + u * 8 * K);
#pragma unroll
      for (int u = 0; u < 8; u++) add(v[u]);
    }
    for (; r < r1; r += 8, p += 8 * K) add(*reinterpret_cast<const uint2*>(p));
    if (DT == ESPARSE_F16) {
#pragma unroll
      for (int j = 0; j < 4; j++) {  // units of 2^-24 = bit 120: bin 7, 8 bits up; the upper half 32 bits higher
        unsigned long long* acc = &s_acc[(j * 32 + cl) * AB_NB];
        atomicAdd(acc + (AB_OFF - 24) / 16, (sum[j] & 0xffffffffull) << ((AB_OFF - 24) % 16));
        if (sum[j] >> 32) atomicAdd(acc + (AB_OFF - 24) / 16 + 2, (sum[j] >> 32) << ((AB_OFF - 24) % 16));
      }
    }
  }
  __syncthreads();
  const long long cbase = (long long)blockIdx.x * 128;
  for (int i = tid; i < 128 * AB_NB; i += 256) {
    const int row = i / AB_NB;
    const long long ch = cbase + (row & 31) * 4 + (row >> 5);
    const unsigned long long v = s_acc[i];
    if (ch < K && v) atomicAdd(&out[ch * AB_NB + (i % AB_NB)], v);
  }
}

// eq. 2: AM_c^2 per channel, rounded once
__global__ void __launch_bounds__(64) k_sumsq_finish(const unsigned long long* __restrict__ sq, long long K, double* __restrict__ out) {
  const long long c = (long long)blockIdx.x * 64 + threadIdx.x;
  if (c < K) out[c] = exact_bins_to_double<SQ_NB>(sq + c * SQ_NB, SQ_EOFF + SQ_SIG);
}

// The terms p ln p of eq. 1 for counts below T, taken on the host (the logarithm that the result is defined by is the host's) while the
// scans run: as many as the counts can be, into device memory.  Gathered from host memory every one would be a trip over the bus.
__global__ void __launch_bounds__(256) k_fetch_terms(const double* __restrict__ host_terms, long long T, const unsigned int* __restrict__ most, int nmost,
                                                      double* __restrict__ terms) {
  __shared__ unsigned int s_most;
  if (threadIdx.x == 0) s_most = 0u;
  __syncthreads();
  unsigned int mine = 0u;
  for (int i = threadIdx.x; i < nmost; i += 256) mine = most[i] > mine ? most[i] : mine;
  atomicMax(&s_most, mine);
  __syncthreads();
  const long long n = (long long)s_most + 1 < T ? (long long)s_most + 1 : T;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) terms[i] = host_terms[i];
}

// eq. 1 and 3: s_c = IR_c + alpha AM_c, each term behind its switch; IR_c adds its terms in ascending order of the bins.
// 16 channels per workgroup: their terms into LDS, then one thread each.
__global__ void __launch_bounds__(256) k_scores(const unsigned int* __restrict__ hist /*[K][bins] or null*/, const double* __restrict__ terms, long long T,
                                                 int bins, const unsigned long long* __restrict__ sq /*or null*/, double alpha, long long K,
                                                 double* __restrict__ out) {
  extern __shared__ double s_term[];  // [16][bins | 1]
  const int tid = threadIdx.x, stride = bins | 1;
  const long long c0 = (long long)blockIdx.x * 16;
  if (hist)
    for (int i = tid; i < 16 * bins; i += 256) {
      const int row = i / bins;
      const unsigned int n = c0 + row < K ? hist[c0 * bins + i] : 0u;
      s_term[row * stride + i - row * bins] = n && n < T ? terms[n] : 0.0;  // an empty bin adds nothing, one with all tokens 1 ln 1
    }
  __syncthreads();
  const long long c = c0 + tid;
  if (tid >= 16 || c >= K) return;
  double v = 0.0;
  if (hist) {
    double acc = 0.0;
#pragma unroll 10
    for (int b = 0; b < bins; b++) acc = acc + s_term[tid * stride + b];
    v = v + -acc;
  }
  if (sq) v = v + alpha * sqrt(exact_bins_to_double<SQ_NB>(sq + c * SQ_NB, SQ_EOFF + SQ_SIG));
  out[c] = v;
}

// channel means of the metric: g_c = (s_c * sum_j |w_jc|) / N
__global__ void __launch_bounds__(64) k_channel_means(const unsigned long long* __restrict__ bins, const double* __restrict__ score, long long N,
                                                       long long K, double* __restrict__ g) {
  const long long c = (long long)blockIdx.x * 64 + threadIdx.x;
  if (c < K) g[c] = (score[c] * exact_bins_to_double<AB_NB>(bins + c * AB_NB, AB_OFF)) / (double)N;
}

// Global naive shuffle: the rank of a channel is the number of channels with a larger mean, or the same and a lower number
// (NaN behind all numbers); rank r goes to position (r mod G) m + r / G.  16 channels per workgroup, the comparisons with
// all others split over 64 lanes each; K^2 comparisons instead of a sort on the host (4096 channels: 22 us against about 400).
// Beyond RANK_ON_DEVICE channels the host sorts (whole prune calls without a block shuffle, 16 rows, sorted / compared: 196608
// channels 14.7 / 16.7 ms, 262144 20 / 29, 524288 44 / 138: the comparisons grow fourfold with each doubling; 131072: 7.6 compared).
#define RANK_ON_DEVICE (3ll << 16)
__global__ void __launch_bounds__(1024) k_naive_shuffle(const double* __restrict__ g, const double* __restrict__ score, int K, int m, int use_gns,
                                                         int32_t* __restrict__ theta0, double* __restrict__ sp) {
  __shared__ int s_rank[16];
  const int tid = threadIdx.x, l = tid & 15, part = tid >> 4;
  if (tid < 16) s_rank[tid] = 0;
  __syncthreads();
  const int c = blockIdx.x * 16 + l;
  if (use_gns) {
    const double mine = c < K ? g[c] : 0.0;
    const bool mine_nan = mine != mine;
    int ahead = 0;
#pragma unroll 8
    for (int q = part; q < K; q += 64) {
      const double other = g[q];
      const bool other_nan = other != other;
      ahead += (other_nan ? (mine_nan && q < c) : (mine_nan || other > mine || (other == mine && q < c))) ? 1 : 0;
    }
    atomicAdd(&s_rank[l], ahead);
  }
  __syncthreads();
  if (part == 0 && c < K) {
    const int G = K / m, r = s_rank[l];
    const int p = use_gns ? (r % G) * m + r / G : c;
    theta0[p] = c;
    sp[p] = score[c];
  }
}

#define ENTROPY_COUNTS 65536  // of a thread of esp_entropies at least
#define ENTROPY_TERMS 4096    // and of entropy_terms
// Threads that share work of the host, which is worth starting one for every `share` of it, and about how long they take (us; starting them is most
// of it).
static inline int host_threads(long long work, long long share) { return (int)std::max<long long>(1, std::min<long long>(8, work / share)); }
static inline double threads_us(double alone, int threads) { return alone / threads + (threads > 1 ? 14.0 * threads - 2.0 : 0.0); }

// eq. 1: IR_c = - sum_k p_k ln p_k, ascending k, empty bins skipped.  K * bins logarithms on the host (the host's log is
// the one the result is defined by); the counts of a channel set repeat, so each thread keeps the terms it has met (a
// logarithm of a count below 16384 is taken about once in ten times at T = 262144).  Without memory for the terms or without
// another thread the work is done all the same.
void esp_entropies(const unsigned int* hist, long long K, int bins, long long T, double* out) {
  const unsigned int known = (unsigned int)std::min<long long>(T + 1, 16384);
  auto entropy_of = [=](long long c0, long long c1) {
    std::unique_ptr<double[]> term(new (std::nothrow) double[known]());  // 0: not met yet (p ln p = 0 for p = 1 only)
    for (long long c = c0; c < c1; c++) {
      double acc = 0.0;
      for (int k = 0; k < bins; k++) {
        const unsigned int nk = hist[(size_t)c * bins + k];
        if (!nk) continue;
        const bool keep = term && nk < known;
        double t = keep ? term[nk] : 0.0;
        if (t == 0.0) {
          const double p = (double)nk / (double)T;
          t = p * std::log(p);
          if (keep) term[nk] = t;
        }
        acc = acc + t;
      }
      out[c] = -acc;
    }
  };
  const int nthr = host_threads(K * bins, ENTROPY_COUNTS);
  std::thread pool[8];
  int started = 1;
  try {
    for (; started < nthr; started++) pool[started] = std::thread(entropy_of, K * started / nthr, K * (started + 1) / nthr);
  } catch (...) {  // no thread to be had: its share and the rest are done here
  }
  entropy_of(0, K / nthr);
  entropy_of(K * started / nthr, K);
  for (int i = 1; i < started; i++) pool[i].join();
}

// ------------------------------------------------------------------------------------------------
// host driver of the statistics
// ------------------------------------------------------------------------------------------------
// what the scans leave on the device: zeroed ahead of them (the minimum is kept inverted)
struct Scans {
  unsigned long long* sq;  // [K][SQ_NB]
  unsigned int *nmin, *max;  // [K] each
  unsigned int* most;        // [nmost]
  double* sums;              // [K], not zeroed
  unsigned int* hist;        // [K][bins], right behind sums
  size_t nmost;
};

static int launch_scans(esparse_ctx* ctx, Scratch& scratch, const void* calib, long long T, long long K, int dtype, int bins, bool want_hist, bool want_sq,
                        Scans* out) {
  hipStream_t st = ctx->stream;
  const int cpl = K % 4 == 0 ? 4 : 2;  // channels per lane: 8-byte loads where the rows allow them
  const long long gx = (K + 32 * cpl - 1) / (32 * cpl);
  const size_t nmost = (size_t)(gx + 1) / 2 * 2;  // keeps what follows aligned to 8 bytes
  const size_t sq_bytes = (size_t)K * SQ_NB * 8, hist_bytes = (size_t)K * bins * 4, all = sq_bytes + (size_t)K * 8 + nmost * 4 + (size_t)K * 8 + hist_bytes;
  unsigned char* d_all = scratch.get<unsigned char>(all);
  if (!d_all) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation for channel statistics failed");
  unsigned long long* d_sq = reinterpret_cast<unsigned long long*>(d_all);
  unsigned int* d_nmin = reinterpret_cast<unsigned int*>(d_all + sq_bytes);
  unsigned int* d_max = d_nmin + K;
  unsigned int* d_most = d_max + K;
  double* d_sums = reinterpret_cast<double*>(d_most + nmost);
  unsigned int* d_hist = reinterpret_cast<unsigned int*>(d_sums + K);
  *out = Scans{d_sq, d_nmin, d_max, d_most, d_sums, d_hist, nmost};
  ESP_HIP(ctx, hipMemsetAsync(d_all, 0, all, st));
  const uint16_t* X = reinterpret_cast<const uint16_t*>(calib);
  // 1024 workgroups, two rounds of the two per CU that fit at once (one more chunk would be a third round), whole trips of 256 rows
  const long long nchunk = std::max<long long>(1, std::min<long long>((T + 255) / 256, 1024 / gx));
  long long rpb = (T + nchunk - 1) / nchunk;
  rpb = (rpb + 255) / 256 * 256;
  dim3 grid((unsigned)gx, (unsigned)((T + rpb - 1) / rpb));
#define ESP_SCAN_A(DTv, CPLv)                                                                                        \
  hipLaunchKernelGGL((k_minmax_sumsq<DTv, CPLv>), grid, dim3(1024), 0, st, X, T, K, rpb, d_nmin, d_max, d_sq, want_sq ? 1 : 0)
#define ESP_SCAN_B(DTv, CPLv)                                                                                        \
  hipLaunchKernelGGL((k_hist<DTv, CPLv>), grid, dim3(1024), (size_t)32 * CPLv * (bins | 1) * 4, st, X, T, K, rpb, bins, d_nmin, d_max, d_hist, d_most)
  if (dtype == ESPARSE_F16) {
    if (cpl == 4) ESP_SCAN_A(ESPARSE_F16, 4);
    else ESP_SCAN_A(ESPARSE_F16, 2);
  } else {
    if (cpl == 4) ESP_SCAN_A(ESPARSE_BF16, 4);
    else ESP_SCAN_A(ESPARSE_BF16, 2);
  }
  ESP_HIP(ctx, hipGetLastError());
  if (want_hist) {
    // 32 * 4 channels x 256 bins x 4 bytes = 128 KiB of LDS at most
    const size_t smem = (size_t)32 * cpl * (bins | 1) * 4;
    if (smem > 48 * 1024) {
      ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<ESPARSE_F16, 4>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
      ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<ESPARSE_BF16, 4>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
      ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<ESPARSE_F16, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
      ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<ESPARSE_BF16, 2>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    }
    if (dtype == ESPARSE_F16) {
      if (cpl == 4) ESP_SCAN_B(ESPARSE_F16, 4);
      else ESP_SCAN_B(ESPARSE_F16, 2);
    } else {
      if (cpl == 4) ESP_SCAN_B(ESPARSE_BF16, 4);
      else ESP_SCAN_B(ESPARSE_BF16, 2);
    }
    ESP_HIP(ctx, hipGetLastError());
  }
#undef ESP_SCAN_A
#undef ESP_SCAN_B
  return ESPARSE_OK;
}

int esp_stats_device(esparse_ctx* ctx, const void* calib, long long T, long long K, int dtype, int bins,
                     std::vector<double>* ir, std::vector<double>* am) {
  if (!ir && !am) return ESPARSE_OK;
  hipStream_t st = ctx->stream;
  std::vector<unsigned char> pageable;
  Scratch scratch(ctx);
  // what goes to the host: sums of squares, histogram
  const size_t out_bytes = (size_t)K * 8 + (ir ? (size_t)K * bins * 4 : 0);
  unsigned char* h_out = reinterpret_cast<unsigned char*>(esp_host_stage(ctx, out_bytes));
  if (!h_out) {
    pageable.resize(out_bytes);
    h_out = pageable.data();
  }
  Scans sc;
  const int rc = launch_scans(ctx, scratch, calib, T, K, dtype, bins, ir != nullptr, am != nullptr, &sc);
  if (rc) return rc;
  if (am) {
    hipLaunchKernelGGL(k_sumsq_finish, dim3((unsigned)((K + 63) / 64)), dim3(64), 0, st, sc.sq, K, sc.sums);
    ESP_HIP(ctx, hipGetLastError());
  }
  ESP_HIP(ctx, hipMemcpyAsync(h_out, sc.sums, out_bytes, hipMemcpyDeviceToHost, st));
  ESP_HIP(ctx, hipStreamSynchronize(st));
  scratch.idle();
  if (am) {
    // eq. 2: AM_c = sqrt(exact sum of squares rounded once)
    const double* sums = reinterpret_cast<const double*>(h_out);
    am->assign((size_t)K, 0.0);
    for (long long c = 0; c < K; c++) (*am)[c] = std::sqrt(sums[c]);
  }
  if (ir) {
    ir->assign((size_t)K, 0.0);
    esp_entropies(reinterpret_cast<const unsigned int*>(h_out + (size_t)K * 8), K, bins, T, ir->data());
  }
  return ESPARSE_OK;
}

// terms[n] = p ln p of a count n of T, for n < T (0 for 0); by several threads, without them by this one
static void entropy_terms(long long T, double* terms) {
  auto fill = [=](long long n0, long long n1) {
    for (long long n = n0; n < n1; n++) {
      const double p = (double)n / (double)T;
      terms[n] = n ? p * std::log(p) : 0.0;
    }
  };
  const int nthr = host_threads(T, ENTROPY_TERMS);
  std::thread pool[8];
  int started = 1;
  try {
    for (; started < nthr; started++) pool[started] = std::thread(fill, T * started / nthr, T * (started + 1) / nthr);
  } catch (...) {  // no thread to be had: its share and the rest are done here
  }
  fill(0, T / nthr);
  fill(T * started / nthr, T);
  for (int i = 1; i < started; i++) pool[i].join();
}

// The scores of eq. 3 on the device, without a look from the host: terms (T of them, pinned) are taken while the scans run.
static int launch_scores(esparse_ctx* ctx, Scratch& scratch, const EspCalib& in, long long K, int dtype, double* h_terms, double* d_score) {
  hipStream_t st = ctx->stream;
  Scans sc;
  const int rc = launch_scans(ctx, scratch, in.calib, in.T, K, dtype, in.bins, in.entropy, in.norm, &sc);
  if (rc) return rc;
  double* d_terms = nullptr;
  if (in.entropy) {
    d_terms = scratch.get<double>((size_t)in.T);
    if (!d_terms) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation for channel statistics failed");
    entropy_terms(in.T, h_terms);
    hipLaunchKernelGGL(k_fetch_terms, dim3((unsigned)std::min<long long>(256, (in.T + 255) / 256)), dim3(256), 0, st, h_terms, in.T, sc.most, (int)sc.nmost, d_terms);
    ESP_HIP(ctx, hipGetLastError());
  }
  hipLaunchKernelGGL(k_scores, dim3((unsigned)((K + 15) / 16)), dim3(256), in.entropy ? (size_t)16 * (in.bins | 1) * 8 : 0, st, in.entropy ? sc.hist : nullptr, d_terms,
                     in.T, in.bins, in.norm ? sc.sq : nullptr, in.alpha, K, d_score);
  ESP_HIP(ctx, hipGetLastError());
  return ESPARSE_OK;
}

// The same on the host, for any T, K and alpha.
static int scores_on_host(esparse_ctx* ctx, const EspCalib& in, long long K, int dtype, std::vector<double>& s) {
  std::vector<double> ir, am;
  const int rc = esp_stats_device(ctx, in.calib, in.T, K, dtype, in.bins, in.entropy ? &ir : nullptr, in.norm ? &am : nullptr);
  if (rc) return rc;
  s.assign((size_t)K, 0.0);
  for (long long c = 0; c < K; c++) {
    double v = 0.0;
    if (in.entropy) v = v + ir[c];
    if (in.norm) {
      double t = in.alpha * am[c];
      v = v + t;
    }
    s[c] = v;
  }
  return ESPARSE_OK;
}

// ------------------------------------------------------------------------------------------------
// local block shuffle
// ------------------------------------------------------------------------------------------------
// Panel: P[blk][j][c] = |W[j, theta0[blk B + c]]| as raw 16-bit magnitudes: the N x B values of a block are
// contiguous, so that a block's share (512 KiB for N = 4096, B = 64) stays in the L2 of the XCD that works on it, and
// PT[blk][c][j], the same by columns (the members of a group for consecutive rows).  Npad >= N rows per block; what
// lies past N is read but never used and stays as it is.
//
// A workgroup copies RB whole rows into LDS and gathers from there: a gather from global memory goes through the
// vector-memory path one lane at a time (52 us for 4096 x 4096).  RB = 0: rows that do not fit the LDS, gathered from
// global memory, one per workgroup.
__global__ void __launch_bounds__(512) k_build_panel(const uint16_t* __restrict__ W, const int32_t* __restrict__ theta0,
                                                      long long N, long long Npad, long long K, long long first_row, int B, int RB, unsigned int inf_bits,
                                                      const double* __restrict__ sp, uint16_t* __restrict__ P, int* __restrict__ not_finite) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  uint16_t* s_w = reinterpret_cast<uint16_t*>(smem_raw);
  const int tid = threadIdx.x, rows = RB ? RB : 1;
  const long long j0 = first_row + (long long)blockIdx.x * rows;
  const int nr = (int)(N - j0 < rows ? N - j0 : rows);
  if (RB) {
    const uint16_t* src = W + j0 * K;  // the rows are contiguous; K is a multiple of 4 and W of 16 bytes
    const long long n4 = nr * K / 4;
    for (long long e = tid; e < n4; e += 512) reinterpret_cast<uint2*>(s_w)[e] = reinterpret_cast<const uint2*>(src)[e];
    __syncthreads();
  }
  const int q4 = B / 4, nblk = (int)(K / B);  // four columns per thread and step
  bool bad = false;
  if (j0 == 0)  // the scores as well
    for (long long c = tid; c < K; c += 512) bad = bad || !(fabs(sp[c]) < INFINITY);
  for (int e = tid; e < nblk * nr * q4; e += 512) {
    const int c = e % q4, t = e / q4, r = t % nr, blk = t / nr;
    const int4 col = reinterpret_cast<const int4*>(theta0)[blk * q4 + c];
    const uint16_t* row = RB ? s_w + (size_t)r * K : W + j0 * K;
    const unsigned int v0 = row[col.x] & 0x7fffu, v1 = row[col.y] & 0x7fffu, v2 = row[col.z] & 0x7fffu, v3 = row[col.w] & 0x7fffu;
    bad = bad || v0 >= inf_bits || v1 >= inf_bits || v2 >= inf_bits || v3 >= inf_bits;
    reinterpret_cast<uint2*>(P + ((long long)blk * Npad + j0 + r) * B)[c] = uint2{v0 | (v1 << 16), v2 | (v3 << 16)};
  }
  if (bad) atomicOr(not_finite, 1);
}

// 64 rows x 64 columns of a block per workgroup, through LDS
__global__ void __launch_bounds__(256) k_panel_columns(const uint16_t* __restrict__ P, long long Npad, int nblk, int B, uint16_t* __restrict__ PT) {
  __shared__ uint16_t s_t[64 * 66];
  const int tid = threadIdx.x, blk = (int)(blockIdx.x % (unsigned)nblk);
  const long long j0 = (long long)(blockIdx.x / (unsigned)nblk) * 64;
  const int c0 = (int)blockIdx.y * 64, nc = B - c0 < 64 ? B - c0 : 64;
  const int nj = (int)(Npad - j0 < 64 ? Npad - j0 : 64);
  const uint16_t* src = P + ((long long)blk * Npad + j0) * B + c0;
  const int cx = (tid & 31) * 2, ry = tid >> 5;
  for (int r = ry; r < nj; r += 8)
    if (cx < nc) *reinterpret_cast<uint32_t*>(s_t + r * 66 + cx) = *reinterpret_cast<const uint32_t*>(src + (long long)r * B + cx);
  __syncthreads();
  uint16_t* dst = PT + ((long long)blk * B + c0) * Npad + j0;
  for (int c = ry; c < nc; c += 8)
    if (cx < nj) *reinterpret_cast<uint32_t*>(dst + (long long)c * Npad + cx) = s_t[cx * 66 + c] | ((uint32_t)s_t[(cx + 1) * 66 + c] << 16);
}

template <int NKEEP, int MG>
__device__ __forceinline__ double top_n_sum(double* v) {
  // the NKEEP largest of v[0..MG), added largest first
#pragma unroll
  for (int a = 0; a < NKEEP; a++) {
#pragma unroll
    for (int b = MG - 1; b > a; b--) {
      // bubble the maximum of v[a..MG) to v[a]
      double hi = fmax(v[b - 1], v[b]), lo = fmin(v[b - 1], v[b]);
      v[b - 1] = hi;
      v[b] = lo;
    }
  }
  double t = v[0];
#pragma unroll
  for (int a = 1; a < NKEEP; a++) t = t + v[a];
  return t;
}

// Order of every sum over output rows (eq. 5 prescribes none): ROW_LANES = 16 interleaved sub-sums -
// sub-sum l adds the rows j = l, l + 16, l + 32, ... in ascending order - which are then added in
// ascending l.  A fixed order that 16 lanes can work on at once; the lanes of one sum are 16
// neighbouring lanes of a wave.  It differs from an ascending-row sum in the last bits only.
#define ROW_LANES 16

__device__ __forceinline__ double lanes_total(double part) {
  // lane 0 of each group of 16 neighbouring lanes gets ((part_0 + part_1) + part_2) + ... + part_15
  double acc = __shfl(part, 0, ROW_LANES);
#pragma unroll
  for (int l = 1; l < ROW_LANES; l++) acc = acc + __shfl(part, l, ROW_LANES);
  return acc;
}

// ------------------------------------------------------------------------------------------------
// The exchanges are found with a table of its own that is cheaper to evaluate and proven close enough.
//
// With the members of a row in order, w_0 >= w_1 >= ..., and n = NKEEP: what a candidate x adds in place of member i depends on
// whether i is among the n largest.  If not, the others keep w_0 + .. + w_(n-2) and max(w_(n-1), x); if it is, they keep
// the n largest without i and max(w_n, x).  With L = max(w_n, x) and D = max(w_(n-1), x) - L, both the same for all members, the
// value of the group with member i replaced by x is
//   base_i + sum over the rows of L + sum over the rows where i is not among the n largest of D,
// base_i a number per member.  That is four float64 operations per row and candidate for the whole group and a product of a matrix
// of zeros and ones with D, four members at a time on the matrix instruction (which runs on the float64 pipes: 16 clocks against 4 of an
// addition), where the exact table takes 5 operations (2:4) or about 60 (4:8) per member.
//
// With no negative value all terms are at least zero, so the sum, in whatever order, is within (N + 6) 2^-53 of the real one, relatively,
// and what base_i loses where the n largest without i come from a subtraction is below 4 2^-53 v(g) in all; the exact
// table's is within (N + 4) 2^-53.  A group's value with a member replaced is at most twice the largest v(g) (a channel's column is
// nowhere larger than its own group's largest).  So two deltas of
// this table that differ by more than LBS_TOL (N + 64) 2^-53 max v(g) are in the same order in the exact table (four
// values of both deltas, in both tables: 32 (N + 8) 2^-53 max v(g) and roundings; LBS_TOL is twice that), and a delta is
// above or below zero in both if it is farther than that from it.  A round whose best exchange is not proven that way - a
// tie, an exchange that moves the total by rounding only, weights or scores that are not finite or scores below zero -
// leaves the block to the exact table from there on, so the exchanges made are those of the exact table in every case.
//
// Replacing the member that the last exchange brought into a group leaves the same other members as before it, so those
// entries stay valid and are not written again.
//
// A workgroup (8 waves) takes two groups and 16 QC columns, a wave an equal share of the rows.  A lane owns QC columns and
// every fourth row of its wave, so the panel value and its product with the score are formed once for both groups.  A wave forms the
// operands of its next 32 rows itself (one lane per row and group, members read from PT - gathered
// from P they cost the vector-memory path a third of the kernel's time) and needs no barrier.
//
// Bound by float64 instructions.  64 blocks of 4096 x 64, 2:4: all groups 139 us (exact table 677), a round of two touched groups
// 12 of its 17 us (k_lbs_rounds; with two operations per row, candidate and member 18, exact 142); 80 blocks of 5120 x 64, 4:8: 227 (4525) and 50
// of 58 us (two operations per member: 254 and 57; exact 1034).
#define LBS_WAVES 8
#define LBS_ROWS 32  // rows whose operands a wave keeps in LDS
#define LBS_ROUNDS_QUEUED 12
#define LBS_ROUNDS_MAX 64     // times block^2: a block shuffle that has not ended by then is reported
#define LBS_REC 12  // ints per touched group: exchanged position (-1: none), columns of the members
#define LBS_TOL 64.0
enum { LBS_FAST = 0, LBS_DONE = 1, LBS_EXACT = 2 };  // state of a block

// group of the first (0) or second (1) exchanged position of a block; -1: none
template <int MG>
__device__ __forceinline__ int exchanged_group(const int* __restrict__ rec, int blk, int which) {
  const int p = rec[(blk * 2 + which) * LBS_REC];
  return p < 0 ? -1 : p / MG;
}

// ---- the exact table
// V[blk][g][i][x] = retained metric of group g of block blk with its i-th member replaced by panel
// column x of the block (x == the member itself gives v(g)).  grid (entries / 64, blocks), block 1024 =
// 64 entries x 16 row lanes.  `rec` = the exchanged positions, whose groups are refreshed (or NULL = all
// groups).  Entries whose x sits in group g (other than the member itself) are skipped.
// The block's metric values go through LDS in chunks of rows_chunk rows (a multiple of 16; rows are
// padded by one value so that the 16 row lanes of an entry read different banks); the panel values of
// the next chunk are loaded into registers before the current chunk is evaluated.
template <int DT, int NKEEP, int MG>
__global__ void __launch_bounds__(1024) k_lbs_exact(const uint16_t* __restrict__ P, const double* __restrict__ sp /*[K] score in panel order*/,
                                                    const int* __restrict__ lp /*[nblk][B] position -> panel column*/,
                                                    const int* __restrict__ rec /*[nblk][2][LBS_REC] or null*/,
                                                    const int* __restrict__ state /*[nblk]*/, long long N, long long Npad, int B,
                                                    int rows_chunk, double* __restrict__ V /*[nblk][G][MG][B]*/) {
  extern __shared__ unsigned char smem_raw[];
  double* s_xi = reinterpret_cast<double*>(smem_raw);  // [rows_chunk][B + 1]
  __shared__ int s_lp[1024];
  const int blk = blockIdx.y;
  if (state[blk] != LBS_EXACT) return;
  const int G = B / MG;
  const int tid = threadIdx.x;
  const int rl = tid & (ROW_LANES - 1);                  // row lane
  const int eid = blockIdx.x * 64 + (tid >> 4);          // entry within this block's refresh list
  const int per_group = MG * B;
  const int ngroups = rec ? 2 : G;
  const int stride = B + 1;
  for (int i = tid; i < B; i += 1024) s_lp[i] = lp[blk * B + i];
  __syncthreads();
  bool active = eid < ngroups * per_group;
  int g = 0, i = 0, x = 0;
  int cols[MG];
#pragma unroll
  for (int k = 0; k < MG; k++) cols[k] = 0;
  if (active) {
    int gsel = eid / per_group;
    g = rec ? exchanged_group<MG>(rec, blk, gsel) : gsel;
    i = (eid / B) % MG;
    x = eid % B;
    if (g < 0) active = false;
  }
  if (active) {
    bool in_group = false;
#pragma unroll
    for (int k = 0; k < MG; k++) {
      int ck = s_lp[g * MG + k];
      if (ck == x && k != i) in_group = true;
      cols[k] = (k == i) ? x : ck;
    }
    if (in_group) active = false;
  }
  const uint16_t* Pb = P + (long long)blk * Npad * B;
  const double* spb = sp + (long long)blk * B;
  // this thread's share of a chunk: values tid, tid + 1024, ... of the rows_chunk x B values (the same
  // places in every chunk)
  constexpr int EPT = 4;
  const int elems = rows_chunk * B;  // <= EPT * 1024: the host picks rows_chunk <= 4096 / B (B <= 256)
  uint16_t nextv[EPT];
  int rq[EPT], cq[EPT];
  double sq[EPT];
#pragma unroll
  for (int q = 0; q < EPT; q++) {
    const int e = tid + 1024 * q;
    rq[q] = e < elems ? e / B : rows_chunk;  // rows_chunk = "no such value"
    cq[q] = e % B;
    sq[q] = spb[cq[q]];
  }
  auto fetch = [&](long long r0) {
    const int nr = (int)((N - r0) < rows_chunk ? (N - r0) : rows_chunk);
#pragma unroll
    for (int q = 0; q < EPT; q++) nextv[q] = (rq[q] < nr) ? Pb[(r0 + rq[q]) * B + cq[q]] : (uint16_t)0;
  };
  double acc = 0.0;  // this lane's sub-sum
  fetch(0);
  for (long long r0 = 0; r0 < N; r0 += rows_chunk) {
    const int nr = (int)((N - r0) < rows_chunk ? (N - r0) : rows_chunk);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EPT; q++)
      if (rq[q] < nr) s_xi[rq[q] * stride + cq[q]] = (double)esp_to_float<DT>(nextv[q]) * sq[q];
    __syncthreads();
    if (r0 + rows_chunk < N) fetch(r0 + rows_chunk);
    if (active) {
      // rows r0 + rl, r0 + rl + 16, ...: r0 is a multiple of 16, so they are this lane's rows
#pragma unroll 4
      for (int rr = rl; rr < nr; rr += ROW_LANES) {
        double v[MG];
#pragma unroll
        for (int k = 0; k < MG; k++) v[k] = s_xi[rr * stride + cols[k]];
        acc = acc + top_n_sum<NKEEP, MG>(v);
      }
    }
  }
  const double total = lanes_total(active ? acc : 0.0);
  if (active && rl == 0) V[(((long long)blk * G + g) * MG + i) * B + x] = total;
}

// The same table for 2:4, several times faster.  The B candidates x of one (group g, member i)
// combination share the group's three other members, so the two largest of those three are found
// once per row (m1 >= m2) and a candidate's retained metric in that row is
// max(m1, xi_x) + max(m2, min(m1, xi_x)): the two largest of the four values, the same two doubles
// the general network adds.  A workgroup (1024 threads = up to 64 candidates x 16 row lanes) stages the
// block's metric values once per chunk and evaluates NC units with them; a unit is a combination and
// a slice of XL = min(B, 64) candidates.  grid (ceil(units / NC), blocks); B % 64 == 0 or B < 64.
template <int DT, int NC>
__global__ void __launch_bounds__(1024) k_lbs_exact_2_4(const uint16_t* __restrict__ P, const double* __restrict__ sp,
                                                        const int* __restrict__ lp, const int* __restrict__ rec,
                                                        const int* __restrict__ state, long long N, long long Npad, int B, int rows_chunk,
                                                        double* __restrict__ V) {
  constexpr int MG = 4;
  extern __shared__ unsigned char smem_raw[];
  double* s_xi = reinterpret_cast<double*>(smem_raw);  // [rows_chunk][B + 1]
  __shared__ int s_lp[256];
  const int blk = blockIdx.y;
  if (state[blk] != LBS_EXACT) return;
  const int G = B / MG;
  const int tid = threadIdx.x;
  const int rl = tid & (ROW_LANES - 1), xl = tid >> 4;
  const int XL = B < 64 ? B : 64, xslices = B / XL;
  const int ngroups = rec ? 2 : G;
  const int nunits = ngroups * MG * xslices;
  const int stride = B + 1;
  double* s_pair = s_xi + (size_t)rows_chunk * stride;  // [NC][rows_chunk][2]: the 16 row lanes read 256 contiguous bytes
  for (int i = tid; i < B; i += 1024) s_lp[i] = lp[blk * B + i];
  __syncthreads();
  // per unit: group, member, candidate of this thread, and whether the entry exists
  int ug[NC], ui[NC], ux[NC];
  bool uact[NC];
#pragma unroll
  for (int c = 0; c < NC; c++) {
    const int u = blockIdx.x * NC + c;
    const int cmb = u / xslices;
    ux[c] = (u % xslices) * XL + xl;
    ui[c] = cmb % MG;
    const int gsel = cmb / MG;
    ug[c] = -1;
    if (u < nunits) ug[c] = rec ? exchanged_group<MG>(rec, blk, gsel) : gsel;
    uact[c] = ug[c] >= 0 && xl < XL;
    if (!uact[c]) ux[c] = 0;
    if (uact[c]) {
#pragma unroll
      for (int k = 0; k < MG; k++)
        if (k != ui[c] && s_lp[ug[c] * MG + k] == ux[c]) uact[c] = false;  // x is another member of the group
    }
  }
  const uint16_t* Pb = P + (long long)blk * Npad * B;
  const double* spb = sp + (long long)blk * B;
  constexpr int EPT = 4;
  const int elems = rows_chunk * B;  // <= EPT * 1024
  uint16_t nextv[EPT];
  int rq[EPT], cq[EPT];
  double sq[EPT];
#pragma unroll
  for (int q = 0; q < EPT; q++) {
    const int e = tid + 1024 * q;
    rq[q] = e < elems ? e / B : rows_chunk;
    cq[q] = e % B;
    sq[q] = spb[cq[q]];
  }
  auto fetch = [&](long long r0) {
    const int nr = (int)((N - r0) < rows_chunk ? (N - r0) : rows_chunk);
#pragma unroll
    for (int q = 0; q < EPT; q++) nextv[q] = (rq[q] < nr) ? Pb[(r0 + rq[q]) * B + cq[q]] : (uint16_t)0;
  };
  double acc[NC];
#pragma unroll
  for (int c = 0; c < NC; c++) acc[c] = 0.0;
  fetch(0);
  for (long long r0 = 0; r0 < N; r0 += rows_chunk) {
    const int nr = (int)((N - r0) < rows_chunk ? (N - r0) : rows_chunk);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EPT; q++)
      if (rq[q] < nr) s_xi[rq[q] * stride + cq[q]] = (double)esp_to_float<DT>(nextv[q]) * sq[q];
    __syncthreads();
    if (r0 + rows_chunk < N) fetch(r0 + rows_chunk);
    for (int t = tid; t < nr * NC; t += 1024) {
      const int row = t / NC, c = t % NC;
      const int u = blockIdx.x * NC + c;
      const int cmb = u / xslices, mi = cmb % MG, gsel = cmb / MG;
      double m1 = 0.0, m2 = 0.0;
      if (u < nunits) {
        const int gg = rec ? exchanged_group<MG>(rec, blk, gsel) : gsel;
        if (gg >= 0) {
          double o[3];
          int c3 = 0;
#pragma unroll
          for (int k = 0; k < MG; k++)
            if (k != mi) o[c3++] = s_xi[row * stride + s_lp[gg * MG + k]];
          const double hi = fmax(o[0], o[1]), lo = fmin(o[0], o[1]);
          m1 = fmax(hi, o[2]);
          m2 = fmax(lo, fmin(hi, o[2]));
        }
      }
      s_pair[2 * (c * rows_chunk + row)] = m1;
      s_pair[2 * (c * rows_chunk + row) + 1] = m2;
    }
    __syncthreads();
    // rows r0 + rl, r0 + rl + 16, ...: r0 is a multiple of 16, so they are this lane's rows
    for (int rr = rl; rr < nr; rr += ROW_LANES) {
#pragma unroll
      for (int c = 0; c < NC; c++) {  // entries that do not exist compute along (column 0) and are dropped at the end
        const double xv = s_xi[rr * stride + ux[c]];
        const double2 mm = *reinterpret_cast<const double2*>(s_pair + 2 * (c * rows_chunk + rr));
        acc[c] = acc[c] + (fmax(mm.x, xv) + fmax(mm.y, fmin(mm.x, xv)));
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; c++) {
    const double total = lanes_total(uact[c] ? acc[c] : 0.0);
    if (uact[c] && rl == 0) V[(((long long)blk * G + ug[c]) * MG + ui[c]) * B + ux[c]] = total;
  }
}

// ---- the table that is cheaper to evaluate
__device__ __forceinline__ int uniform(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readfirstlane(v);
#else
  return v;
#endif
}

// the value of lane `at` (wave-uniform)
__device__ __forceinline__ int lane_of(int v, int at) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_readlane(v, at);
#else
  return v;
#endif
}
__device__ __forceinline__ double lane_of(double v, int at) {
  const long long b = __double_as_longlong(v);
  return __longlong_as_double(((long long)lane_of((int)(b >> 32), at) << 32) | (unsigned int)lane_of((int)b, at));
}

// orders the LDS accesses of one wave as they are written (its lanes exchange data through LDS)
__device__ __forceinline__ void wave_lds_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#endif
}

// v_max_f64 / v_min_f64 as they are: fmax / fmin come with a canonicalising instruction for every operand that was
// loaded from memory
__device__ __forceinline__ double max_f64(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
#else
  return fmax(a, b);
#endif
}
__device__ __forceinline__ double min_f64(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
#else
  return fmin(a, b);
#endif
}

// the largest of 2^STEPS neighbouring lanes in each of them (STEPS = 3, 4 or 6)
template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true), hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return fmax(v, __longlong_as_double(((long long)hi << 32) | (unsigned int)lo));
#else
  return v;
#endif
}
template <int STEPS>
__device__ __forceinline__ double lanes_max(double v) {
  v = dpp_max<0xb1>(v);   // lanes 1 0 3 2
  v = dpp_max<0x4e>(v);   // lanes 2 3 0 1
  v = dpp_max<0x141>(v);  // lane 7 - l of each 8
  if (STEPS > 3) v = dpp_max<0x140>(v);  // lane 15 - l of each 16
  if (STEPS > 4) {
    v = fmax(v, __shfl_xor(v, 16));
    v = fmax(v, __shfl_xor(v, 32));
  }
  return v;
}

// c + the sum over the four rows k = lane / 16 of a[m][k] b[k][x], m = lane % 4 on the A side, x = lane % 16 on the B side; the result for
// (m, x) is in lane 16 m + x (v_mfma_f64_4x4x4: four independent blocks of four columns; measured with one-hot operands)
__device__ __forceinline__ double mfma_rows(double a, double b, double c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
#else
  return c + a * b;
#endif
}

// what a wave of k_lbs_eval or k_lbs_rounds takes: all members of two groups, 16 QC columns
template <int MG, int QC>
struct LbsShape {
  static_assert((MG == 4 || MG == 8) && (QC == 2 || QC == 4), "");
  static constexpr int NG = 2;              // groups: one per half of the operand lanes
  static constexpr int RLW = 4;             // rows of a wave at a time, 16 lanes each
  static constexpr int U = LBS_ROWS / RLW;  // ... per batch
  static constexpr int NC = NG * MG;        // combinations of group and member
  static constexpr int NS = MG / 4;         // matrix instructions per group and column
  static constexpr int XC = 16 * QC;        // columns
  static constexpr int SUMS = NC * (XC + 1);                       // doubles: a wave's sums, the last of a row its base
  static constexpr int OPS = LBS_ROWS * (2 * NG + NG * MG / 2);    // doubles: a wave's operands
  static constexpr int LDS = LBS_WAVES * OPS > LBS_WAVES / 2 * SUMS ? LBS_WAVES * OPS : LBS_WAVES / 2 * SUMS;
};

// the QC values of a lane in the row at `p`
template <int QC>
__device__ __forceinline__ uint2 lbs_row(const uint16_t* __restrict__ p) {
  if (QC == 4) return *reinterpret_cast<const uint2*>(p);
  return uint2{*reinterpret_cast<const uint32_t*>(p), 0u};
}

// rows of one wave, a multiple of 16: wave w of a block's waves takes rows [w n, w n + n)
__host__ __device__ __forceinline__ long long lbs_wave_rows(long long N, long long waves) { return (N + 16 * waves - 1) / (16 * waves) * 16; }

// A workgroup's sums over its waves' rows [r0, r0 + nrows).  prow: the lane's place in the wave's first rows; next: its values
// there, loaded.  smc, sms: the wave's columns and scores of the members, [NG][MG].  At the end s_o holds, complete after the barrier the function ends with, LBS_WAVES / 2
// partial sums [NC][XC + 1] (lbs_sum adds them).
template <int DT, int NKEEP, int MG, int QC>
__device__ __forceinline__ void lbs_sums(const uint16_t* __restrict__ prow, uint2& next, const double (&s)[QC],
                                         const uint16_t* __restrict__ PTb, const int* smc, const double* sms, long long r0, long long nrows, long long N,
                                         long long Npad, int B, double* s_o, int wave, int lane) {
  using Sh = LbsShape<MG, QC>;
  constexpr int NG = Sh::NG, RLW = Sh::RLW, XC = Sh::XC, NS = Sh::NS;
  const int rlw = lane / 16, xl = lane % 16;
  const int ir = lane % LBS_ROWS, ih = lane / LBS_ROWS;  // operand lane: row ir of the batch, group ih
  double* sw = s_o + wave * Sh::OPS;                                            // [row][NG][2]: the NKEEP-th and the next largest member
  uint32_t* sm = reinterpret_cast<uint32_t*>(sw + LBS_ROWS * 2 * NG);           // [row][NG][MG]: upper half of 0.0 or 1.0
  const long long r1 = r0 + nrows < N ? r0 + nrows : N;
  uint16_t mraw[MG];
  auto load_members = [&](long long rb) {
    const long long r = rb + ir < N ? rb + ir : N - 1;
#pragma unroll
    for (int k = 0; k < MG; k++) mraw[k] = PTb[smc[ih * MG + k] * Npad + r];
  };
  if (r0 < r1) load_members(r0);
  double acc[NG][NS][QC], low[NG][QC];  // sum of D for the members that are not among the NKEEP largest; sum of max(o', x)
#pragma unroll
  for (int g = 0; g < NG; g++)
#pragma unroll
    for (int q = 0; q < QC; q++) {
      low[g][q] = 0.0;
#pragma unroll
      for (int t = 0; t < NS; t++) acc[g][t][q] = 0.0;
    }
  double base[MG];  // operand lanes: what the other members keep besides the candidate's place
#pragma unroll
  for (int k = 0; k < MG; k++) base[k] = 0.0;

  for (long long rb = r0; rb < r1; rb += LBS_ROWS) {
    const bool live = rb + ir < r1;
    wave_lds_fence();
    {
      const double* sc = sms + ih * MG;
      double w[NKEEP + 1];  // the largest members in order
      int raw[MG];
#pragma unroll
      for (int k = 0; k < MG; k++) raw[k] = live ? mraw[k] : 0;
      auto member = [&](int k) { return (double)esp_to_float<DT>((uint16_t)raw[k]) * sc[k]; };
      w[0] = member(0);
#pragma unroll
      for (int k = 1; k < MG; k++) {
        double t = member(k);
#pragma unroll
        for (int q = 0; q <= NKEEP && q < k; q++) {
          const double hi = max_f64(w[q], t);
          t = min_f64(w[q], t);
          w[q] = hi;
        }
        if (k <= NKEEP) w[k] = t;
      }
      double most = w[0];
#pragma unroll
      for (int k = 1; k < NKEEP - 1; k++) most = most + w[k];
      const double all = most + w[NKEEP - 1];
      uint32_t out[MG];
#pragma unroll
      for (int k = 0; k < MG; k++) {
        raw[k] = opaque(raw[k]);  // formed a second time: kept, the values would push sums out of the registers
        const double v = member(k);
        const bool top = v >= w[NKEEP - 1];
        base[k] = base[k] + (top ? all - v : most);
        out[k] = top ? 0u : 0x3ff00000u;
      }
      const int at = ir * NG + ih;
      *reinterpret_cast<double2*>(sw + at * 2) = double2{w[NKEEP - 1], w[NKEEP]};
#pragma unroll
      for (int k = 0; k < MG; k += 4) *reinterpret_cast<uint4*>(sm + at * MG + k) = uint4{out[k], out[k + 1], out[k + 2], out[k + 3]};
    }
    wave_lds_fence();
    if (rb + LBS_ROWS < r1) load_members(rb + LBS_ROWS);
    const int nu = r0 + nrows - rb < LBS_ROWS ? Sh::U / 2 : Sh::U;
    const bool full = rb + nu * RLW <= N;
    const double* wrow = sw + rlw * 2 * NG;
    const uint32_t* mrow = sm + rlw * NG * MG + lane % 4;
    // (The next row's values are loaded one step of four ahead: with four waves per SIMD a step takes as long as a load from the caches.
    // Registers moved on from step to step would wait for the newest load all the same, and unrolled steps take a
    // second set of registers for the results of the matrix instruction.)
#pragma unroll 1
    for (int u = 0; u < nu; u++) {
      const uint2 raw = next;
      prow += RLW * B;
      next = lbs_row<QC>(prow);
      double2 o[NG];
      double m[NG][NS];
#pragma unroll
      for (int g = 0; g < NG; g++) {
        o[g] = *reinterpret_cast<const double2*>(wrow + 2 * g);
#pragma unroll
        for (int t = 0; t < NS; t++) m[g][t] = __longlong_as_double((long long)mrow[g * MG + 4 * t] << 32);
      }
      wrow += RLW * 2 * NG;
      mrow += RLW * NG * MG;
      double x[QC];
#pragma unroll
      for (int q = 0; q < QC; q++) {
        const uint32_t two = q < 2 ? raw.x : raw.y;
        x[q] = (double)esp_to_float<DT>((uint16_t)(q & 1 ? two >> 16 : two & 0xffffu)) * s[q];
      }
      if (!full) {  // no such row: adds exactly 0
        const bool there = rb + u * RLW + rlw < N;
#pragma unroll
        for (int q = 0; q < QC; q++) x[q] = there ? x[q] : 0.0;
      }
#pragma unroll
      for (int g = 0; g < NG; g++)
#pragma unroll
        for (int q = 0; q < QC; q++) {
          const double hi = max_f64(o[g].x, x[q]), lo = max_f64(o[g].y, x[q]);
          low[g][q] = low[g][q] + lo;
#pragma unroll
          for (int t = 0; t < NS; t++) acc[g][t][q] = mfma_rows(m[g][t], hi - lo, acc[g][t][q]);
        }
    }
  }
#pragma unroll
  for (int g = 0; g < NG; g++)
#pragma unroll
    for (int t = 0; t < NS; t++)
#pragma unroll
      for (int q = 0; q < QC; q++) acc[g][t][q] = mfma_rows(1.0, low[g][q], acc[g][t][q]);
#pragma unroll
  for (int k = 0; k < MG; k++)
#pragma unroll
    for (int d = 1; d < LBS_ROWS; d <<= 1) base[k] = base[k] + __shfl_xor(base[k], d);
  // the upper half of the waves leaves its sums in LDS, the lower half adds its own
  double* red = s_o + (wave % (LBS_WAVES / 2)) * Sh::SUMS;
#pragma unroll
  for (int half = 1; half >= 0; half--) {
    __syncthreads();  // half = 1: nobody needs operands any more
    if (wave / (LBS_WAVES / 2) == half) {
      auto leave = [&](double* to, double v) { *to = half ? v : v + *to; };
#pragma unroll
      for (int g = 0; g < NG; g++)
#pragma unroll
        for (int t = 0; t < NS; t++)
#pragma unroll
          for (int q = 0; q < QC; q++) leave(red + (g * MG + 4 * t + rlw) * (XC + 1) + QC * xl + q, acc[g][t][q]);
      if (ir == 0)
#pragma unroll
        for (int k = 0; k < MG; k++) leave(red + (ih * MG + k) * (XC + 1) + XC, base[k]);
    }
  }
  __syncthreads();
}

// the sum of combination c and column x
template <int MG, int QC>
__device__ __forceinline__ double lbs_sum(const double* s_o, int c, int x) {
  using Sh = LbsShape<MG, QC>;
  const double* sums = s_o + c * (Sh::XC + 1);
  double t = sums[x], tb = sums[Sh::XC];
#pragma unroll
  for (int w = 1; w < LBS_WAVES / 2; w++) {
    t = t + sums[w * Sh::SUMS + x];
    tb = tb + sums[w * Sh::SUMS + Sh::XC];
  }
  return t + tb;
}

// the first table: groups 2 gset and 2 gset + 1 of every block
template <int DT, int NKEEP, int MG, int QC>
__global__ void __launch_bounds__(64 * LBS_WAVES, 4) k_lbs_eval(const uint16_t* __restrict__ P, const uint16_t* __restrict__ PT, const double* __restrict__ sp /*[K] score in panel order*/,
                                                              long long N, long long Npad, int B, int slices, double* __restrict__ S /*[nsplit][nblk][B][B]*/) {
  using Sh = LbsShape<MG, QC>;
  constexpr int NG = Sh::NG, NC = Sh::NC, XC = Sh::XC;
  __shared__ __align__(16) double s_o[Sh::LDS];
  __shared__ double s_ms[LBS_WAVES * NC];
  __shared__ int s_mc[LBS_WAVES * NC];
  const int blk = blockIdx.x, nblk = gridDim.x, split = blockIdx.y, nsplit = gridDim.y;
  const int slice = (int)blockIdx.z % slices, gset = (int)blockIdx.z / slices;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int col0 = slice * XC + QC * (lane % 16);
  const int colc = col0 < B ? col0 : 0;  // columns past the block compute along and are dropped at the end
  const long long nrows = lbs_wave_rows(N, nsplit * LBS_WAVES), r0 = (split * LBS_WAVES + wave) * nrows;
  const uint16_t* prow = P + ((long long)blk * Npad + r0 + lane / 16) * B + colc;
  uint2 next = lbs_row<QC>(prow);
  int* smc = s_mc + wave * NC;
  double* sms = s_ms + wave * NC;
  if (lane < NC) {  // positions are columns; past the last group: the first one again, dropped at the end
    const int g = gset * NG + lane / MG;
    const int c = (g < B / MG ? g : 0) * MG + lane % MG;
    smc[lane] = c;
    sms[lane] = sp[(long long)blk * B + c];
  }
  wave_lds_fence();
  double s[QC];
#pragma unroll
  for (int q = 0; q < QC; q++) s[q] = sp[(long long)blk * B + colc + q];
  lbs_sums<DT, NKEEP, MG, QC>(prow, next, s, PT + (long long)blk * B * Npad, smc, sms, r0, nrows, N, Npad, B, s_o, wave, lane);
  double* Sb = S + ((long long)split * nblk + blk) * B * B;
  for (int e = tid; e < NC * XC; e += 64 * LBS_WAVES) {
    const int c = e / XC, x = slice * XC + e % XC, g = gset * NG + c / MG, i = c % MG;
    if (x < B && g < B / MG) Sb[(long long)(g * MG + i) * B + x] = lbs_sum<MG, QC>(s_o, c, e % XC);
  }
}

// ---- rounds in a launch of their own (blocks of more than LBS_TEAM_BLOCK columns, teams that gave up)
// Such a round is short and leaves many CUs idle, so the form above, which makes one wave do all members of both groups, loses to the one it is derived from:
// without member i, with o the NKEEP largest of the other members, a candidate x adds o_0 + .. + o_(NKEEP-2) + max(o_(NKEEP-1), x) to a row, a number per
// member and two operations per row, candidate and member.  2:4 takes both groups in a workgroup, 4:8 one; the member that the last exchange brought in is
// left out.  The sums are as near to the real ones as those above.  A lane owns QC columns and every fourth row of its wave; the 16 lanes of a
// row read its operands once and pass them around.
// Calls with 40 exchanges, 4:8: 8 blocks of 512 x 72 880 -> 692 us with this form, 2 of 256 x 128 1209 -> 1006, 32 of 4096 x 256 5538 -> 5077; 2:4: 860 -> 816,
// 973 -> 925, 64 of 4096 x 128 2661 -> 2484.  Of 81 sizes three are slower: 4:8, 72 columns, 64 blocks of 8192 and 36 of 9216 rows (5672 -> 6040, 4152 ->
// 4365), 2:4, 256 columns, 16 blocks of 2048 rows (2338 -> 2449).
// the value of lane LANE of each row of 16 lanes in all lanes of that row
template <int LANE>
__device__ __forceinline__ double row_bcast(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + LANE, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + LANE, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
#else
  return v;
#endif
}

// a + b with half of the lanes of each exchanged: lanes 0-31 get a[l] + a[l + 32], lanes 32-63 b[l - 32] + b[l]
// (HALF), or the same within each pair of 16-lane rows
template <bool HALF>
__device__ __forceinline__ double swap_add(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  unsigned int r[4];
  if (HALF) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned int)x, (unsigned int)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned int)(x >> 32), (unsigned int)(y >> 32), false, false);
    r[0] = lo[0]; r[1] = lo[1]; r[2] = hi[0]; r[3] = hi[1];
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned int)x, (unsigned int)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned int)(x >> 32), (unsigned int)(y >> 32), false, false);
    r[0] = lo[0]; r[1] = lo[1]; r[2] = hi[0]; r[3] = hi[1];
  }
  return __longlong_as_double(((long long)r[2] << 32) | r[0]) + __longlong_as_double(((long long)r[3] << 32) | r[1]);
#else
  return a + b;
#endif
}

template <int DT, int NKEEP, int MG, int QC>
__global__ void __launch_bounds__(64 * LBS_WAVES, 4) k_lbs_refresh(const uint16_t* __restrict__ P, const uint16_t* __restrict__ PT, const double* __restrict__ sp /*[K] score in panel order*/,
                                                              const int* __restrict__ rec /*[nblk][2][LBS_REC] exchanged positions and their groups*/,
                                                              long long N, long long Npad, int B, int slices, double* __restrict__ S /*[nsplit][nblk][B][B]*/) {
  constexpr int RLW = 4;                 // rows of a wave at a time, 16 lanes each
  constexpr int U = LBS_ROWS / RLW;      // rows of a lane per batch
  constexpr int NG = MG == 4 ? 2 : 1;    // groups of a workgroup
  constexpr int NM = MG - 1;             // members to evaluate
  constexpr int NC = NG * NM;            // combinations of group and member
  constexpr int XC = 16 * QC;            // columns of a workgroup
  static_assert(NC <= 16 && (QC == 2 || QC == 4), "a row's operands fit its 16 lanes");
  constexpr int NCP = NC | 1;            // operands of a row in LDS
  constexpr int ROOM = LBS_ROWS * NCP > NC * (XC + 1) ? LBS_ROWS * NCP : NC * (XC + 1);
  __shared__ __align__(16) double s_o[LBS_WAVES * ROOM];  // per wave: operands; at the end its sums
  __shared__ double s_ms[LBS_WAVES * 2 * MG];
  __shared__ int s_mc[LBS_WAVES * 2 * MG];
  const int blk = blockIdx.x, nblk = gridDim.x, split = blockIdx.y, nsplit = gridDim.y;
  const int slice = (int)blockIdx.z % slices, gset = (int)blockIdx.z / slices;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int rlw = lane / 16, xl = lane % 16;
  const int col0 = slice * XC + QC * xl;
  const int colc = col0 < B ? col0 : 0;  // columns past the block compute along and are dropped at the end
  // operand lane: row ir of the batch; NG = 2: group ih, all members; NG = 1: members ih, ih + 2, ...
  const int ir = lane % LBS_ROWS, ih = lane / LBS_ROWS;
  // batches of 32 rows: rows rb + u RLW + rlw of the panel, which is padded to whole batches; rows past N are replaced
  // by zeros
  const long long step = (long long)nsplit * LBS_WAVES * LBS_ROWS;
  const long long rb0 = (long long)(split * LBS_WAVES + wave) * LBS_ROWS;
  const uint16_t* Pb = P + (long long)blk * Npad * B;
  const int xoff = rlw * B + colc;
  // the values are loaded AHEAD rows ahead: a row takes about 1700 clocks with four waves per SIMD, a load from the
  // last-level cache as long
  constexpr int AHEAD = 3;
  const uint16_t* prow = Pb + rb0 * B;
  const long long jump = (step - LBS_ROWS) * B;  // from one batch of the wave to the next
  uint2 next[AHEAD];
  auto load_row = [&]() {
    if (QC == 4) return *reinterpret_cast<const uint2*>(prow + xoff);
    return uint2{*reinterpret_cast<const uint32_t*>(prow + xoff), 0u};
  };
#pragma unroll
  for (int q = 0; q < AHEAD; q++, prow += RLW * B) next[q] = load_row();
  // groups of this workgroup: their number, the member that needs no evaluation, the members' columns
  int wg[NG], wskip[NG];
  int* smc = s_mc + (wave * 2 + (NG == 2 ? ih : 0)) * MG;  // the lane's group: columns and scores of the members
  double* sms = s_ms + (wave * 2 + (NG == 2 ? ih : 0)) * MG;
#pragma unroll
  for (int k = 0; k < NG; k++) {
    const int* rg = rec + (blk * 2 + gset * NG + k) * LBS_REC;
    if (rg[0] < 0) return;  // the block is done
    wg[k] = rg[0] / MG;
    wskip[k] = rg[0] % MG;
    if (NG == 1 || ih == k)
#pragma unroll
      for (int i = 0; i < MG; i++) smc[i] = rg[1 + i];
  }
  const int iskip = NG == 2 && ih == 1 ? wskip[NG - 1] : wskip[0];
  wave_lds_fence();
  const uint16_t* PTb = PT + (long long)blk * B * Npad + ir;
  uint16_t mraw[MG];
  auto load_members = [&](long long rb) {
#pragma unroll
    for (int k = 0; k < MG; k++) mraw[k] = PTb[smc[k] * Npad + rb];
  };
  if (rb0 < N) load_members(rb0);
  double s[QC];
#pragma unroll
  for (int q = 0; q < QC; q++) s[q] = sp[(long long)blk * B + colc + q];
#pragma unroll
  for (int k = 0; k < MG; k++) sms[k] = sp[(long long)blk * B + smc[k]];
  double* so = s_o + wave * ROOM;
  constexpr int NA = (NC * QC + 3) / 4 * 4;
  double acc[NA];  // [NC][QC], a multiple of four
#pragma unroll
  for (int f = 0; f < NA; f++) acc[f] = 0.0;
  constexpr int NB = NG == 2 ? NM : (NM + 1) / 2;  // members of an operand lane
  double base[NB];  // operand lanes: what the other members keep besides the operand
#pragma unroll
  for (int c = 0; c < NB; c++) base[c] = 0.0;

  for (long long rb = rb0; rb < N; rb += step) {
    {
      const bool live = rb + ir < N;
      double w[NKEEP + 1];  // the largest members, in order
      wave_lds_fence();
      auto member = [&](int k) {
        const double v = (double)esp_to_float<DT>(mraw[k]) * sms[k];
        return live ? v : 0.0;
      };
      w[0] = member(0);
#pragma unroll
      for (int k = 1; k < MG; k++) {
        double v = member(k);
#pragma unroll
        for (int q = 0; q <= NKEEP && q < k; q++) {
          const double hi = max_f64(w[q], v);
          v = min_f64(w[q], v);
          w[q] = hi;
        }
        if (k <= NKEEP) w[k] = v;
      }
#pragma unroll
      for (int q = 0; q < NB; q++) {  // without member i: the largest, with the next one in place of that member
        const int c = NG == 2 ? q : 2 * q + ih;
        double v;
        if (NG == 2) v = member(q);
        else v = ih ? member(2 * q + 1 < MG ? 2 * q + 1 : 2 * q) : member(2 * q);
        double vn;
        if (NG == 2) vn = member(q + 1);
        else vn = ih ? member(2 * q + 2 < MG ? 2 * q + 2 : 2 * q) : member(2 * q + 1 < MG ? 2 * q + 1 : 2 * q);
        v = c >= iskip ? vn : v;
        double kept = v >= w[0] ? w[1] : w[0];
#pragma unroll
        for (int k = 1; k < NKEEP - 1; k++) kept = kept + (v >= w[k] ? w[k + 1] : w[k]);
        base[q] = base[q] + kept;
        if (c < NM) so[ir * NCP + (NG == 2 ? ih : 0) * NM + c] = v >= w[NKEEP - 1] ? w[NKEEP] : w[NKEEP - 1];
      }
      wave_lds_fence();
    }
    const long long rnext = rb + step;
    const bool full = rb + LBS_ROWS <= N;
    if (rnext < N) load_members(rnext);
    // lane c of a row reads the operand of combination c and hands it to the other 15
    const double* src = so + rlw * NCP + (xl < NC ? xl : NC - 1);
    double o_next = *src;
#pragma unroll 1
    for (int u = 0; u < U; u++) {
      const uint2 raw = next[0];
#pragma unroll
      for (int q = 1; q < AHEAD; q++) next[q - 1] = next[q];
      if (u == U - AHEAD) prow += jump;
      next[AHEAD - 1] = load_row();
      prow += RLW * B;
      const double o = o_next;
      src += u < U - 1 ? RLW * NCP : 0;
      o_next = *src;
      double x[QC];
#pragma unroll
      for (int q = 0; q < QC; q++) {
        const uint32_t two = q < 2 ? raw.x : raw.y;
        x[q] = (double)esp_to_float<DT>((uint16_t)(q & 1 ? two >> 16 : two & 0xffffu)) * s[q];
      }
      if (!full) {  // no such row: adds exactly 0 whatever the scores are
        const bool live = rb + u * RLW + rlw < N;
#pragma unroll
        for (int q = 0; q < QC; q++) x[q] = live ? x[q] : 0.0;
      }
#define LBS_ADD(c)                                                                                         \
  if constexpr (c < NC) {                                                                                  \
    const double oc = row_bcast<c>(o);                                                                     \
    _Pragma("unroll") for (int q = 0; q < QC; q++) acc[c * QC + q] = acc[c * QC + q] + max_f64(oc, x[q]);  \
  }
      LBS_ADD(0) LBS_ADD(1) LBS_ADD(2) LBS_ADD(3) LBS_ADD(4) LBS_ADD(5) LBS_ADD(6) LBS_ADD(7)
#undef LBS_ADD
    }
  }
  // the four rows of the wave: row lane r ends up with the sums number 4 k + {0, 2, 1, 3}[r]
#pragma unroll
  for (int f = 0; f < NA; f += 4) acc[f / 4] = swap_add<false>(swap_add<true>(acc[f], acc[f + 1]), swap_add<true>(acc[f + 2], acc[f + 3]));
  // operand lanes: over the 32 rows; NG = 1: the other half of the lanes holds the other members
#pragma unroll
  for (int q = 0; q < NB; q++)
#pragma unroll
    for (int d = 1; d < LBS_ROWS; d <<= 1) base[q] = base[q] + __shfl_xor(base[q], d);
  wave_lds_fence();
  double* red = so;  // [NC][XC + 1]: the wave's sums and, last in a row, its base
#pragma unroll
  for (int k = 0; k < NA / 4; k++) {
    const int f = 4 * k + ((rlw & 1) << 1 | rlw >> 1), c = f / QC;
    if (c < NC) red[c * (XC + 1) + QC * xl + f % QC] = acc[k];
  }
  if (ir == 0) {
#pragma unroll
    for (int q = 0; q < NB; q++) {
      const int c = NG == 2 ? q : 2 * q + ih;
      if (c < NM) red[((NG == 2 ? ih : 0) * NM + c) * (XC + 1) + XC] = base[q];
    }
  }
  __syncthreads();
  double* Sb = S + ((long long)split * nblk + blk) * B * B;
  for (int e = tid; e < NC * XC; e += 64 * LBS_WAVES) {
    const int c = e / XC, x = slice * XC + e % XC;
    const double* sums = s_o + c * (XC + 1);
    double t = sums[e % XC], tb = sums[XC];
#pragma unroll
    for (int wv = 1; wv < LBS_WAVES; wv++) {
      t = t + sums[wv * ROOM + e % XC];
      tb = tb + sums[wv * ROOM + XC];
    }
    t = t + tb;
    const int k = c / NM, g = NG == 2 && k == 1 ? wg[NG - 1] : wg[0], skip = NG == 2 && k == 1 ? wskip[NG - 1] : wskip[0];
    int i = c % NM;
    if (i >= skip) i++;
    if (x < B) Sb[(long long)(g * MG + i) * B + x] = t;
  }
}

// One workgroup per block in the given mode: the best exchange (largest delta, ties -> smallest (i, j)), applied if
// delta > 0.  LBS_FAST first adds the workgroups' sums of the entries evaluated last (all of them in the first round) into
// V, and leaves the block to the exact table if the best exchange is not proven to be that table's.
// count[0] / count[1]: blocks in LBS_FAST / LBS_EXACT.
template <int MG>
__global__ void __launch_bounds__(1024) k_lbs_select(const double* __restrict__ S, int nsplit, double* __restrict__ V, int* __restrict__ lp,
                                                      int* __restrict__ rec, int* __restrict__ state, long long* __restrict__ swaps,
                                                      long long max_swaps, long long N, int B, int first, int mode,
                                                      const int* __restrict__ not_finite, int* __restrict__ count) {
  const int blk = blockIdx.x, nblk = gridDim.x;
  int* recb = rec + blk * 2 * LBS_REC;
  const int st = state[blk], pa = first ? 0 : recb[0], pb = first ? 0 : recb[LBS_REC];
  const bool fast = mode == LBS_FAST, bad = *not_finite != 0;
  if (st != mode) return;
  const int G = B / MG;
  const int tid = threadIdx.x;
  __shared__ int s_lp[256];
  __shared__ double s_v[128];  // v(g)
  __shared__ double s_best[16], s_next[16];
  __shared__ int s_pair[16];
  if (tid < B) s_lp[tid] = lp[blk * B + tid];
  double* Vb = V + (long long)blk * B * B;
  if (fast) {
    const double* Sb = S + (long long)blk * B * B;
    const long long sstride = (long long)nblk * B * B;
    auto combine = [&](int e) {
      double t = Sb[e];
      for (int q = 1; q < nsplit; q++) t = t + Sb[q * sstride + e];
      Vb[e] = t;
    };
    if (first) {
      for (int e = tid; e < B * B; e += 1024) combine(e);
    } else {
      for (int e = tid; e < 2 * (MG - 1) * B; e += 1024) {
        const int r = e / B, x = e - r * B;
        const int p = r < MG - 1 ? pa : pb;
        int i = r < MG - 1 ? r : r - (MG - 1);
        if (i >= p % MG) i++;
        combine((p / MG * MG + i) * B + x);
      }
    }
  }
  __syncthreads();
  if (tid < G) s_v[tid] = Vb[(tid * MG) * B + s_lp[tid * MG]];
  __syncthreads();
  // best and second best delta of the pairs i < j in different groups
  double best = -INFINITY, next = -INFINITY;
  int best_pair = -1;
  const int tx = tid & 63, ty = tid >> 6;
  for (int i = ty; i < B; i += 16) {  // pairs i * B + j in ascending order per thread
    const int a = i / MG;
    for (int j = (a + 1) * MG + tx; j < B; j += 64) {
      const int b = j / MG;
      const double va2 = Vb[i * B + s_lp[j]];
      const double vb2 = Vb[j * B + s_lp[i]];
      const double delta = (va2 + vb2) - (s_v[a] + s_v[b]);
      if (delta > best) {
        next = best;
        best = delta;
        best_pair = i * B + j;
      } else if (delta > next) {
        next = delta;
      }
    }
  }
  auto merge = [&](double od, double on, int op) {
    const bool take = op >= 0 && (best_pair < 0 || od > best || (od == best && op < best_pair));
    const double lose = take ? best : od;
    next = fmax(fmax(next, on), lose);
    if (take) {
      best = od;
      best_pair = op;
    }
  };
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    const double od = __shfl_xor(best, s), on = __shfl_xor(next, s);
    const int op = __shfl_xor(best_pair, s);
    merge(od, on, op);
  }
  if (tx == 0) {
    s_best[ty] = best;
    s_next[ty] = next;
    s_pair[ty] = best_pair;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; w++) merge(s_best[w], s_next[w], s_pair[w]);
    int to = LBS_DONE;
    if (fast) {
      double vmax = 0.0;
      bool fine = !bad;
      for (int g = 0; g < G; g++) {
        fine = fine && s_v[g] < 1e300;
        vmax = fmax(vmax, s_v[g]);
      }
      const double tol = LBS_TOL * 0x1p-53 * ((double)N + 64.0) * vmax;
      if (fine && best_pair >= 0 && best > tol && best - next > tol) to = LBS_FAST;
      else if (!(fine && (best_pair < 0 || best < -tol))) to = LBS_EXACT;
    } else if (best_pair >= 0 && best > 0.0) {
      to = LBS_EXACT;
    }
    if (to == mode) {  // exchange
      const int i = best_pair / B, j = best_pair % B;
      lp[blk * B + i] = s_lp[j];
      lp[blk * B + j] = s_lp[i];
      for (int k = 0; k < MG; k++) {
        const int qa = i / MG * MG + k, qb = j / MG * MG + k;
        recb[1 + k] = qa == i ? s_lp[j] : s_lp[qa];
        recb[LBS_REC + 1 + k] = qb == j ? s_lp[i] : s_lp[qb];
      }
      recb[0] = i;
      recb[LBS_REC] = j;
      const long long sw = swaps[blk] + 1;
      swaps[blk] = sw;
      if (max_swaps > 0 && sw >= max_swaps) to = LBS_DONE;
    }
    if (to != mode) {
      state[blk] = to;
      recb[0] = recb[LBS_REC] = -1;
      atomicSub(&count[fast ? 0 : 1], 1);
      if (to == LBS_EXACT) atomicAdd(&count[1], 1);
    }
  }
}

// ---- the rounds in one launch
// After the first table the exchanges of a block depend on that block alone.  A team of workgroups takes a block through
// all its rounds: each workgroup evaluates its rows for the touched groups, reads the sums of the whole team and makes the same choice as all
// others from its own copy of the table (V, in LDS) and of the positions.  A launch per kernel and round left the chip idle for about 12 of 28 us
// (launches, first loads behind a chain of three, a selection by 64 workgroups on tables in global memory) and kept every
// block waiting for the one with the most exchanges.
//
// Exchange of the sums: through agent-scope accesses only (they pass by the caches that are not coherent between XCDs).  A
// place holds LBS_EMPTY, no sum's bits, until its owner has written it, and the readers look until it does not: no
// counter, one trip through memory.  Three buffers in turn: in round r the owner empties its places of buffer (r + 1) mod 3 and waits for these stores before it
// writes its sums of round r.  Whoever sees those therefore finds emptied places in round r + 1, and whoever empties has seen every
// member's sums of round r - 1, which come after that member's last read of that buffer (round r - 2).  Buffer 0 is empty at the start.
//
// Waiting: workgroups are dispatched in the order of their numbers, in turn to the 8 XCDs (b mod 8); a team is consecutive
// numbers of one XCD, at most 16 of the 64 workgroups that an XCD holds at a time.  So of one launch at most the last team of an XCD is there
// in part, and parts of four launches at a time (as many as the hardware queues of a process) leave four places of the 64, enough to complete one
// of them: all others finish without anyone's help and make room.  Only progress hangs
// on that: a wait ends after `wait` ticks of 10 ns (the context's team_wait) or once another one has ended that way, the block then stays in
// LBS_FAST as it was before the launch and the caller goes on with a launch per round.
// (Teams of up to 32: 512 channels, 16384 rows 841 instead of 1003 us for 2:4, 1170 instead of 1397 for 4:8; 1024 channels 1133 instead of 1085 and
// 1541 instead of 1650; 1536 channels 1696 instead of 1512 and 2320 both; the same up to 4096 rows.  But parts of three launches then fill an XCD.)
#define LBS_EMPTY 0xffffffffffffffffull
#define LBS_TEAM_MAX 16
#define LBS_XCDS 8
#define LBS_XCD_GROUPS 64          // workgroups of an XCD at a time, two per CU
#define LBS_TEAM_BLOCK 64          // largest block: V in LDS

template <int DT, int NKEEP, int MG, int QC>
__global__ void __launch_bounds__(64 * LBS_WAVES, 4) k_lbs_rounds(const uint16_t* __restrict__ P, const uint16_t* __restrict__ PT, const double* __restrict__ sp,
                                                                const double* __restrict__ V, int* __restrict__ lp, int* __restrict__ rec, int* __restrict__ state,
                                                                long long* __restrict__ swaps, long long max_swaps, long long N, long long Npad, int nblk, int B,
                                                                int T, unsigned long long* __restrict__ S /*[3][nblk][T][2 MG][B]*/, int* __restrict__ gave_up, unsigned long long wait,
                                                                const int* __restrict__ not_finite, int* __restrict__ count) {
  using Sh = LbsShape<MG, QC>;
  constexpr int NC = Sh::NC, XC = Sh::XC, NT = 64 * LBS_WAVES;
  constexpr int VS = XC + 1;  // a row of V in LDS: a column's entries stand in different banks
  __shared__ __align__(16) double s_o[Sh::LDS];
  __shared__ double s_V[XC * VS];
  __shared__ double s_ms[LBS_WAVES * NC];
  __shared__ int s_mc[LBS_WAVES * NC];
  __shared__ double s_sp[XC], s_best[LBS_WAVES], s_next[LBS_WAVES];
  __shared__ int s_lp[XC], s_pair[LBS_WAVES], s_go;
  const int tid = threadIdx.x, wave = uniform(tid >> 6);
  const int j8 = (int)blockIdx.x / 8, blk = j8 / T * 8 + (int)blockIdx.x % 8, member = j8 % T;
  if (blk >= nblk || state[blk] != LBS_FAST) return;  // a team's members read the same
  int pa = rec[blk * 2 * LBS_REC], pb = rec[(blk * 2 + 1) * LBS_REC];  // positions exchanged last
  const bool bad = *not_finite != 0;
  long long sw = swaps[blk];
  if (tid < B) {
    s_lp[tid] = lp[blk * B + tid];
    s_sp[tid] = sp[(long long)blk * B + tid];
  }
  if (tid == 0) s_go = 1;
  for (int e = tid; e < B * B; e += NT) s_V[e / B * VS + e % B] = V[(long long)blk * B * B + e];
  const long long nrows = lbs_wave_rows(N, T * LBS_WAVES), r0 = (member * LBS_WAVES + wave) * nrows;
  const uint16_t* first_row = P + ((long long)blk * Npad + r0) * B;  // the wave's
  const uint16_t* PTb = PT + (long long)blk * B * Npad;
  uint2 next;
  auto column = [&](int lane) { return QC * (lane % 16) < B ? QC * (lane % 16) : 0; };
  auto load_first = [&](int lane) { next = lbs_row<QC>(first_row + (lane / 16 * B + column(lane))); };
  load_first(tid & 63);
  __syncthreads();
  const int per = 2 * MG * B;  // sums of a member and round
  const double tol_n = LBS_TOL * 0x1p-53 * ((double)N + 64.0);
  int to = LBS_FAST;
  for (int round = 0; to == LBS_FAST; round++) {
    if (round >= B * B * LBS_ROUNDS_MAX) return;  // the caller reports it
    // ---- this workgroup's rows
    {
      unsigned long long* Se = S + (((long long)((round + 1) % 3) * nblk + blk) * T + member) * per;
      for (int e = opaque(tid); e < per; e += NT) __hip_atomic_store(Se + e, LBS_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int lane = opaque(tid & 63), colc = column(lane);
      int* smc = s_mc + wave * NC;
      double* sms = s_ms + wave * NC;
      if (lane < NC) {
        const int c = s_lp[(lane / MG == 0 ? pa : pb) / MG * MG + lane % MG];
        smc[lane] = c;
        sms[lane] = s_sp[c];
      }
      double s[QC];
#pragma unroll
      for (int q = 0; q < QC; q++) s[q] = s_sp[colc + q];
      wave_lds_fence();
      lbs_sums<DT, NKEEP, MG, QC>(first_row + (lane / 16 * B + colc), next, s, PTb, smc, sms, r0, nrows, N, Npad, B, s_o, wave, lane);
    }
    // ---- the team's sums, the touched entries of the table
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the emptied places of this wave have arrived
#endif
    __syncthreads();
    unsigned long long* Sb = S + ((long long)(round % 3) * nblk + blk) * T * per;
    for (int e = opaque(tid); e < NC * XC; e += NT) {
      const int c = e / XC, x = e % XC;
      unsigned long long bits = (unsigned long long)__double_as_longlong(lbs_sum<MG, QC>(s_o, c, x));
      if (bits == LBS_EMPTY) bits = 0x7ff8000000000000ull;  // another NaN
      if (x < B) __hip_atomic_store(Sb + (long long)member * per + c * B + x, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the first rows of the next round do not depend on the exchange: on their way meanwhile
    load_first(opaque(tid & 63));
    for (int e = opaque(tid); e < per; e += NT) {
      const int r = e / B, x = e - r * B, p = r < MG ? pa : pb, i = r % MG;
      if (i == p % MG) continue;  // the other members are what they were
      double t = 0.0;
      for (int q0 = 0; q0 < T; q0 += 4) {
        unsigned long long v[4];
        auto look = [&]() {
#pragma unroll
          for (int q = 0; q < 4; q++)
            v[q] = __hip_atomic_load(Sb + (long long)(q0 + q < T ? q0 + q : q0) * per + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return v[0] != LBS_EMPTY && v[1] != LBS_EMPTY && v[2] != LBS_EMPTY && v[3] != LBS_EMPTY;
        };
        if (!look()) {
          const unsigned long long t0 = wall_clock64();
          while (!look()) {
            if (__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > wait) {
              __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              s_go = 0;
              break;
            }
          }
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const double d = __longlong_as_double((long long)v[q]);
          t = q0 + q == 0 ? d : (q0 + q < T ? t + d : t);
        }
      }
      s_V[(p / MG * MG + i) * VS + x] = t;
    }
    __syncthreads();
    if (!s_go) return;
    // ---- best and second best delta of the pairs i < j in different groups, as in k_lbs_select (of equal ones the best is also the
    // second best: no exchange is made then, so which of them is taken does not matter)
    const int lane = opaque(tid & 63), j = lane < B ? lane : 0, b = j / MG;
    const int lpj = s_lp[j];
    const double vb = s_V[(b * MG) * VS + s_lp[b * MG]];
    double best = -INFINITY, second = -INFINITY;
    int pair = 0;
#pragma unroll
    for (int k = 0; k < XC / LBS_WAVES; k++) {
      const int i = wave + k * LBS_WAVES < B ? wave + k * LBS_WAVES : B - 1;  // (again: no j comes after the last group)
      const double sum = s_V[i * VS + lpj] + s_V[j * VS + lane_of(lpj, i)];
      double delta = sum - (lane_of(vb, i) + vb);
      delta = j / MG > i / MG ? delta : -INFINITY;
      second = max_f64(second, min_f64(best, delta));
      pair = delta > best ? i * B + j : pair;
      best = max_f64(best, delta);
    }
    {
      const double top = lanes_max<6>(best);
      const int win = __ffsll((unsigned long long)__ballot(best == top)) - 1;
      second = lanes_max<6>(lane == win ? second : best);
      if (lane == (win < 0 ? 0 : win)) {
        s_best[wave] = top;
        s_next[wave] = second;
        s_pair[wave] = pair;
      }
    }
    const int gl = lane % 16 * MG < B ? lane % 16 : 0;
    const double vg = s_V[(gl * MG) * VS + s_lp[gl * MG]];
    const bool fine = !bad && __all(vg < 1e300);
    const double tol = tol_n * lanes_max<4>(vg);
    __syncthreads();
    {
      const double mine = s_best[lane % LBS_WAVES];
      best = lanes_max<3>(mine);
      const int win = __ffsll((unsigned long long)__ballot(mine == best)) - 1;
      second = lanes_max<3>(lane % LBS_WAVES == win ? s_next[lane % LBS_WAVES] : mine);
      pair = s_pair[win < 0 ? 0 : win];
    }
    if (fine && best > tol && best - second > tol) {  // exchange
      pa = uniform(pair / B);
      pb = uniform(pair % B);
      __syncthreads();  // everyone has read the positions
      if (tid == 0) {
        const int c = s_lp[pa];
        s_lp[pa] = s_lp[pb];
        s_lp[pb] = c;
      }
      sw++;
      if (max_swaps > 0 && sw >= max_swaps) to = LBS_DONE;
      __syncthreads();
    } else {
      to = fine && best < -tol ? LBS_DONE : LBS_EXACT;
    }
  }
  if (member == 0) {
    if (tid < B) lp[blk * B + tid] = s_lp[tid];
    if (tid == 0) {
      swaps[blk] = sw;
      state[blk] = to;
      rec[blk * 2 * LBS_REC] = rec[(blk * 2 + 1) * LBS_REC] = -1;
      atomicSub(&count[0], 1);
      if (to == LBS_EXACT) atomicAdd(&count[1], 1);
    }
  }
}

__global__ void k_lbs_init(int* lp, int* state, int state0, long long* swaps, int* count, unsigned long long* meet /*of the teams*/, long long empty /*of its places*/, int nblk, int B) {
  int t = blockIdx.x * 256 + threadIdx.x;
  if (t < nblk * B) lp[t] = t % B;
  for (long long e = t; e < empty; e += (long long)gridDim.x * 256) meet[e] = LBS_EMPTY;
  if (t < nblk) {
    state[t] = state0;
    swaps[t] = 0;
  }
  if (t < 4) count[t] = t == (state0 == LBS_FAST ? 0 : 1) ? nblk : 0;  // [2]: weights that are not finite; [3]: a team gave up waiting
}

__global__ void k_lbs_final_theta(const int32_t* theta0, const int* lp, int B, long long K, int32_t* theta) {
  long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= K) return;
  long long blk = p / B;
  theta[p] = theta0[blk * B + lp[p]];
}

// ------------------------------------------------------------------------------------------------
// n:m mask on the final order, one thread per (row, group); ties -> lower position kept
// ------------------------------------------------------------------------------------------------
template <int DT, int NKEEP, int MG>
__global__ void __launch_bounds__(256) k_nm_mask(const uint16_t* __restrict__ W, const double* __restrict__ s /*original order*/,
                                                  const int32_t* __restrict__ theta, long long N, long long K,
                                                  uint8_t* __restrict__ mask) {
  const long long ng = K / MG;
  long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= N * ng) return;
  long long j = e / ng, g = e % ng;
  double xi[MG];
#pragma unroll
  for (int k = 0; k < MG; k++) {
    int c = theta[g * MG + k];
    xi[k] = fabs((double)esp_to_float<DT>(W[j * K + c])) * s[c];
  }
  uint8_t out[MG];
#pragma unroll
  for (int k = 0; k < MG; k++) {
    int ahead = 0;
#pragma unroll
    for (int q = 0; q < MG; q++) ahead += (xi[q] > xi[k] || (xi[q] == xi[k] && q < k)) ? 1 : 0;
    out[k] = ahead < NKEEP ? 1 : 0;
  }
  uint8_t* dst = mask + j * K + g * MG;
  if (MG == 4) {
    *reinterpret_cast<uint32_t*>(dst) = (uint32_t)out[0] | ((uint32_t)out[1] << 8) | ((uint32_t)out[2] << 16) | ((uint32_t)out[3] << 24);
  } else {
#pragma unroll
    for (int k = 0; k < MG; k++) dst[k] = out[k];
  }
}

// The same from the panel (after a block shuffle): mask and, if part is given, the retained metric of every group.
// Workgroup (blk, 64 rows): the rows' values through LDS, a thread takes one group and every (256 / G)-th row; its sums meet in
// ascending order of the row lanes, then the workgroups' in ascending order (k_add_parts).  Where a weight or a score (odd) is
// not finite, the kept metric comes from the network of k_group_values, which passes over NaN; the weights the mask keeps are
// the same sum otherwise.
template <int DT, int NKEEP, int MG>
__global__ void __launch_bounds__(256) k_nm_mask_panel(const uint16_t* __restrict__ P, const double* __restrict__ sp, const int* __restrict__ lp,
                                                        long long N, long long Npad, long long K, int B, uint8_t* __restrict__ mask,
                                                        const int* __restrict__ not_finite, int odd,
                                                        double* __restrict__ part /*[row blocks][K / MG] or null*/) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int G = B / MG, nblk = (int)(K / B), tid = threadIdx.x, blk = (int)(blockIdx.x % (unsigned)nblk);
  const long long rowblk = blockIdx.x / (unsigned)nblk;
  const int stride = B + 2;
  double* s_sum = reinterpret_cast<double*>(smem_raw);                    // [256]
  uint16_t* s_p = reinterpret_cast<uint16_t*>(smem_raw + 256 * 8);        // [64][B + 2]
  const long long j0 = rowblk * 64;
  const int nr = (int)(N - j0 < 64 ? N - j0 : 64);
  const uint32_t* src = reinterpret_cast<const uint32_t*>(P + ((long long)blk * Npad + j0) * B);
  for (int e = tid; e < nr * B / 2; e += 256) {
    const int r = e / (B / 2), c = e - r * (B / 2);
    *reinterpret_cast<uint32_t*>(s_p + r * stride + 2 * c) = src[e];
  }
  const int lanes = 256 / G, g = tid % G, rl = tid / G;
  int col[MG];
  double sc[MG];
#pragma unroll
  for (int k = 0; k < MG; k++) {
    col[k] = lp[blk * B + g * MG + k];
    sc[k] = sp[(long long)blk * B + col[k]];
  }
  const bool network = part && (odd || *not_finite);
  __syncthreads();
  double acc = 0.0;
  if (rl < lanes)
    for (int r = rl; r < nr; r += lanes) {
      double xi[MG];
#pragma unroll
      for (int k = 0; k < MG; k++) xi[k] = (double)esp_to_float<DT>(s_p[r * stride + col[k]]) * sc[k];
      uint32_t out[MG / 4];
#pragma unroll
      for (int h = 0; h < MG / 4; h++) out[h] = 0;
      double kept = 0.0;
#pragma unroll
      for (int k = 0; k < MG; k++) {
        int ahead = 0;
#pragma unroll
        for (int q = 0; q < MG; q++) ahead += (xi[q] > xi[k] || (xi[q] == xi[k] && q < k)) ? 1 : 0;
        out[k / 4] |= (ahead < NKEEP ? 1u : 0u) << (8 * (k % 4));
        kept = kept + (ahead < NKEEP ? xi[k] : 0.0);
      }
      if (network) kept = top_n_sum<NKEEP, MG>(xi);
      acc = acc + kept;
      uint32_t* dst = reinterpret_cast<uint32_t*>(mask + (j0 + r) * K + (long long)blk * B + g * MG);
#pragma unroll
      for (int h = 0; h < MG / 4; h++) dst[h] = out[h];
    }
  if (part) {
    s_sum[tid] = acc;
    __syncthreads();
    if (tid < G) {
      double t = s_sum[tid];
      for (int q = 1; q < lanes; q++) t = t + s_sum[q * G + tid];
      part[rowblk * (K / MG) + (long long)blk * G + tid] = t;
    }
  }
}

__global__ void __launch_bounds__(64) k_add_parts(const double* __restrict__ part, int np, long long n, double* __restrict__ out) {
  const long long e = (long long)blockIdx.x * 64 + threadIdx.x;
  if (e >= n) return;
  double t = part[e];
#pragma unroll 8
  for (int q = 1; q < np; q++) t = t + part[q * n + e];
  out[e] = t;
}

// retained metric of every group under the final order (eq. 5 terms), rows summed in order
template <int DT, int NKEEP, int MG>
__global__ void __launch_bounds__(64) k_group_values(const uint16_t* __restrict__ W, const double* __restrict__ s,
                                                      const int32_t* __restrict__ theta, long long N, long long K,
                                                      double* __restrict__ out) {
  // 4 groups per workgroup, 16 row lanes per group
  const int rl = threadIdx.x & (ROW_LANES - 1);
  const long long g = (long long)blockIdx.x * 4 + (threadIdx.x >> 4);
  const bool active = g < K / MG;
  int c[MG];
  double sc[MG];
#pragma unroll
  for (int k = 0; k < MG; k++) {
    c[k] = active ? theta[g * MG + k] : 0;
    sc[k] = active ? s[c[k]] : 0.0;
  }
  double acc = 0.0;
  if (active) {
    for (long long j = rl; j < N; j += ROW_LANES) {
      double v[MG];
#pragma unroll
      for (int k = 0; k < MG; k++) v[k] = fabs((double)esp_to_float<DT>(W[j * K + c[k]])) * sc[k];
      acc = acc + top_n_sum<NKEEP, MG>(v);
    }
  }
  const double total = lanes_total(acc);
  if (active && rl == 0) out[g] = total;
}

// ------------------------------------------------------------------------------------------------
// host driver: GNS -> LBS -> mask
// ------------------------------------------------------------------------------------------------
#define DISPATCH_DT_NM(dtype, n, KERNEL, ...)                                      \
  do {                                                                             \
    if ((dtype) == ESPARSE_F16 && (n) == 2) KERNEL(ESPARSE_F16, 2, 4, __VA_ARGS__); \
    else if ((dtype) == ESPARSE_F16) KERNEL(ESPARSE_F16, 4, 8, __VA_ARGS__);        \
    else if ((n) == 2) KERNEL(ESPARSE_BF16, 2, 4, __VA_ARGS__);                     \
    else KERNEL(ESPARSE_BF16, 4, 8, __VA_ARGS__);                                   \
  } while (0)

// Whether the scores of calibration features stay on the device, so that nothing comes back to the host before the end: where a score below zero can be
// ruled out (the cheaper table of exchanges needs that), the channels are ranked on the device, and the host is done with the T terms of eq. 1, which it
// makes while the scans run (0.9 ps per token and channel), sooner than it would have the scores from K x bins counts: a term takes it 3 ns, a count
// 1.1 ns, a channel 16 ns on its way, and a look in between 8 us.  Over 512 to 524288 tokens, 64 to 2048 channels, 10 to 256 bins (534 calls, fp16) a call
// takes 1.004 of the faster way's time in the geometric mean, 1.22 at worst (131072 tokens, 256 channels, 256 bins: 243 and 200 us); all scores from the
// host: 1.34 and 4.3, all on the device: 1.10 and 2.9.  By channels alone (768 and more, fewer up to 4096 tokens) 6000 tokens of 640 channels and 256 bins took
// 184 us, 86 on the device, and 32768 of 768 and 10 bins 194, 123 from the host.
bool esp_scores_on_device(long long T, long long K, int bins, bool entropy, bool norm, double alpha) {
  if (K > RANK_ON_DEVICE || (norm && !(alpha >= 0.0))) return false;
  const double wait = threads_us(0.003 * (double)T, host_threads(T, ENTROPY_TERMS)) - 0.9e-6 * (double)T * (double)K;
  return !entropy || wait <= 8.0 + 0.016 * (double)K + threads_us(1.1e-3 * (double)K * bins, host_threads(K * bins, ENTROPY_COUNTS));
}

// Workgroups of a block's team in k_lbs_rounds, 0: a launch per round.  As many as fill the places of an XCD, which takes every eighth block, and
// have a batch of rows for each wave.  A device with fewer compute units is a part of the chip, with fewer XCDs: numbers eight apart are then not on one XCD, and
// its places hold parts of many teams of which none can end.
// One or two teams of the largest size per XCD leave CUs idle that the launches use, three share them unevenly: with many rows for each workgroup launches are
// faster.  Of times with a team over without, 4:8 and 64 columns: 1 to 8 blocks 0.83 - 0.95 at 375 rows, 0.83 - 1.07 at 625, 1.02 - 1.18 at 1000, 1.18 - 1.32 at
// 1500, 1.37 - 1.54 at 2500; 9 and 16 blocks 0.96 and 0.91 at 1000, 1.14 and 1.00 at 1500, 1.40 and 1.04 at 2500.  2:4 and fewer columns: 1 to 8 blocks 0.61 - 1.08 at
// 2500, 1.06 at 3750, 1.13 - 1.48 at 7500; 9 to 16 blocks 0.8 - 1.05 at any number.  17 to 24 blocks of 64 columns 0.96 - 1.00 at 1500, 1.18 at 2500.  More take
// 0.5 - 1.14 (1.16 for 4:8 with 576 blocks of 9216 rows).  Over 561 sizes up to 120000 rows a call takes 1.001 of the faster way's time in the geometric mean;
// always with teams 1.013 and 2.5 at worst.
int esp_lbs_team(long long N, long long nblk, int B, int m, int compute_units) {
  if (B > LBS_TEAM_BLOCK || 2 * compute_units < LBS_XCDS * LBS_XCD_GROUPS) return 0;
  const long long teams = (nblk + LBS_XCDS - 1) / LBS_XCDS, rows = (N + LBS_WAVES * LBS_ROWS - 1) / (LBS_WAVES * LBS_ROWS);
  long long limit = N;
  if (teams == 1) limit = m == 8 && B > 32 ? 850 : 2750;
  else if (B > 32 && (teams == 3 || (teams == 2 && m == 8))) limit = teams == 3 ? 1500 : 1200;
  if (N > limit * LBS_TEAM_MAX) return 0;
  return (int)std::max<long long>(1, std::min(std::min<long long>(LBS_XCD_GROUPS / teams, LBS_TEAM_MAX), rows));
}

// How long the block shuffles of a context wait for a team of workgroups; returns how many of them have given up so far.  (The launches that take over
// then give the same result, which only a wait that is too short shows.)
int esp_team_wait(esparse_ctx* ctx, unsigned long long ticks) {
  ctx->team_wait = ticks;
  return ctx->teams_left;
}

int esp_prune_device(esparse_ctx* ctx, const double* score, const EspCalib* calib, const void* Wv, long long N, long long K, int dtype,
                     const esparse_prune_opts* o, int32_t* perm_out, uint8_t* mask_out, double* score_out, int64_t* swaps_out,
                     double* retained_out) {
  hipStream_t st = ctx->stream;
  const uint16_t* W = reinterpret_cast<const uint16_t*>(Wv);
  const int n = o->n_keep, m = o->m_group;
  const bool use_gns = o->flags & ESPARSE_USE_GNS, use_lbs = o->flags & ESPARSE_USE_LBS;
  const int B = o->block;
  const long long nblk = use_lbs ? K / B : 0;
  if (swaps_out && !use_lbs && o->block > 0 && K % o->block == 0) memset(swaps_out, 0, sizeof(int64_t) * (K / o->block));

  std::vector<double> host_score;
  size_t terms = calib && calib->entropy ? (size_t)calib->T : 0;
  const size_t results = (size_t)(K + 8 + nblk + K / m);
  bool on_device = calib && esp_scores_on_device(calib->T, K, calib->bins, calib->entropy, calib->norm, calib->alpha);
  on_device = on_device && esp_host_stage(ctx, (results + terms) * 8);
  if (!on_device) terms = 0;
  if (calib && !on_device) {
    const int rc = scores_on_host(ctx, *calib, K, dtype, host_score);
    if (rc) return rc;
    score = host_score.data();
    if (score_out) memcpy(score_out, score, (size_t)K * 8);
  }

  // pinned, each part used for one thing: scores, counts, exchanges per block, group values (beyond the largest pinned block
  // from pageable memory), terms of eq. 1
  std::vector<double> pageable;
  Scratch scratch(ctx);
  double* d_s = scratch.get<double>(K);
  double* d_sp = scratch.get<double>(K);
  int32_t* d_theta0 = scratch.get<int32_t>(K);
  double* h_stage = reinterpret_cast<double*>(esp_host_stage(ctx, (results + terms) * 8));
  if (!h_stage) {
    pageable.resize(results);
    h_stage = pageable.data();
  }
  if (!d_s || !d_sp || !d_theta0) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
  if (on_device) {
    const int rc = launch_scores(ctx, scratch, *calib, K, dtype, h_stage + results, d_s);
    if (rc) return rc;
  } else {
    memcpy(h_stage, score, (size_t)K * 8);
    ESP_HIP(ctx, hipMemcpyAsync(d_s, h_stage, (size_t)K * 8, hipMemcpyHostToDevice, st));
  }
  // device scores to the caller, with the results at the end
  auto fetch_scores = [&]() -> int {
    if (on_device && score_out) ESP_HIP(ctx, hipMemcpyAsync(h_stage, d_s, (size_t)K * 8, hipMemcpyDeviceToHost, st));
    return ESPARSE_OK;
  };
  auto leave_scores = [&]() {
    if (on_device && score_out) memcpy(score_out, h_stage, (size_t)K * 8);
  };
  double* h_gv = h_stage + K + 8 + nblk;
  auto leave_retained = [&]() {
    if (!retained_out) return;
    double tot = 0.0;
    for (long long g = 0; g < K / m; g++) tot = tot + h_gv[g];
    *retained_out = tot;
  };

  // ---- global naive shuffle
  double* d_g = nullptr;
  if (use_gns) {
    d_g = scratch.get<double>(K);
    unsigned long long* d_cs = scratch.get<unsigned long long>((size_t)K * AB_NB);
    if (!d_g || !d_cs) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
    ESP_HIP(ctx, hipMemsetAsync(d_cs, 0, (size_t)K * AB_NB * 8, st));
    const long long nchunk = std::max<long long>(1, std::min<long long>(N / 64, 1024 / std::max<long long>(1, (K + 127) / 128) + 1));
    const long long rpb = ((N + nchunk - 1) / nchunk + 7) / 8 * 8;
    dim3 grid((unsigned)((K + 127) / 128), (unsigned)((N + rpb - 1) / rpb));
    if (dtype == ESPARSE_F16)
      hipLaunchKernelGGL(k_abs_colsum<ESPARSE_F16>, grid, dim3(256), 0, st, W, N, K, rpb, d_cs);
    else
      hipLaunchKernelGGL(k_abs_colsum<ESPARSE_BF16>, grid, dim3(256), 0, st, W, N, K, rpb, d_cs);
    ESP_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(k_channel_means, dim3((unsigned)((K + 63) / 64)), dim3(64), 0, st, d_cs, d_s, N, K, d_g);
    ESP_HIP(ctx, hipGetLastError());
  }
  if (use_gns && K > RANK_ON_DEVICE) {
    std::vector<double> g((size_t)K);
    std::vector<int32_t> order((size_t)K), theta0((size_t)K);
    ESP_HIP(ctx, hipMemcpyAsync(g.data(), d_g, (size_t)K * 8, hipMemcpyDeviceToHost, st));
    ESP_HIP(ctx, hipStreamSynchronize(st));
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return g[a] > g[b] || (g[a] == g[a] && g[b] != g[b]); });
    const long long G = K / m;
    for (long long r = 0; r < K; r++) theta0[(size_t)((r % G) * m + r / G)] = order[(size_t)r];
    for (long long p = 0; p < K; p++) g[(size_t)p] = score[theta0[(size_t)p]];
    ESP_HIP(ctx, hipMemcpyAsync(d_theta0, theta0.data(), (size_t)K * 4, hipMemcpyHostToDevice, st));
    ESP_HIP(ctx, hipMemcpyAsync(d_sp, g.data(), (size_t)K * 8, hipMemcpyHostToDevice, st));
    ESP_HIP(ctx, hipStreamSynchronize(st));  // the host copies end here
  } else {
    hipLaunchKernelGGL(k_naive_shuffle, dim3((unsigned)((K + 15) / 16)), dim3(1024), 0, st, d_g, d_s, (int)K, m, use_gns ? 1 : 0, d_theta0, d_sp);
    ESP_HIP(ctx, hipGetLastError());
  }

  // ---- local block shuffle
  if (use_lbs) {
    // columns of a workgroup (16 lanes of qc) and workgroups per block, see k_lbs_eval: rows are split so that two
    // workgroups per CU share the two groups that an exchange touches (at least one batch of rows per wave)
    const int qc = B <= 32 ? 2 : 4;
    const int slices = (B + 16 * qc - 1) / (16 * qc);
    const long long most_splits = (N + LBS_WAVES * LBS_ROWS - 1) / (LBS_WAVES * LBS_ROWS);
    const int nsplit = (int)std::max<long long>(1, std::min<long long>(512 / (nblk * slices), most_splits));
    const int refresh_sets = m == 4 ? 1 : 2;  // k_lbs_refresh: workgroups for the two groups
    const int nsplit_refresh = (int)std::max<long long>(1, std::min<long long>(512 / (nblk * slices * refresh_sets), most_splits));
    int cus = 0;
    ESP_HIP(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    const int team = esp_lbs_team(N, nblk, B, m, cus);
    const long long batch = (long long)std::max(nsplit, team) * LBS_WAVES * LBS_ROWS;  // rows that are read past the panel's end, at most
    const long long Npad = (N + LBS_ROWS - 1) / LBS_ROWS * LBS_ROWS;
    bool finite = true, fast = true;  // of the scores: all finite (on the device: k_build_panel looks); and none negative
    for (long long c = 0; c < K && score; c++) {
      finite = finite && std::isfinite(score[c]);
      fast = fast && score[c] >= 0.0;
    }
    fast = fast && finite;
    const size_t ventries = (size_t)nblk * B * B;
    // the cheaper table looks ahead past the panel's end and needs the panel by columns and its workgroups' sums as well: where
    // the device has no room for them (2 more bytes per weight), the exact table does without
    uint16_t* d_P = scratch.get<uint16_t>((size_t)(Npad * K + (fast ? batch * B : 0)));
    if (!d_P && fast) {
      fast = false;
      d_P = scratch.get<uint16_t>((size_t)(Npad * K));
    }
    double* d_V = scratch.get<double>(ventries);
    int* d_lp = scratch.get<int>(K);
    int* d_rec = scratch.get<int>(nblk * 2 * LBS_REC);
    int* d_state = scratch.get<int>(nblk);
    long long* d_swaps = scratch.get<long long>(nblk);
    int* d_count = scratch.get<int>(4);
    if (!d_P || !d_V || !d_lp || !d_rec || !d_state || !d_swaps || !d_count)
      return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation for the block shuffle failed");
    double* d_S = fast ? scratch.get<double>(ventries * nsplit) : nullptr;
    uint16_t* d_PT = d_S ? scratch.get<uint16_t>((size_t)(Npad * K)) : nullptr;
    fast = d_PT != nullptr;
    const long long meet = 2ll * K * m * team;  // places of the teams' sums, one of three buffers
    unsigned long long* d_meet = fast && team ? scratch.get<unsigned long long>((size_t)(3 * meet)) : nullptr;
    int* count = reinterpret_cast<int*>(h_stage + K);
    long long* h_swaps = reinterpret_cast<long long*>(h_stage + K + 8);
    hipLaunchKernelGGL(k_lbs_init, dim3((unsigned)std::max<long long>((K + 255) / 256, d_meet ? 512 : 0)), dim3(256), 0, st, d_lp, d_state,
                       fast ? LBS_FAST : LBS_EXACT, d_swaps, d_count, d_meet, d_meet ? meet : 0, (int)nblk, B);
    {
      // whole rows of W in LDS: two workgroups per CU where a row leaves the room, else what one workgroup can hold
      const size_t row_bytes = (size_t)K * 2;
      const int RB = (int)std::min<size_t>(16, (row_bytes <= 64 * 1024 ? 64 * 1024 : 144 * 1024) / row_bytes);
      const size_t smem_w = RB * row_bytes;
      if (smem_w > 64 * 1024)
        ESP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_build_panel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_w));
      const long long rows = RB ? RB : 1;
      // a launch has fewer than 2^32 threads (more are cut off without an error): 2^31 at most, in several launches if need be
      for (long long j = 0; j < N; j += rows << 22)
        hipLaunchKernelGGL(k_build_panel, dim3((unsigned)((std::min(N - j, rows << 22) + rows - 1) / rows)), dim3(512), smem_w, st, W, d_theta0,
                           N, Npad, K, j, B, RB, dtype == ESPARSE_F16 ? 0x7c00u : 0x7f80u, d_sp, d_P, d_count + 2);
      ESP_HIP(ctx, hipGetLastError());
    }
    auto panel_columns = [&]() -> int {
      hipLaunchKernelGGL(k_panel_columns, dim3((unsigned)(nblk * ((Npad + 63) / 64)), (unsigned)((B + 63) / 64)), dim3(256), 0, st,
                         d_P, Npad, (int)nblk, B, d_PT);
      ESP_HIP(ctx, hipGetLastError());
      return ESPARSE_OK;
    };
    int rc = fast ? panel_columns() : ESPARSE_OK;
    if (rc) return rc;
    // LDS of the exact evaluation: a chunk of a multiple of 16 rows, about 4096 metric values (at most 16 per thread)
    const int rows_chunk = std::max(16, (4096 / B) / 16 * 16);
    const size_t smem = (size_t)rows_chunk * (B + 1) * 8;
    count[0] = fast ? (int)nblk : 0;
    count[1] = fast ? 0 : (int)nblk;
    // one round of all blocks in the given mode; first: all groups are evaluated
    auto launch_round = [&](int mode, bool first) -> int {
      if (mode == LBS_FAST) {
#define LAUNCH_EVAL(DTv, NK, MGv, QCv)                                                                                              \
  do {                                                                                                                              \
    if (first)                                                                                                                      \
      hipLaunchKernelGGL((k_lbs_eval<DTv, NK, MGv, QCv>), dim3((unsigned)nblk, (unsigned)nsplit, (unsigned)(slices * ((B / MGv + 1) / 2))), \
                         dim3(64 * LBS_WAVES), 0, st, d_P, d_PT, d_sp, N, Npad, B, slices, d_S);                                    \
    else                                                                                                                            \
      hipLaunchKernelGGL((k_lbs_refresh<DTv, NK, MGv, QCv>), dim3((unsigned)nblk, (unsigned)nsplit_refresh, (unsigned)(slices * refresh_sets)), \
                         dim3(64 * LBS_WAVES), 0, st, d_P, d_PT, d_sp, d_rec, N, Npad, B, slices, d_S);                             \
  } while (0)
#define LAUNCH_EVALS(DTv, NK, MGv, ...)           \
  do {                                            \
    if (qc == 4) LAUNCH_EVAL(DTv, NK, MGv, 4);    \
    else LAUNCH_EVAL(DTv, NK, MGv, 2);            \
  } while (0)
        DISPATCH_DT_NM(dtype, n, LAUNCH_EVALS, 0);
#undef LAUNCH_EVALS
#undef LAUNCH_EVAL
      } else {
        const int* rec = first ? nullptr : d_rec;
        if (m == 4 && (B % 64 == 0 || B < 64)) {
          // 2:4: 8 units per workgroup while every group is evaluated, 2 in the refresh rounds (more workgroups)
          const int units = (first ? B / m : 2) * m * (B < 64 ? 1 : B / 64);
          const int nc = first ? 8 : 2;
          dim3 grid((unsigned)((units + nc - 1) / nc), (unsigned)nblk);
          const size_t smem2 = smem + (size_t)rows_chunk * nc * 16;
#define LAUNCH_EXACT24(DTv, NCv)                                                                                             \
  hipLaunchKernelGGL((k_lbs_exact_2_4<DTv, NCv>), grid, dim3(1024), smem2, st, d_P, d_sp, d_lp, \
                     rec, d_state, N, Npad, B, rows_chunk, d_V)
          if (dtype == ESPARSE_F16) {
            if (first) LAUNCH_EXACT24(ESPARSE_F16, 8);
            else LAUNCH_EXACT24(ESPARSE_F16, 2);
          } else {
            if (first) LAUNCH_EXACT24(ESPARSE_BF16, 8);
            else LAUNCH_EXACT24(ESPARSE_BF16, 2);
          }
#undef LAUNCH_EXACT24
        } else {
          dim3 grid((unsigned)(((first ? B / m : 2) * m * B + 63) / 64), (unsigned)nblk);
#define LAUNCH_EXACT(DT, NK, MGv, ...)                                                                                        \
  hipLaunchKernelGGL((k_lbs_exact<DT, NK, MGv>), grid, dim3(1024), smem, st, d_P, d_sp, d_lp, \
                     rec, d_state, N, Npad, B, rows_chunk, d_V)
          DISPATCH_DT_NM(dtype, n, LAUNCH_EXACT, 0);
#undef LAUNCH_EXACT
        }
      }
      ESP_HIP(ctx, hipGetLastError());
#define LAUNCH_SELECT(MGv)                                                                                                     \
  hipLaunchKernelGGL(k_lbs_select<MGv>, dim3((unsigned)nblk), dim3(1024), 0, st, d_S, first ? nsplit : nsplit_refresh, d_V, d_lp, \
                     d_rec, d_state, d_swaps, o->max_swaps, N, B, first ? 1 : 0, mode,  \
                     d_count + 2, d_count)
      if (m == 4) LAUNCH_SELECT(4);
      else LAUNCH_SELECT(8);
#undef LAUNCH_SELECT
      ESP_HIP(ctx, hipGetLastError());
      return ESPARSE_OK;
    };
    // order, mask and retained metric under the order as it is, the counts of blocks that are not done: queued, then waited for
    const long long ng = K / m;
    const int row_blocks = (int)((N + 63) / 64);
    double* d_gv = retained_out ? scratch.get<double>(ng) : nullptr;
    if (retained_out && !d_gv) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
    // the workgroups' sums (8 / m bytes per column and 64 rows) take the place of the panel by columns, which nothing reads any more
    double* d_part = nullptr;
    if (retained_out) d_part = d_PT ? reinterpret_cast<double*>(d_PT) : scratch.get<double>((size_t)row_blocks * ng);
    auto finish = [&]() -> int {
      ESP_HIP(ctx, hipMemcpyAsync(count, d_count, 8, hipMemcpyDeviceToHost, st));
      hipLaunchKernelGGL(k_lbs_final_theta, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, d_theta0, d_lp, B,
                         K, perm_out);
      ESP_HIP(ctx, hipGetLastError());
      if (swaps_out) ESP_HIP(ctx, hipMemcpyAsync(h_swaps, d_swaps, nblk * 8, hipMemcpyDeviceToHost, st));
      const size_t smem_m = 256 * 8 + (size_t)64 * (B + 2) * 2;
      dim3 grid((unsigned)(nblk * row_blocks));
#define LAUNCH_MASK(DT, NK, MGv, ...)                                                                                        \
  hipLaunchKernelGGL((k_nm_mask_panel<DT, NK, MGv>), grid, dim3(256), smem_m, st, d_P, d_sp, d_lp, N, \
                     Npad, K, B, mask_out, d_count + 2, finite ? 0 : 1, d_part)
      DISPATCH_DT_NM(dtype, n, LAUNCH_MASK, 0);
#undef LAUNCH_MASK
      ESP_HIP(ctx, hipGetLastError());
      if (retained_out) {
#define LAUNCH_GV(DT, NK, MGv, ...) \
  hipLaunchKernelGGL((k_group_values<DT, NK, MGv>), dim3((unsigned)((ng + 3) / 4)), dim3(64), 0, st, W, d_s, perm_out, N, K, d_gv)
        if (d_part) hipLaunchKernelGGL(k_add_parts, dim3((unsigned)((ng + 63) / 64)), dim3(64), 0, st, d_part, row_blocks, ng, d_gv);
        else DISPATCH_DT_NM(dtype, n, LAUNCH_GV, 0);
#undef LAUNCH_GV
        ESP_HIP(ctx, hipGetLastError());
        ESP_HIP(ctx, hipMemcpyAsync(h_gv, d_gv, ng * 8, hipMemcpyDeviceToHost, st));
      }
      int rc = fetch_scores();
      if (rc) return rc;
      ESP_HIP(ctx, hipStreamSynchronize(st));
      return ESPARSE_OK;
    };
    bool first_fast = true;
    if (d_meet) {
      // the first round, all others in one launch, and the results behind them, which stand unless a block is left to the exact table
      // or a team gave up waiting
      if ((rc = launch_round(LBS_FAST, true))) return rc;
      first_fast = false;
#define LAUNCH_ROUNDS2(DTv, NK, MGv, QCv)                                                                                             \
  hipLaunchKernelGGL((k_lbs_rounds<DTv, NK, MGv, QCv>), dim3((unsigned)((nblk + 7) / 8 * 8 * team)), dim3(64 * LBS_WAVES), 0, st, d_P, d_PT, d_sp, \
                     d_V, d_lp, d_rec, d_state, d_swaps, o->max_swaps, N, Npad, (int)nblk, B, team, d_meet, d_count + 3, ctx->team_wait, d_count + 2, d_count)
#define LAUNCH_ROUNDS(DTv, NK, MGv, ...)               \
  do {                                                 \
    if (qc == 4) LAUNCH_ROUNDS2(DTv, NK, MGv, 4);      \
    else LAUNCH_ROUNDS2(DTv, NK, MGv, 2);              \
  } while (0)
      DISPATCH_DT_NM(dtype, n, LAUNCH_ROUNDS, 0);
#undef LAUNCH_ROUNDS
#undef LAUNCH_ROUNDS2
      ESP_HIP(ctx, hipGetLastError());
      if ((rc = finish())) return rc;
      if (count[0] > 0) {
        ctx->teams_left++;
        if ((rc = panel_columns())) return rc;  // the results' sums are where it was
      }
    }
    if (!d_meet || count[0] > 0 || count[1] > 0) {
      for (int mode : {LBS_FAST, LBS_EXACT}) {
        int& active = count[mode == LBS_FAST ? 0 : 1];
        bool first = mode == LBS_FAST ? first_fast : true;
        long long iter = 0;
        while (active > 0) {
          // rounds are queued several at a time: a round after the last exchange of every block only finds that (about
          // 5 us), a look at the count from the host costs about 25
          for (int r = 0; r < LBS_ROUNDS_QUEUED; r++) {
            if ((rc = launch_round(mode, first))) return rc;
            first = false;
          }
          iter += LBS_ROUNDS_QUEUED;
          ESP_HIP(ctx, hipMemcpyAsync(count, d_count, 8, hipMemcpyDeviceToHost, st));
          ESP_HIP(ctx, hipStreamSynchronize(st));
          if (active > 0 && iter > (long long)B * B * LBS_ROUNDS_MAX)
            return esp_fail(ctx, ESPARSE_EHIP, "block shuffle did not terminate after %lld rounds", iter);
        }
      }
      if ((rc = finish())) return rc;
    }
    scratch.idle();
    leave_scores();
    if (swaps_out) memcpy(swaps_out, h_swaps, nblk * 8);
    leave_retained();
    return ESPARSE_OK;
  }
  ESP_HIP(ctx, hipMemcpyAsync(perm_out, d_theta0, K * 4, hipMemcpyDeviceToDevice, st));

  // ---- n:m mask under the final order
  {
    dim3 grid((unsigned)((N * (K / m) + 255) / 256));
#define LAUNCH_MASK(DT, NK, MGv, ...) \
  hipLaunchKernelGGL((k_nm_mask<DT, NK, MGv>), grid, dim3(256), 0, st, W, d_s, perm_out, N, K, mask_out)
    DISPATCH_DT_NM(dtype, n, LAUNCH_MASK, 0);
#undef LAUNCH_MASK
    ESP_HIP(ctx, hipGetLastError());
  }
  if (retained_out) {
    const long long ng = K / m;
    double* d_gv = scratch.get<double>(ng);
    if (!d_gv) return esp_fail(ctx, ESPARSE_ENOMEM, "scratch allocation failed");
    dim3 grid((unsigned)((ng + 3) / 4));
#define LAUNCH_GV(DT, NK, MGv, ...) \
  hipLaunchKernelGGL((k_group_values<DT, NK, MGv>), grid, dim3(64), 0, st, W, d_s, perm_out, N, K, d_gv)
    DISPATCH_DT_NM(dtype, n, LAUNCH_GV, 0);
#undef LAUNCH_GV
    ESP_HIP(ctx, hipGetLastError());
    ESP_HIP(ctx, hipMemcpyAsync(h_gv, d_gv, ng * 8, hipMemcpyDeviceToHost, st));
  }
  const int rc = fetch_scores();
  if (rc) return rc;
  ESP_HIP(ctx, hipStreamSynchronize(st));  // the one wait: for scores and group values
  scratch.idle();
  leave_scores();
  leave_retained();
  return ESPARSE_OK;
}
