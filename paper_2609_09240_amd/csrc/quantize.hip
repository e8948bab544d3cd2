// E2M-ATQ group ternarisation (gfx950): the step that produces the planes
// and scales the packed format stores.
//
// Paper: section 4.2 (E2M-ATQ), eqs. 4-6, for the representation of section
// 3, eq. 3.  Per 128-weight group:
//
// * one plane (no stored offset): T0 = +-1 where |w| exceeds 0.75 mean|w|,
//   s0 = <T0, w> / <T0, T0> (the least-squares scale, 0 on an empty
//   support);
// * two planes: mu = mean(w), T0 and s0 from w - mu as above, T1 and s1 from
//   the residual w - mu - s0 T0 the same way, then `iters` sweeps updating
//   mu, s0, s1 in turn with the supports fixed (block coordinate descent on
//   the squared error);
// * for every group, the residual energy ||w - s0 T0||^2 of the one-plane
//   fit, which ranks groups for the second plane;
// * with an offset on every group (the paper's own representation), the
//   one-plane fit also takes mu = mean(w), thresholds w - mu and refines mu
//   and s0; two-plane groups store their mu as the group's offset and 0 as
//   the record's.
//
// Two launches: every group's one-plane fit (and its energy), then the
// two-plane groups alone, one thread per record.  A thread owns one group
// and works in fp64 with every sum taken in index order 0..127 (where a sum is
// exact, as that of 128 fp16 values is, in any order), so each threshold
// decision and each stored value is a deterministic function of the group's
// 128 inputs.  The stored mu, s0, s1 are rounded from fp64 to fp16 once, to
// nearest even.
//
// A group's weights stay in 64 registers, two to a register, and its trits in
// another 64 as fp16 (in LDS, two bytes a read, they cost more than the
// arithmetic).  Waves load whole lines and hand the rows to their lanes
// through LDS, and the trits back.  Products with a trit are exact, so a
// product and the sum it goes into are one fma.

#include "tq_internal.h"

// Products and sums are rounded as written: no fused multiply-add.
#pragma clang fp contract(off)

namespace tq {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int64_t kMaxBlocks = 1 << 16;
constexpr double kThreshold = 0.75;
constexpr int kRowBytes = 128 + 16;   // a lane's row of the exchange buffer: 16 rows cover the LDS banks once

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

// fp64 -> fp16 bits, rounded once to nearest even (overflow to inf, NaN to
// the quiet NaN 0x7E00).
__device__ inline uint16_t f64_to_f16(double d) {
  const uint64_t b = __builtin_bit_cast(uint64_t, d);
  const uint32_t sign = (uint32_t)(b >> 48) & 0x8000u;
  const uint64_t a = b & 0x7FFFFFFFFFFFFFFFull;
  if (a >= 0x7FF0000000000000ull) return (uint16_t)(sign | (a > 0x7FF0000000000000ull ? 0x7E00u : 0x7C00u));
  if (a == 0) return (uint16_t)sign;
  int e = (int)(a >> 52) - 1023;
  uint64_t m = a & 0x000FFFFFFFFFFFFFull;
  if ((a >> 52) == 0) {   // fp64 subnormal: far below the fp16 range
    return (uint16_t)sign;
  }
  m |= 1ull << 52;                      // 53-bit significand, value m * 2^(e - 52)
  const int q = e < -14 ? -24 : e - 10; // fp16 quantum at this magnitude
  const int drop = q - (e - 52);        // significand bits below the quantum
  if (drop > 53) return (uint16_t)sign; // below half the smallest subnormal
  uint64_t sig = m >> drop;
  const uint64_t rem = m & ((1ull << drop) - 1);
  const uint64_t half = 1ull << (drop - 1);
  if (rem > half || (rem == half && (sig & 1))) ++sig;
  uint32_t bits;
  if (q == -24) {
    bits = (uint32_t)sig;               // subnormal (1024 reads as the smallest normal)
  } else {
    bits = ((uint32_t)(e + 15) << 10) + (uint32_t)(sig - 1024);   // sig == 2048 carries into the exponent
  }
  if (bits >= 0x7C00u) bits = 0x7C00u;
  return (uint16_t)(sign | bits);
}

__device__ inline double h2d(uint32_t bits) { return (double)__builtin_bit_cast(_Float16, (uint16_t)bits); }

__device__ inline double ls_ratio(double num, int n) { return n > 0 ? num / (double)n : 0.0; }

// Element i of a row of packed halves.
__device__ __attribute__((always_inline)) inline uint32_t half_bits(const uint32_t (&v)[64], int i) {
  return (v[i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
}
__device__ __attribute__((always_inline)) inline double at(const uint32_t (&v)[64], int i) { return h2d(v[i >> 1] >> (16 * (i & 1))); }

// A pass over a group's elements in index order.  The registers it reads are
// made opaque first, and the scheduler is held to eight elements at a time:
// left alone, the compiler keeps every element's conversion to fp64 from one
// pass to the next (twice the register file) or starts them all at once.
__device__ __attribute__((always_inline)) inline void again(uint32_t (&v)[64]) {
#pragma unroll
  for (int i = 0; i < 64; ++i) asm volatile("" : "+v"(v[i]));
}
// `sum` (and the trits written, where given) end eight elements and begin the
// next eight.
template <typename F>
__device__ __attribute__((always_inline)) inline void each(double& sum, F&& body) {
#pragma unroll
  for (int o = 0; o < kGroup; o += 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) body(o + i);
    asm volatile("" : "+v"(sum));
  }
}
template <typename F>
__device__ __attribute__((always_inline)) inline void each(double& sum, uint32_t (&t)[64], F&& body) {
#pragma unroll
  for (int o = 0; o < kGroup; o += 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) body(o + i);
    asm volatile("" : "+v"(sum), "+v"(t[o / 2]), "+v"(t[o / 2 + 1]), "+v"(t[o / 2 + 2]), "+v"(t[o / 2 + 3]));
  }
}

// Nonzero trits of a group (both 0x3C00 and 0xBC00 have bit 13).
__device__ __attribute__((always_inline)) inline int support(uint32_t (&t)[64]) {
  again(t);
  int n = 0;
#pragma unroll
  for (int i = 0; i < 64; ++i) n += __builtin_popcount(t[i] & 0x20002000u);
  return n;
}

// The wave's rows: lane l gets the 256 bytes at `base` of group f, which it
// names (any lane may name any group).  Every load instruction takes eight
// half rows, whole lines each.
__device__ __attribute__((always_inline)) inline void load_rows(uint32_t (&v)[64], const uint16_t* __restrict__ w,
                                                                int64_t f, unsigned char* lds, int lane) {
  u4v in[2][8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t r = __shfl(f, 8 * j + (lane >> 3));
    const unsigned char* src = reinterpret_cast<const unsigned char*>(w + r * kGroup) + 16 * (lane & 7);
    in[0][j] = *reinterpret_cast<const u4v*>(src);
    in[1][j] = *reinterpret_cast<const u4v*>(src + 128);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      *reinterpret_cast<u4v*>(lds + (8 * j + (lane >> 3)) * kRowBytes + 16 * (lane & 7)) = in[h][j];
    __builtin_amdgcn_wave_barrier();   // (a wave's LDS accesses complete in order)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const u4v x = *reinterpret_cast<const u4v*>(lds + lane * kRowBytes + 16 * j);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[32 * h + 4 * j + k] = x[k];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Trits as int8 to row r of `out`, which the lane names (r < 0: not stored),
// whole lines again.  kFp16: they come as fp16 bits (+1 = 0x3C00, -1 = 0xBC00,
// 0), else as 16-bit integers.
template <bool kFp16>
__device__ __attribute__((always_inline)) inline void store_trits(int8_t* __restrict__ out, const uint32_t (&t)[64],
                                                                  int64_t r, unsigned char* lds, int lane) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    u4v x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t lo = t[8 * c + 2 * k], hi = t[8 * c + 2 * k + 1];
      if constexpr (kFp16) {
        // Bytes 1 and 3 of the words: 0x3C, 0xBC or 0.  0x3C -> 0x01: bit 2
        // moved to bit 0; 0xBC -> 0xFF: every bit set by the sign.
        const uint32_t b = __builtin_amdgcn_perm(hi, lo, 0x07050301u);
        const uint32_t one = (b >> 2) & 0x01010101u, neg = (b >> 7) & 0x01010101u;
        x[k] = one | (neg * 0xFFu);
      } else {
        x[k] = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
      }
    }
    *reinterpret_cast<u4v*>(lds + lane * kRowBytes + 16 * c) = x;
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const u4v x = *reinterpret_cast<const u4v*>(lds + (8 * j + (lane >> 3)) * kRowBytes + 16 * (lane & 7));
    const int64_t to = __shfl(r, 8 * j + (lane >> 3));
    if (to >= 0) *reinterpret_cast<u4v*>(out + to * kGroup + 16 * (lane & 7)) = x;
  }
  __builtin_amdgcn_wave_barrier();
}

// Trits of v > delta (+1), v < -delta (-1) as fp16 bits.
__device__ inline uint32_t trit_bits(double v, double delta) {
  const uint32_t sign = (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 48) & 0x8000u;
  return fabs(v) > delta ? 0x3C00u | sign : 0u;
}

// The largest fp16 not above d (d >= 0; NaN gives bits above every number):
// an fp16 magnitude is above d exactly where its bits are above these.
__device__ inline uint32_t floor_half(double d) {
  if (d != d) return 0x7FFFu;
  const auto c = __builtin_amdgcn_cvt_pkrtz((float)d, 0.0f);   // (float)d may have been rounded up past an fp16
  const uint32_t b = __builtin_bit_cast(uint32_t, c) & 0xFFFFu;
  return h2d(b) > d ? b - 1u : b;
}

// Pass 1, every group: the one-plane fit and its residual energy.  Two-plane
// groups are stored too (pass 2 stores them again) and leave their index in
// the first 8 bytes of their record's t1 row, which pass 2 reads and then
// overwrites, so pass 2 can run over the records alone (no wave then mixes
// the two fits).  kOff: with an offset on every group.
template <bool kOff>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 3))) one_plane_kernel(const uint16_t* __restrict__ w, int64_t n,
                                                             const int32_t* __restrict__ rec_index, int64_t nnz,
                                                             int iters, int8_t* __restrict__ t0_out,
                                                             uint16_t* __restrict__ s0_out, int8_t* __restrict__ t1_out,
                                                             uint16_t* __restrict__ off0_out,
                                                             double* __restrict__ energy_out) {
  __shared__ __attribute__((aligned(16))) unsigned char rows[kWaves][64 * kRowBytes];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned char* lds = rows[wave];
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  // Waves share no LDS data, so no workgroup barrier is needed.
  for (int64_t base = (int64_t)blockIdx.x * kThreads + 64 * wave; base < n; base += stride) {
    const bool have = base + lane < n;
    const int64_t f = have ? base + lane : n - 1;
    uint32_t x[64], t[64];
    load_rows(x, w, f, lds, lane);
    int64_t k = rec_index != nullptr ? (int64_t)rec_index[f] : -1;
    double mu = 0.0, s0, e = 0.0;
    if constexpr (!kOff) {
      // The raw weights are thresholded.  Their sums are exact in fp64 (47
      // bits), and the sign of a weight is that of its trit: magnitudes do.
      double sabs = 0.0;
      again(x);
      each(sabs, [&](int i) { sabs = sabs + fabs(at(x, i)); });
      const uint32_t thr = floor_half(kThreshold * (sabs / kGroup));
      // Two weights at a time in 16-bit arithmetic: m is 1 where the magnitude
      // is above the threshold, m times the magnitude goes into the sum and m
      // times the sign is the trit (a 12288x4096 matrix: 46 us, with energies;
      // with a compare and selects for each weight 52).
      const u16x2 thr2 = {(uint16_t)thr, (uint16_t)thr};
      // Opaque, or the compiler turns min() back into compares and selects.
      u16x2 one = {1, 1};
      asm("" : "+v"(one));
      u16x2 count = {0, 0};
      double num = 0.0;
      again(x);
      each(num, t, [&](int i) {
        if (i & 1) return;
        const u16x2 mag = __builtin_bit_cast(u16x2, x[i >> 1] & 0x7FFF7FFFu);
        const u16x2 m = __builtin_elementwise_min(__builtin_elementwise_sub_sat(mag, thr2), one);
        count += m;
        const uint32_t kept = __builtin_bit_cast(uint32_t, (u16x2)(mag * m));
        num = num + h2d(kept);
        num = num + h2d(kept >> 16);
        const u16x2 sign = __builtin_bit_cast(u16x2, (i16x2)(__builtin_bit_cast(i16x2, x[i >> 1]) >> 15)) | one;
        t[i >> 1] = __builtin_bit_cast(uint32_t, (u16x2)(m * sign));
      });
      s0 = ls_ratio(num, (int)count.x + (int)count.y);
      if (energy_out != nullptr) {
        again(x);
        again(t);
        each(e, [&](int i) {
          const double d = fabs(at(x, i)) - (half_bits(t, i) != 0u ? s0 : 0.0);
          e = e + d * d;
        });
      }
    } else {
      double sw = 0.0;   // exact in any order
      again(x);
      each(sw, [&](int i) { sw = sw + at(x, i); });
      mu = sw / kGroup;
      const double mu_c = mu;
      double sabs = 0.0;
      again(x);
      each(sabs, [&](int i) { sabs = sabs + fabs(at(x, i) - mu_c); });
      const double delta = kThreshold * (sabs / kGroup);
      double num = 0.0;
      again(x);
      each(num, t, [&](int i) {
        const double v = at(x, i) - mu_c;
        const uint32_t b = trit_bits(v, delta);
        if (i & 1) t[i >> 1] |= b << 16;
        else t[i >> 1] = b;
        num = num + (b != 0u ? fabs(v) : 0.0);
      });
      const int n_one = support(t);
      s0 = ls_ratio(num, n_one);
      for (int it = 0; it < iters; ++it) {
        double a = 0.0;
        again(x);
        again(t);
        each(a, [&](int i) { a = a + __builtin_fma(-s0, at(t, i), at(x, i)); });
        mu = a / kGroup;
        double b = 0.0;
        again(x);
        again(t);
        each(b, [&](int i) { b = __builtin_fma(at(t, i), at(x, i) - mu, b); });
        s0 = ls_ratio(b, n_one);
      }
      if (energy_out != nullptr) {
        again(x);
        again(t);
        each(e, [&](int i) {
          const double d = __builtin_fma(-s0, at(t, i), at(x, i) - mu);
          e = e + d * d;
        });
      }
    }
    store_trits<kOff>(t0_out, t, have ? f : -1, lds, lane);
    if (have) {
      s0_out[f] = f64_to_f16(s0);
      if constexpr (kOff) off0_out[f] = f64_to_f16(mu);
      if (energy_out != nullptr) energy_out[f] = e;
      if (k >= 0 && k < nnz) *reinterpret_cast<int64_t*>(t1_out + k * kGroup) = f;
    }
  }
}

// Pass 2, one thread per record: the two-plane fit of the group that named
// it (a record no group names, or one named twice, is skipped).
// One wave a workgroup: 10 % of a 12288x4096 matrix are 615 waves for 1024 SIMDs.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) two_plane_kernel(const uint16_t* __restrict__ w, int64_t n,
                                                             const int32_t* __restrict__ rec_index, int64_t nnz,
                                                             int iters, int8_t* __restrict__ t0_out,
                                                             uint16_t* __restrict__ s0_out, int8_t* __restrict__ t1_out,
                                                             uint16_t* __restrict__ mu_out, uint16_t* __restrict__ s1_out,
                                                             uint16_t* __restrict__ off0_out) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[64 * kRowBytes];
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * 64;
  for (int64_t base = (int64_t)blockIdx.x * 64; base < nnz; base += stride) {
    const int64_t k = base + lane < nnz ? base + lane : nnz - 1;
    int64_t f = *reinterpret_cast<const int64_t*>(t1_out + k * kGroup);
    bool have = base + lane < nnz && f >= 0 && f < n;
    f = f >= 0 && f < n ? f : 0;
    have = have && (int64_t)rec_index[f] == k;
    uint32_t x[64], t0[64], t1[64];
    load_rows(x, w, f, lds, lane);

    // Offset, centred first support, residual second support.
    double sw = 0.0;   // exact in any order
    again(x);
    each(sw, [&](int i) { sw = sw + at(x, i); });
    double mu = sw / kGroup;
    const double mu_c = mu;
    double sc = 0.0;
    again(x);
    each(sc, [&](int i) { sc = sc + fabs(at(x, i) - mu_c); });
    const double delta0 = kThreshold * (sc / kGroup);
    double n0 = 0.0;
    again(x);
    each(n0, t0, [&](int i) {
      const double v = at(x, i) - mu_c;
      const uint32_t b = trit_bits(v, delta0);
      if (i & 1) t0[i >> 1] |= b << 16;
      else t0[i >> 1] = b;
      n0 = n0 + (b != 0u ? fabs(v) : 0.0);
    });
    const int c0 = support(t0);
    double s0 = ls_ratio(n0, c0);
    const double s0_c = s0;
    double sr = 0.0;
    again(x);
    again(t0);
    each(sr, [&](int i) { sr = sr + fabs(__builtin_fma(-s0_c, at(t0, i), at(x, i) - mu_c)); });
    const double delta1 = kThreshold * (sr / kGroup);
    double n1 = 0.0;
    again(x);
    again(t0);
    each(n1, t1, [&](int i) {
      const double v = __builtin_fma(-s0_c, at(t0, i), at(x, i) - mu_c);
      const uint32_t b = trit_bits(v, delta1);
      if (i & 1) t1[i >> 1] |= b << 16;
      else t1[i >> 1] = b;
      n1 = n1 + (b != 0u ? fabs(v) : 0.0);
    });
    const int c1 = support(t1);
    double s1 = ls_ratio(n1, c1);
    // Refinement with the supports fixed.
    for (int it = 0; it < iters; ++it) {
      double a = 0.0;
      again(x);
      again(t0);
      again(t1);
      each(a, [&](int i) { a = a + __builtin_fma(-s1, at(t1, i), __builtin_fma(-s0, at(t0, i), at(x, i))); });
      mu = a / kGroup;
      double b = 0.0;
      again(x);
      again(t0);
      again(t1);
      each(b, [&](int i) { b = __builtin_fma(at(t0, i), __builtin_fma(-s1, at(t1, i), at(x, i) - mu), b); });
      s0 = ls_ratio(b, c0);
      double c = 0.0;
      again(x);
      again(t0);
      again(t1);
      each(c, [&](int i) { c = __builtin_fma(at(t1, i), __builtin_fma(-s0, at(t0, i), at(x, i) - mu), c); });
      s1 = ls_ratio(c, c1);
    }
    store_trits<true>(t0_out, t0, have ? f : -1, lds, lane);
    store_trits<true>(t1_out, t1, have ? k : -1, lds, lane);
    if (have) {
      s0_out[f] = f64_to_f16(s0);
      if (off0_out != nullptr) {   // the offset belongs to the group; the record's is 0
        off0_out[f] = f64_to_f16(mu);
        mu_out[k] = 0;
      } else {
        mu_out[k] = f64_to_f16(mu);
      }
      s1_out[k] = f64_to_f16(s1);
    }
  }
}

}  // namespace

hipError_t launch_ternarize(const uint16_t* w, int64_t n, const int32_t* rec_index, int64_t nnz, int iters,
                            int8_t* t0, uint16_t* s0, int8_t* t1, uint16_t* mu, uint16_t* s1, uint16_t* off0,
                            double* energy, hipStream_t s) {
  auto blocks_for = [](int64_t work, int threads) {
    const int64_t b = (work + threads - 1) / threads;
    return (unsigned)(b < 1 ? 1 : (b > kMaxBlocks ? kMaxBlocks : b));
  };
  const bool two = rec_index != nullptr && nnz > 0;
  const auto one = off0 != nullptr ? one_plane_kernel<true> : one_plane_kernel<false>;
  hipLaunchKernelGGL(one, dim3(blocks_for(n, kThreads)), dim3(kThreads), 0, s, w, n, two ? rec_index : nullptr,
                     two ? nnz : 0, iters, t0, s0, t1, off0, energy);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !two) return e;
  hipLaunchKernelGGL(two_plane_kernel, dim3(blocks_for(nnz, 64)), dim3(64), 0, s, w, n, rec_index, nnz, iters, t0, s0,
                     t1, mu, s1, off0);
  return hipGetLastError();
}

}  // namespace tq
