// Small-batch packed GEMM Y = X W^T with MFMA (gfx950).
//
// Paper: section 3, eq. 3 (the weight), section 18 (kernel work across
// shapes and batch sizes is the stated next step).  For a batch of B
// activation rows the product is a dense contraction, so it runs on
// v_mfma_f32_16x16x32_f16: A = 16 batch rows, B = 16 weight rows, C = the
// 16 x 16 block of Y.
//
// k order.  MFMA sums over k in any order, so a group's 128 inputs are laid
// on the four lane blocks (lanes 16q .. 16q+15) by whole code bytes: block
// q < 3 takes code bytes 8q .. 8q+7 (40 trits, inputs 40q .. 40q+39), block 3
// the two tail bytes (inputs 120 .. 127); its other inputs read as zeros.
// The 40 trits are five windows of 8, one per MFMA, so every lane decodes
// its 8 bytes with the same code, and the X operand of window u is the
// aligned 16-byte chunk of X at input 40q + 8u.  (Five k-steps for 128
// inputs, four would be the minimum; in exchange a step holds one group.)
//
// Decode.  A table in LDS maps a code to the high bytes of its five fp16
// trits (+1 = 0x3C00, 0, -1 = 0xBC00) in 8 bytes; a pair of trits is one
// v_perm of two entries.  The weights of the operand are the bare trits: as
// every MFMA of an accumulator belongs to one group, s0 multiplies the
// group's fp32 sums, four per 16 x 16 block and lane, instead of every
// weight, and no weight is rounded to fp16.  A lane's four sums belong to
// the weight row it decoded, so its scale, offset and record are its own.
// Offsets multiply the group's sum of x, one more tile with ones as weights.
//
// Plane 1.  The workgroup's records are staged in LDS by (group, row % 16):
// a group's records are decoded as one more row tile whose row n holds a
// record of one of the weight rows n, n + 16, ..., and s1 times its sums is
// added to the totals of that row, which are in the same lane.  Rows that
// share n and both have a record take one more pass each (10 % two-plane
// groups and three row tiles: 1.4 passes a group, where decoding plane 1
// along with every row tile under a per-lane branch cost as much as three).
//
// Work split.  A workgroup of 8 waves owns 16 RT consecutive rows and the
// waves take the groups in turn, each wave all row tiles and all batch
// columns of its group, so every weight is decoded once and a CU reads X
// once.  A wave streams the codes of its groups through registers, kRing
// groups ahead, without waiting for the other waves; tails, scales and
// records are staged in LDS, for chunks of groups where a row is too long.
// The waves' partial sums are added in a fixed order through LDS
// (bit-reproducible).
//
// What bounds it: instruction issue (about three quarters of the slots, two
// waves a SIMD), and below 8 us the set-up of a launch.  Graph-timed, weights
// from HBM, 10 % two-plane groups, before (quads of groups, s0 and s1 put into
// fp16 weights, plane 1 under a per-lane branch) and now:
//   12288 x 4096  B = 16 15.8 -> 12.3 us, B = 32 20.7 -> 16.6, B = 64 28.0 -> 26.1
//   4096 x 12288  B = 4 14.8 -> 12.9, B = 16 18.9 -> 14.6, B = 64 54.0 -> 34.9
//   4096 x 4096   B = 16 8.7 -> 7.8, B = 64 22.9 -> 13.3
//   4096 x 20480  B = 16 928 -> 20.7 (a kernel of its own for a long K before)
// A ring of 4 to 12 groups is slower (13.1 us at 12288 x 4096, B = 16): the
// unrolled code no longer fits the instruction cache.

#include "tq_internal.h"

namespace tq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));

constexpr int kCus = 256;
constexpr int kLdsLimit = 160 * 1024;
constexpr int kWaves = 8;                            // two per SIMD
constexpr int kThreads = 64 * kWaves;
constexpr int kRing = 2;                             // groups of a wave whose codes are in registers or in flight
constexpr int kLutCopies = 32;                       // 8-byte entries: 32 lanes cover the 64 banks once
constexpr int kLutBytes = 256 * kLutCopies * 8;      // 64 KiB
constexpr int kMaxPairs = 1536;                      // (row, group) pairs staged at a time
constexpr int kMaxRanges = 640;                      // workgroups with record ranges in the kernel arguments
constexpr uint32_t kOnes = 0x3C003C00u;

// Arguments behind the leading ones, which arrive in SGPRs.
struct TileArgs {
  const uint16_t* offset0;
  const uint8_t* codes1;
  const uint16_t* gidx1;
  const uint16_t* offset1;
  const uint16_t* scale1;
  void* Y;
  // With ranges from the host row pointers: the first record of every
  // workgroup, then nnz1, so record loads need no dependent load.
  int32_t rec_begin[kMaxRanges + 1];
};

// All arguments as a launch lays them out.
struct KernelArgs {
  const uint8_t* codes0;
  const uint16_t* scale0;
  const uint16_t* X;
  const int32_t* rowptr1;
  int32_t n_out, G, B, opts, nnz1;
  TileArgs a;
};

// Dynamic LDS of a workgroup of R = 16 RT rows, NW waves and a chunk of C
// groups (byte offsets): per wave 16 rows of a group of X, with 16 bytes
// between rows so that one 16-byte read's 16 rows cover the banks; 64 zero
// bytes; the 32-byte record slots [group][pass][16] (code bytes 0..23, tail,
// row tile, s1 | mu << 16); a byte per (group, row % 16) with its number of
// records; per row and group the words tail | s0 << 16 and offset, with an odd
// row stride so that 16 rows spread over the banks.  After the main loop
// the partial sums [waves][RT][CT][64 lanes] x 16 B overlay it.
constexpr int kXRow = 2 * kGroup + 16;
__host__ __device__ constexpr int tile_stride(int C) { return C | 1; }
__host__ __device__ constexpr int tile_zero_off(int NW) { return NW * 16 * kXRow; }
__host__ __device__ constexpr int tile_slot_off(int NW) { return tile_zero_off(NW) + 64; }
__host__ __device__ constexpr int tile_count_off(int NW, int R, int C) { return tile_slot_off(NW) + 32 * R * C; }
__host__ __device__ constexpr int tile_word_off(int NW, int R, int C) { return tile_count_off(NW, R, C) + 16 * C; }
__host__ __device__ constexpr int tile_lds(int NW, int R, int C) {
  return tile_word_off(NW, R, C) + 8 * R * tile_stride(C);
}
__host__ __device__ constexpr int tile_red_bytes(int NW, int RT, int CT) { return NW * RT * CT * 64 * 16; }
static_assert(kLutBytes + tile_lds(kWaves, 16, 96) <= kLdsLimit && kLutBytes + tile_lds(kWaves, 32, 48) <= kLdsLimit &&
                  kLutBytes + tile_lds(kWaves, 48, 32) <= kLdsLimit && kLutBytes + tile_lds(kWaves, 64, 24) <= kLdsLimit,
              "a full chunk fits");

__device__ inline float h2f(uint32_t b) { return (float)__builtin_bit_cast(_Float16, (uint16_t)b); }
__device__ inline uint32_t f2h(float a) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a); }

// Table entry of code c: the high bytes of the fp16 patterns of t0..t3 and,
// in the second dword, t4; codes 243..255 read as zeros.
__device__ inline u2v table_entry(int c) {
  uint32_t t[5];
  uint32_t d = (uint32_t)c;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const uint32_t qd = (d * 171u) >> 9;   // d / 3 for d < 256
    const uint32_t u = d - 3u * qd;
    t[i] = c >= 243 || u == 1u ? 0u : (u == 2u ? 0x3Cu : 0xBCu);
    d = qd;
  }
  return u2v{t[0] | (t[1] << 8) | (t[2] << 16) | (t[3] << 24), t[4]};
}

// LDS byte address of this lane's table copy for byte BY of dword w:
// bytes [slot, code, 0, 0].
template <int BY>
__device__ inline uint32_t lut_addr(uint32_t w, uint32_t slot) {
  return __builtin_amdgcn_perm(slot, w, 0x0C0C0004u | (BY << 8));
}

// Table entries of a lane's 8 code bytes.
__device__ __attribute__((always_inline)) inline void read_entries(const unsigned char* lut, uint32_t slot, u2v w,
                                                                   u2v (&e)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t x = h ? w.y : w.x;
    e[4 * h] = *reinterpret_cast<const u2v*>(lut + lut_addr<0>(x, slot));
    e[4 * h + 1] = *reinterpret_cast<const u2v*>(lut + lut_addr<1>(x, slot));
    e[4 * h + 2] = *reinterpret_cast<const u2v*>(lut + lut_addr<2>(x, slot));
    e[4 * h + 3] = *reinterpret_cast<const u2v*>(lut + lut_addr<3>(x, slot));
  }
}

// The operands of the five windows (8 trits each) from the entries.
__device__ __attribute__((always_inline)) inline void expand(const u2v (&e)[8], u4v (&W)[5]) {
  uint32_t d[20];
#pragma unroll
  for (int p = 0; p < 4; ++p) {   // two bytes: ten trits, five dwords
    const u2v a = e[2 * p], b = e[2 * p + 1];
    d[5 * p] = __builtin_amdgcn_perm(a.x, a.x, 0x010C000Cu);       // t0 t1
    d[5 * p + 1] = __builtin_amdgcn_perm(a.x, a.x, 0x030C020Cu);   // t2 t3
    d[5 * p + 2] = __builtin_amdgcn_perm(b.x, a.y, 0x040C000Cu);   // t4 t0'
    d[5 * p + 3] = __builtin_amdgcn_perm(b.x, b.x, 0x020C010Cu);   // t1' t2'
    d[5 * p + 4] = __builtin_amdgcn_perm(b.y, b.x, 0x040C030Cu);   // t3' t4'
  }
#pragma unroll
  for (int u = 0; u < 5; ++u) W[u] = u4v{d[4 * u], d[4 * u + 1], d[4 * u + 2], d[4 * u + 3]};
}

__device__ __attribute__((always_inline)) inline float4v mfma(u4v a, u4v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// Holds MFMA results back until they can be read anywhere.  The compiler puts
// wait states between an MFMA and the first read of its result (8 for
// v_mfma_f32_16x16x32_f16: `s_nop 7` in straight code), but where a branch lies
// between the two it can count those of the longer way round only (seen on an
// `if` directly behind a chain: the first of the four sums was read too early).
// So it belongs between the last MFMA of a chain and every branch whose sides
// read what the chain wrote, with all accumulators that may still be in
// flight; where no branch lies between, nothing is needed.  Its 16 wait states
// are twice this instruction's; one of 16 passes (32 x 32 tiles) wants more.
__device__ __attribute__((always_inline)) inline void settle(float4v& a, float4v& b) {
  asm volatile("s_nop 15" : "+v"(a), "+v"(b));
}

// Workgroup barrier for LDS data only: waits for this wave's LDS accesses
// but leaves its global loads in flight (a plain __syncthreads waits for
// those too).
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS at a byte address: the address of a loop's next access is then one
// register with the offset in the instruction (a pointer into the dynamic
// block, which starts behind the table, costs an add per access).
template <typename V>
__device__ __attribute__((always_inline)) inline V lds_read(uint32_t at) {
  return *reinterpret_cast<const __attribute__((address_space(3))) V*>(at);
}
__device__ __attribute__((always_inline)) inline uint32_t lds_address(const void* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p);
}

// A value the compiler knows nothing about: what depends on it is computed
// here, and not ahead of the loop over chunks, where all of it would be done
// before the first load and held in registers.
__device__ inline int here_v(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ inline int here_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// One plane-1 record as loaded: code bytes 0..23, bytes 24, 25, s1 | mu << 16, group.
struct RecLoad {
  uint64_t v0, v1, v2;
  uint32_t tl, sm;
  int gg;
};

// Record k (0 <= k < nnz1).
__device__ inline RecLoad load_record(const TileArgs& a, int nnz1, int k) {
  const uint32_t n = (uint32_t)nnz1, kk = (uint32_t)k;
  const uint64_t* rm = reinterpret_cast<const uint64_t*>(a.codes1 + (size_t)(24u * kk));
  RecLoad r;
  r.v0 = rm[0];
  r.v1 = rm[1];
  r.v2 = rm[2];
  r.tl = *reinterpret_cast<const uint16_t*>(a.codes1 + (size_t)(24u * n + 2u * kk));
  r.sm = (uint32_t)a.scale1[kk] | ((uint32_t)a.offset1[kk] << 16);
  r.gg = (int)a.gidx1[kk];
  return r;
}

__device__ inline bool not_finite(float a) { return (__builtin_bit_cast(uint32_t, a) & 0x7F800000u) == 0x7F800000u; }

// The arguments where the launch put them, through a pointer the compiler
// knows nothing about: their loads are not done ahead of a rare branch, and
// nothing of them is held through the main loop.
typedef const __attribute__((address_space(4))) KernelArgs* ArgsPtr;
__device__ __attribute__((always_inline)) inline ArgsPtr launch_args() {
  ArgsPtr p = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// What a quarter of group g of a row (code bytes 7 quarter ..) adds to the
// row's output, weight by weight in tq_unpack_fp16's order.  k0, k1: the row's
// records; x: the inputs of the batch row.
template <bool kRec>
__device__ __attribute__((always_inline)) inline float quarter_sum(ArgsPtr p, int row, int g, int quarter, int k0, int k1,
                                                                   const uint16_t* x) {
  const uint32_t n0 = (uint32_t)p->n_out * (uint32_t)p->G, n1 = (uint32_t)p->nnz1;
  const uint32_t f = (uint32_t)row * (uint32_t)p->G + (uint32_t)g;
  const float s0 = h2f(p->scale0[(size_t)f]);
  float mu = p->a.offset0 != nullptr ? h2f(p->a.offset0[(size_t)f]) : 0.f, s1 = 0.f;
  bool two = false;
  if constexpr (kRec) {
    const int end = k1;
    while (k0 < k1) {   // the first record at or behind g
      const int mid = (k0 + k1) >> 1;
      if ((int)p->a.gidx1[mid] < g) k0 = mid + 1;
      else k1 = mid;
    }
    two = k0 < end && (int)p->a.gidx1[k0] == g;
    if (two) {
      mu = mu + h2f(p->a.offset1[k0]);
      s1 = h2f(p->a.scale1[k0]);
    }
  }
  float sum = 0.f;
  for (uint32_t j = 7u * (uint32_t)quarter; j < min(7u * (uint32_t)quarter + 7u, (uint32_t)kGroupBytes); ++j) {
    int c0 = p->codes0[j < 24u ? (size_t)(24u * f + j) : (size_t)(24u * n0 + 2u * f + (j - 24u))], c1 = 121;
    if constexpr (kRec) {
      const uint32_t k = (uint32_t)k0;
      if (two) c1 = p->a.codes1[j < 24u ? (size_t)(24u * k + j) : (size_t)(24u * n1 + 2u * k + (j - 24u))];
    }
    c0 = c0 > 242 ? 121 : c0;   // (invalid codes read as zeros)
    c1 = c1 > 242 ? 121 : c1;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const int at = 5 * (int)j + i;
      float w = mu + s0 * (float)(c0 % 3 - 1);
      if (two) w = w + s1 * (float)(c1 % 3 - 1);
      if (at < kGroup) sum = sum + w * h2f(x[kGroup * g + at]);
      c0 /= 3;
      c1 /= 3;
    }
  }
  return sum;
}

// Outputs of a wave's 16 x 16 tile whose sums are not finite, by the
// definition.  The sums of trits' products say which outputs those are, but
// not what they are: an infinite input under a zero trit puts 0 * inf into its
// group's sum, also where an offset gives the weight a value, and a scale that
// is not finite meets the group's sum and not each of its weights.  So the
// weights are formed one by one, in the groups where the batch row holds a
// value that is not finite (the others add a finite number, which changes
// nothing; with a scale or offset that is not finite in the tile's rows, in
// every group).  Lanes n, n + 16, n + 32 and n + 48 share weight row n.  Finite
// inputs and scales never come here (no sum of theirs leaves the range of
// fp32).  One infinity in a row of X: 12288 x 4096, B = 16, 14.3 -> 25.6 us;
// one in each of 64 rows of X, 27 -> 291 (a lane that reads its output's whole
// row alone takes 269 and 675).  The check costs a call 0.09 us, 0.6 % over
// 960 shapes.  row0, nrows: the tile's weight rows; b0: its first batch row;
// s: the lane's four sums; store(b, y): an output of the lane's weight row.
template <bool kRec, typename Store>
__device__ __attribute__((always_inline)) inline void redo_tile(int row0, int nrows, int b0, float4v s, const Store& store) {
  const ArgsPtr p = launch_args();
  const int G = p->G, lane = (int)__lane_id(), n = lane & 15, q = lane >> 4;
  const int row = row0 + min(n, nrows - 1);
  int k0 = 0, k1 = 0, every = -1;   // (every: not known yet)
  if constexpr (kRec) {   // in bounds whatever the row pointers hold
    k0 = max(0, min(p->rowptr1[row], p->nnz1));
    k1 = max(0, min(p->rowptr1[row + 1], p->nnz1));
  }
#pragma unroll 1
  for (int j = 0; j < min(16, p->B - b0); ++j) {
    const float y = (j & 2) ? ((j & 1) ? s[3] : s[2]) : ((j & 1) ? s[1] : s[0]);
    if (__ballot(q == j >> 2 && n < nrows && not_finite(y)) == 0) continue;
    if (every < 0) {
      bool bad = false;
#pragma unroll 4
      for (int g = q; g < G; g += 4) {
        const size_t f = (size_t)((uint32_t)row * (uint32_t)G + (uint32_t)g);
        bad |= not_finite(h2f(p->scale0[f]));
        if (p->a.offset0 != nullptr) bad |= not_finite(h2f(p->a.offset0[f]));
      }
      if constexpr (kRec) {
#pragma unroll 4
        for (int k = k0 + q; k < k1; k += 4) bad |= not_finite(h2f(p->a.offset1[k])) || not_finite(h2f(p->a.scale1[k]));
      }
      every = __ballot(bad) != 0;
    }
    const uint16_t* x = p->X + (int64_t)(b0 + j) * G * kGroup;
    float sum = 0.f;
    bool known = false;   // every row's output is NaN
#pragma unroll 1
    for (int g0 = 0; g0 < G && !known; g0 += 16) {   // lanes 16 i .. hold the inputs of groups g0 + 4 t + i
      u4v v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        v[t] = *reinterpret_cast<const u4v*>(x + kGroup * min(g0 + 4 * t + q, G - 1) + 8 * n);
#pragma unroll 1
      for (int t = 0; t < 4 && !known; ++t) {
        const u4v u = t == 0 ? v[0] : (t == 1 ? v[1] : (t == 2 ? v[2] : v[3]));
        bool bad = every != 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) bad |= (u[i] & 0x7C00u) == 0x7C00u || (u[i] & 0x7C000000u) == 0x7C000000u;
        const uint64_t m = __ballot(bad);
#pragma unroll 1
        for (int i = 0; i < 4 && !known; ++i) {
          const int g = g0 + 4 * t + i;
          if (g >= G || ((m >> (16 * i)) & 0xFFFFu) == 0) continue;
          sum += quarter_sum<kRec>(p, row, g, q, k0, k1, x);
          sum += __shfl_xor(sum, 16);   // the row's other quarters; the sums of groups are kept in quarter 0
          sum += __shfl_xor(sum, 32);
          known = __ballot(sum == sum) == 0;
          sum = q == 0 || not_finite(sum) ? sum : 0.f;
        }
      }
    }
    if (q == j >> 2 && n < nrows && not_finite(sum)) store(b0 + j, sum);
  }
}

// RT, CT: row tiles of the workgroup, column tiles of the batch.  kRec: the
// matrix has records.  kQuads: quads of rows that the last column tile of X
// can hold (the rest of its LDS rows is left as it is: a row of X is a row of
// the result, which nobody stores).
template <int RT, int CT, bool kRec, int kQuads>
__global__ void __launch_bounds__(kThreads)
tile_kernel(const uint8_t* __restrict__ codes0, const uint16_t* __restrict__ scale0, const uint16_t* __restrict__ X,
            const int32_t* __restrict__ rowptr1, int n_out, int G, int B, int opts, int nnz1, const TileArgs a) {
  // The table is the kernel's only static array, so it sits at LDS address 0
  // and the byte-to-address v_perm is the whole address.
  __shared__ __attribute__((aligned(16))) unsigned char lut[kLutBytes];
  extern __shared__ __attribute__((aligned(32))) unsigned char lds[];
  constexpr int NW = kWaves;
  constexpr bool kLean = RT * CT >= 12;
  constexpr bool kTight = RT > 1 && CT > 1;   // keep the scheduler from holding more in registers than there are
  constexpr int R = 16 * RT, T = kThreads;
  constexpr int kMaxC = kMaxPairs / R;
  constexpr int kPadC = kMaxC > 64 ? 128 : (kMaxC > 32 ? 64 : 32);
  constexpr int kWordLoads = (R * kPadC + T - 1) / T;   // staged pairs per thread

  // opts: the chunk's groups, log2 of the staging threads per row (at least
  // as many), fp32 output, offsets on every group,
  // record ranges in the arguments.
  const int chunk = opts & 0x1FF, bits = (opts >> 9) & 7;
  const bool out_f32 = (opts >> 12) & 1, has_off = (opts >> 13) & 1;
  const int K = G * kGroup;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4;                // lane block: code bytes 8q.. of the group
  const int n16 = lane & 15;              // batch row of the X operand; weight row of the W operand and of C
  const uint32_t slot = (uint32_t)(lane & (kLutCopies - 1)) << 3;
  const int row0 = blockIdx.x * R;
  const int nrows = min(R, n_out - row0);
  const uint32_t f0 = (uint32_t)row0 * (uint32_t)G;   // the workgroup's first group

  // X of one group and 16 batch rows: four loads of four whole rows (256
  // bytes each), staged in the wave's LDS buffer and read back as operands:
  // lane (q, n) and window u take the 16 bytes at 80 q + 16 u of row n, zeros
  // for the windows that block 3 does not have.  (Loaded as operands straight
  // from memory, every load touches 16 rows in 2 to 3 lines each: the address
  // lookups, 40 a load, then took longer than everything else.)  Rows past B
  // repeat the last one; their results are not stored.
  const __amdgpu_buffer_rsrc_t xrsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)const_cast<uint16_t*>(X), 0, 2 * B * K, 0x00020000);
  const uint32_t xo = (uint32_t)q * 2u * (uint32_t)K + 16u * (uint32_t)n16;
  // In the last column tile, whose rows may end early:
  auto last_xo = [&](int j, int qq) {
    return __umul24((uint32_t)min(16 * (CT - 1) + 4 * j + qq, B - 1), 2u * (uint32_t)K) + 16u * (uint32_t)n16;
  };
  uint32_t xol[4];
  if constexpr (!kLean) {
#pragma unroll
    for (int j = 0; j < 4; ++j) xol[j] = last_xo(j, q);
  }
  // X of a step is turned one step ahead where the registers allow it.
  constexpr int kXB = RT == 1 || CT == 1 ? 2 : 1;
  auto load_x = [&](u4v (&xg)[4], int c, int g) {
#pragma unroll
    for (int j = 0; j < (c < CT - 1 ? 4 : kQuads); ++j)
      xg[j] = c < CT - 1 ? __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xo, 2 * kGroup * g + (16 * c + 4 * j) * 2 * K, 0)
                         : __builtin_amdgcn_raw_buffer_load_b128(xrsrc, kLean ? last_xo(j, here_v(q)) : xol[j], 2 * kGroup * g, 0);
  };
  unsigned char* const xw = lds + wave * 16 * kXRow + q * kXRow + 16 * n16;
  const unsigned char* const xr0 = lds + wave * 16 * kXRow + n16 * kXRow + 80 * q;
  const unsigned char* const xr1 = q < 3 ? xr0 : lds + tile_zero_off(NW) - 16;
  // The wave's LDS accesses complete in order, so one buffer serves every
  // column tile and group, without waits.
  auto turn_x = [&](const u4v (&xg)[4], u4v (&dst)[5]) {
#pragma unroll
    for (int j = 0; j < (CT == 1 ? kQuads : 4); ++j) *reinterpret_cast<u4v*>(xw + 4 * j * kXRow) = xg[j];
    __builtin_amdgcn_wave_barrier();
    dst[0] = *reinterpret_cast<const u4v*>(xr0);
#pragma unroll
    for (int u = 1; u < 5; ++u) dst[u] = *reinterpret_cast<const u4v*>(xr1 + 16 * u);
    __builtin_amdgcn_wave_barrier();
  };
  // Step i of a wave: column tile i % CT of its group i / CT.  Steps past the
  // chunk repeat its last group, unused: a load under a condition would make
  // every later wait for an older load wait for it as well.
  auto load_step = [&](u4v (&xg)[4], int c, int g, int glast) { load_x(xg, c % CT, min(g + NW * (c / CT), glast)); };

  // Codes 0..23 of the workgroup's rows: lane (q, n) reads bytes 8q .. 8q+7 of
  // row n of a tile.  Block 3 (whose bytes are the tail's) and rows past the
  // end lie outside the buffer and read as zeros.
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)const_cast<uint8_t*>(codes0 + (size_t)(24u * f0)), 0, 24 * nrows * G, 0x00020000);
  uint32_t wo[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    wo[rt] = q < 3 ? __umul24((uint32_t)(16 * rt + n16), 24u * (uint32_t)G) + 8u * (uint32_t)q : 0x80000000u;
  auto load_codes = [&](u2v (&dst)[RT], int g) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) dst[rt] = __builtin_amdgcn_raw_buffer_load_b64(wrsrc, wo[rt], 24 * g, 0);
  };

  float4v total[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) total[rt][c] = float4v{0.f, 0.f, 0.f, 0.f};

  for (int g0 = 0; g0 < G; g0 += chunk) {
    // ---- 1. Loads, all issued before any wait, in the order of their use,
    // at clamped addresses: X of the wave's first group, tails and scales;
    // behind the table, whose set-up covers the wait for the kernel
    // arguments, row pointers, records, offsets and the codes of the first
    // group.  (The rest goes out behind the first barrier: a CU holds only so
    // many loads in flight, and a wave that waits to issue one holds up the
    // others there.)
    const int gn = min(chunk, G - g0), glast = g0 + gn - 1;
    u4v xg[4], xb[kXB][5];
    u2v ring[kRing][RT];
    load_x(xg, 0, min(g0 + wave, glast));
    uint32_t tv[kWordLoads], sv[kWordLoads], ov[kWordLoads];
    {
      const int t = here_v(tid);
      const uint8_t* tails = codes0 + (size_t)(24u * (uint32_t)n_out * (uint32_t)G) + (size_t)(2u * f0);
      const uint16_t* scales = scale0 + (size_t)f0;
#pragma unroll
      for (int j = 0; j < kWordLoads; ++j) {
        const int r = (j * T + t) >> bits, g = (j * T + t) & ((1 << bits) - 1);
        const uint32_t f = (uint32_t)(min(r, nrows - 1) * G + g0 + min(g, gn - 1));
        tv[j] = *reinterpret_cast<const uint16_t*>(tails + (size_t)(2u * f));
        sv[j] = scales[(size_t)f];
      }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- 2. The table (once; at step k the copies' position is rotated by
    // the code, so the lanes of a store cover the banks), and empty record
    // lists.
    if (g0 == 0) {
      for (int t = here_v(tid); t < 512; t += T) {
        const int c = t & 255, h = t >> 8;
        const u2v e = table_entry(c);
#pragma unroll
        for (int k = 0; k < kLutCopies / 4; ++k)
          reinterpret_cast<u4v*>(lut)[c * (kLutCopies / 2) + ((8 * h + k + c) & (kLutCopies / 2 - 1))] =
              u4v{e.x, e.y, e.x, e.y};
      }
      if (const int t = here_v(tid); t < 16) reinterpret_cast<uint32_t*>(lds + tile_zero_off(NW))[t] = 0u;
    } else {
      lds_barrier();   // the previous chunk's reads are done
    }
    __builtin_amdgcn_sched_barrier(0);
    // Records of the workgroup's rows.
    int kb = 0, ke = 0;
    int rp = 0;   // lane r: first record of row r
    RecLoad rec0;
    if constexpr (kRec) {
      const int32_t* rps = rowptr1 + row0;
      rp = rps[min(here_v(lane), nrows)];
      if ((opts >> 14) & 1) {   // ranges in the arguments
        kb = a.rec_begin[blockIdx.x];
        ke = a.rec_begin[blockIdx.x + 1];
      } else {   // in bounds whatever the row pointers hold
        kb = max(0, min(rps[0], nnz1));
        ke = max(0, min(rps[nrows], nnz1));
      }
      rec0 = load_record(a, nnz1, max(0, min(kb + here_v(tid), ke - 1)));
    }
    {
      const int t = here_v(tid);
      const uint16_t* offs = (has_off ? a.offset0 : scale0) + (size_t)f0;   // (unused without offsets)
#pragma unroll
      for (int j = 0; j < kWordLoads; ++j) {
        const int r = (j * T + t) >> bits, g = (j * T + t) & ((1 << bits) - 1);
        ov[j] = offs[(size_t)(uint32_t)(min(r, nrows - 1) * G + g0 + min(g, gn - 1))];
      }
    }
    load_codes(ring[0], min(g0 + wave, glast));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kRec)
      for (int i = here_v(tid); i < 4 * gn; i += T)
        reinterpret_cast<uint32_t*>(lds + tile_count_off(NW, R, here_s(chunk)))[i] = 0u;
    lds_barrier();

    // ---- 3. Staging.
    const int C = here_s(chunk), t = here_v(tid);
    const int WS = tile_stride(C);
    unsigned char* slot_s = lds + tile_slot_off(NW);
    uint8_t* count_s = lds + tile_count_off(NW, R, C);
    u2v* word_s = reinterpret_cast<u2v*>(lds + tile_word_off(NW, R, C));
    if constexpr (kXB == 2) {
      turn_x(xg, xb[0]);
      load_step(xg, 1, g0 + wave, glast);
    }
#pragma unroll
    for (int d = 1; d < kRing; ++d) load_codes(ring[d], min(g0 + NW * d + wave, glast));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kWordLoads; ++j) {
      const int r = (j * T + t) >> bits, g = (j * T + t) & ((1 << bits) - 1);
      if (r < R && g < C) {
        word_s[r * WS + g] = u2v{tv[j] | (sv[j] << 16), ov[j]};
      }
    }
    if constexpr (kRec) {
      auto stage_record = [&](int k, const RecLoad& r) {
        // Row of record k: the rows after the first that start at or before
        // it (rows past the end hold the end of the records).
        int lo = 0;
#pragma unroll
        for (int r = 1; r < R; ++r) lo += k >= __builtin_amdgcn_readlane(rp, r) ? 1 : 0;
        const int g = r.gg - g0, n = lo & 15;
        if (k < ke && r.gg < G && g >= 0 && g < gn) {
          // Which pass holds a record does not matter for the result: the
          // records of a group belong to different rows.
          const uint32_t old = atomicAdd(reinterpret_cast<uint32_t*>(count_s) + 4 * g + (n >> 2), 1u << (8 * (n & 3)));
          const int p = (int)((old >> (8 * (n & 3))) & 0xFFu);
          if (p < RT) {
            u2v* d = reinterpret_cast<u2v*>(slot_s + 32 * ((g * RT + p) * 16 + n));
            d[0] = __builtin_bit_cast(u2v, r.v0);
            d[1] = __builtin_bit_cast(u2v, r.v1);
            d[2] = __builtin_bit_cast(u2v, r.v2);
            d[3] = u2v{r.tl | ((uint32_t)(lo >> 4) << 16), r.sm};
          }
        }
      };
      if (kb + (t & ~63) < ke) stage_record(kb + t, rec0);
      for (int k = kb + T; k < ke; k += T) stage_record(k + t, load_record(a, nnz1, min(k + t, ke - 1)));
    }
    lds_barrier();

    // ---- 4. Main loop: this wave's groups of the chunk.
    const int ml = here_v(lane), n16 = ml & 15, q = ml >> 4;
    const uint32_t tail_mask = ml >= 48 ? 0xFFFFu : 0u;
    // Staged data of a group, one group ahead where the registers allow it.
    constexpr int SB = kTight ? 1 : 2;
    u2v word[SB][RT];
    int count[SB];
    u2v rw[SB], re[SB];
    const uint32_t word_at = here_v(lds_address(word_s + n16 * WS));
    const uint32_t count_at = here_v(lds_address(count_s + n16)), slot_at = here_v(lds_address(slot_s + 32 * n16));
    auto read_staged = [&](int b, int g) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) word[b][rt] = lds_read<u2v>(word_at + (uint32_t)(8 * (16 * rt * WS + g)));
      if constexpr (kRec) {
        count[b] = lds_read<uint8_t>(count_at + (uint32_t)(16 * g));
        rw[b] = lds_read<u2v>(slot_at + (uint32_t)(512 * RT * g + 8 * q));
        re[b] = lds_read<u2v>(slot_at + (uint32_t)(512 * RT * g + 24));
      }
    };
    read_staged(0, min(wave, gn - 1));
    // Table entries of the next tile, read before the MFMAs of the tile
    // before it.
    u2v e[8];
    read_entries(lut, slot, u2v{ring[0][0].x | (word[0][0].x & tail_mask), ring[0][0].y}, e);
    for (int gb = wave; gb < gn; gb += NW * kRing) {
#pragma unroll
      for (int d = 0; d < kRing; ++d) {
        const int g = gb + NW * d;
        if (g >= gn) break;
        if (d == 0) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        if constexpr (SB == 1) read_staged(0, g);
        else read_staged((d + 1) % 2, min(g + NW, gn - 1));
        // Codes of the next group's first tile.
        const uint32_t next_word = SB == 2 ? word[(d + 1) % SB][0].x : lds_read<u2v>(word_at + (uint32_t)(8 * min(g + NW, gn - 1))).x;
        const u2v next_codes = {ring[(d + 1) % kRing][0].x | (next_word & tail_mask), ring[(d + 1) % kRing][0].y};
        // Whether any of the group's rows has a record: 16 rows at 10 % (3.6 %)
        // two-plane groups have none in 18 % (56 %) of the groups.
        const bool any = kRec && __ballot(count[d % SB] > 0) != 0;
        // The operands of the row tiles and of the first pass of plane 1 are
        // decoded once, for every column tile.
        u4v W[RT + (kRec ? 1 : 0)][5];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const u4v (&xv)[5] = xb[(d * CT + c) % kXB];
          if constexpr (kXB == 2) {
            turn_x(xg, xb[(d * CT + c + 1) % 2]);
            load_step(xg, c + 2, g0 + g, glast);
          } else {
            turn_x(xg, xb[0]);
            load_step(xg, c + 1, g0 + g, glast);
          }
          float4v acc[RT], xs = {0.f, 0.f, 0.f, 0.f};
          auto add_plane0 = [&](int rt) {
            const float s0 = h2f(word[d % SB][rt].x >> 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) total[rt][c][i] = __builtin_fmaf(s0, acc[rt][i], total[rt][c][i]);
          };
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            if (c == 0) {
              expand(e, W[t]);
              if (t + 1 < RT)
                read_entries(lut, slot, u2v{ring[d][(t + 1) % RT].x | (word[d % SB][(t + 1) % RT].x & tail_mask),
                                            ring[d][(t + 1) % RT].y}, e);
              else if (kRec)
                read_entries(lut, slot, any || CT > 1 ? rw[d % SB] : next_codes, e);
            }
            if (t == RT - 1 && c == CT - 1 && (CT > 1 || !kRec)) read_entries(lut, slot, next_codes, e);
            __builtin_amdgcn_sched_barrier(0);
            acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 5; ++u) {
              acc[t] = mfma(xv[u], W[t][u], acc[t]);
              // The sum of x over the group, laid out as the totals (only
              // used with records or offsets).
              if (t == 0) xs = mfma(xv[u], u4v{kOnes, kOnes, kOnes, kOnes}, xs);
            }
            if (t > 0) add_plane0(t - 1);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (c == 0) load_codes(ring[d], min(g0 + g + NW * kRing, glast));
          settle(xs, acc[RT - 1]);
          add_plane0(RT - 1);
          if (has_off) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              const float mu = h2f(word[d % SB][rt].y);
#pragma unroll
              for (int i = 0; i < 4; ++i) total[rt][c][i] = __builtin_fmaf(mu, xs[i], total[rt][c][i]);
            }
          }
          if (any) {
            // Pass p of plane 1: the p-th record of each slot.  Rows without a
            // record keep their totals, also where the sums of the empty slot
            // are not finite.
            auto add_plane1 = [&](int p, u2v r, const u4v (&V)[5]) {
              float4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int u = 0; u < 5; ++u) v = mfma(xv[u], V[u], v);
              settle(xs, v);
              const float s1 = h2f(r.y & 0xFFFFu), mu = h2f(r.y >> 16);
#pragma unroll
              for (int rt = 0; rt < RT; ++rt)
                if (count[d % SB] > p && (RT == 1 || (int)(r.x >> 16) == rt)) {
#pragma unroll
                  for (int i = 0; i < 4; ++i)
                    total[rt][c][i] = __builtin_fmaf(s1, v[i], __builtin_fmaf(mu, xs[i], total[rt][c][i]));
                }
            };
            if constexpr (kRec) {
              if (c == 0) {
                expand(e, W[RT]);
                if constexpr (CT == 1) read_entries(lut, slot, next_codes, e);
                __builtin_amdgcn_sched_barrier(0);
              }
              add_plane1(0, re[d % SB], W[RT]);
            }
            for (int p = 1; p < RT; ++p) {
              if (__ballot(count[d % SB] > p) == 0) break;
              const uint32_t at = slot_at + (uint32_t)(512 * (RT * g + p));
              u2v ev[8];
              u4v V[5];
              if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
              read_entries(lut, slot, lds_read<u2v>(at + (uint32_t)(8 * q)), ev);
              expand(ev, V);
              add_plane1(p, lds_read<u2v>(at + 24u), V);
            }
          }
          if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

  // ---- 5. Partial sums of the waves, added in wave order, then Y.
  lds_barrier();   // every wave is done with the staged data
  float4v* red = reinterpret_cast<float4v*>(lds);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < CT; ++c) red[((wave * RT + rt) * CT + c) * 64 + lane] = total[rt][c];
  lds_barrier();
  constexpr int kItems = RT * CT * 64;
  for (int it = tid; it < kItems; it += T) {
    const int ln = it & 63, c = (it >> 6) % CT, rt = (it >> 6) / CT;
    float4v s = red[it];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w * kItems + it];
    const int r = 16 * rt + (ln & 15), b = 16 * c + 4 * (ln >> 4);
    auto store = [&](int bb, float y) {
      const int64_t o = (int64_t)bb * n_out + row0 + r;
      if (out_f32)
        reinterpret_cast<float*>(a.Y)[o] = y;
      else
        reinterpret_cast<uint16_t*>(a.Y)[o] = (uint16_t)f2h(y);
    };
    if (r < nrows) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (b + i < B) store(b + i, s[i]);
    }
    // (One check for a lane's four sums, outputs or not; the quads of X that
    // were not loaded may hold anything.)
    bool odd = not_finite((s[0] + s[1]) + (s[2] + s[3]));
    if constexpr (kQuads < 4) odd = odd && (ln >> 4) < kQuads;
    if (__builtin_expect(__ballot(odd) != 0, 0)) redo_tile<kRec>(row0 + 16 * rt, nrows - 16 * rt, 16 * c, s, store);
  }
}

typedef void (*TileKernel)(const uint8_t*, const uint16_t*, const uint16_t*, const int32_t*, int, int, int, int, int,
                           const TileArgs);

template <int RT, int CT, int Q>
TileKernel tile_pick_rec(bool rec) {
  return rec ? tile_kernel<RT, CT, true, Q> : tile_kernel<RT, CT, false, Q>;
}

// Most row tiles of a workgroup: the operands of a group's row tiles are kept
// in registers for all column tiles.  Four with two column tiles take 256
// registers, with three they spill (34.8 us at 16384 x 4096, B = 48, where
// two rounds of two row tiles take 28.8).
constexpr int most_row_tiles(int CT) { return CT > 2 ? 3 : 4; }

// Row tiles: a workgroup fills a CU (table and staged data take its LDS), so
// the time is the rounds of 256 workgroups times the time of one, which is
// near 3 + row tiles in units of a tile (4096 inputs, B = 16: 7.9, 9.9, 11.7
// and 16.5 us for 1 to 4 tiles in one round; the last stages two chunks).
// Over 3500 shapes of up to 40000 outputs the choice is within 0.1 % of the
// best of the four on average and 8 % at most.  16384 x 4096, B = 17: 27.2 us
// with three tiles in two rounds, 20.7 with four in one; 16400 x 4096, B = 16:
// 28.8 with four in two rounds, 21.9 with three.
int row_tiles(int n_out, int CT) {
  int best = 1;
  int64_t cost = INT64_MAX;
  for (int rt = 1; rt <= most_row_tiles(CT); ++rt) {
    const int64_t wgs = ((int64_t)n_out + 16 * rt - 1) / (16 * rt);
    const int64_t c = (wgs + kCus - 1) / kCus * (3 + rt);
    if (c <= cost) {
      cost = c;
      best = rt;
    }
  }
  return best;
}

template <int CT, int Q>
TileKernel tile_pick(int RT, bool rec) {
  switch (RT) {
    case 1: return tile_pick_rec<1, CT, Q>(rec);
    case 2: return tile_pick_rec<2, CT, Q>(rec);
    case 3: return tile_pick_rec<3, CT, Q>(rec);
    default: return tile_pick_rec<most_row_tiles(CT), CT, Q>(rec);
  }
}

// Whether a kernel's LDS limit is raised already, by device, column tiles and
// quads, row tiles, records.
bool& tile_attr_set(int CT, int quads, int RT, bool rec) {
  static thread_local bool set[64][4][3][4][2];
  int dev = 0;
  (void)hipGetDevice(&dev);
  return set[dev & 63][CT - 1][quads >> 1][RT - 1][rec ? 1 : 0];
}

}  // namespace

hipError_t launch_gemm_smallbatch(const MatDev& m, const uint16_t* X, int B, void* Y, bool out_f32,
                                  hipStream_t s) {
  const int G = m.n_groups;
  const int CT = (B + 15) / 16;
  const int RT = row_tiles(m.n_out, CT);
  const int R = 16 * RT;
  const int wgs = (m.n_out + R - 1) / R;
  // Chunks of equal size, as few as hold at most kMaxPairs pairs.
  const int most_groups = kMaxPairs / R;
  const int chunks = (G + most_groups - 1) / most_groups;
  const int C = (G + chunks - 1) / chunks;
  int lane_bits = 4;
  while ((1 << lane_bits) < C) ++lane_bits;

  // Record ranges in the kernel arguments where the host has the row
  // pointers and the workgroups are few enough.
  const bool rec = m.nnz1 > 0;
  const bool host = rec && m.rowptr1_host != nullptr && wgs <= kMaxRanges;
  TileKernel kernel;
  switch (CT) {
    // (Instances for few rows where the whole batch is few rows: a quarter of
    // X's loads and LDS writes at B = 4.)
    case 1:
      kernel = B <= 4 ? tile_pick<1, 1>(RT, rec) : (B <= 8 ? tile_pick<1, 2>(RT, rec) : tile_pick<1, 4>(RT, rec));
      break;
    case 2: kernel = tile_pick<2, 4>(RT, rec); break;
    case 3: kernel = tile_pick<3, 4>(RT, rec); break;
    default: kernel = tile_pick<4, 4>(RT, rec); break;
  }
  TileArgs args;
  args.offset0 = m.offset0;
  args.codes1 = m.codes1;
  args.gidx1 = m.gidx1;
  args.offset1 = m.offset1;
  args.scale1 = m.scale1;
  args.Y = Y;
  if (host) {
    for (int w = 0; w <= wgs; ++w) {
      const int64_t r = (int64_t)w * R < m.n_out ? (int64_t)w * R : m.n_out;
      int64_t v = m.rowptr1_host[r];
      v = v < 0 ? 0 : (v > m.nnz1 ? m.nnz1 : v);   // in bounds whatever the host copy holds
      args.rec_begin[w] = (int32_t)v;
    }
  }
  const int staged = tile_lds(kWaves, R, C);
  const int red = tile_red_bytes(kWaves, RT, CT);
  const int dyn = staged > red ? staged : red;
  bool& set = tile_attr_set(CT, CT > 1 || B > 8 ? 4 : (B > 4 ? 2 : 1), RT, rec);
  if (!set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit - kLutBytes);
    if (e != hipSuccess) return e;
    set = true;
  }
  const int opts = C | (lane_bits << 9) | (out_f32 ? 1 << 12 : 0) | (m.offset0 != nullptr ? 1 << 13 : 0) |
                   (host ? 1 << 14 : 0);
  hipLaunchKernelGGL(kernel, dim3(wgs), dim3(kThreads), dyn, s, m.codes0, m.scale0, X, m.rowptr1, m.n_out, G, B, opts,
                     (int)m.nnz1, args);
  return hipGetLastError();
}

}  // namespace tq
