// Choice of the two-plane groups and the plane-1 CSR of a linear (gfx950).
//
// Paper: section 4.2 (E2M-ATQ) gives a second ternary plane to a minority
// of blocks; section 3 chooses them with salience masks fitted on
// calibration activations, which are not available here, so groups are
// ranked by their one-plane residual energy (written by tq_ternarize).  The
// rule: the nnz groups with the largest energy, ties to the lower flat index
// (row-major (r, g)); a NaN energy ranks below every number, -0 and +0 tie.
// Records are numbered in flat order, which is CSR order by row.
//
// Steps, all on the caller's stream, with scratch in the caller's workspace:
// 1. Radix select of the nnz-th largest 64-bit key, in passes of 8-bit digits
//    from the most significant: a histogram over the keys that match the
//    digits found so far, whose last block to finish picks the digit holding
//    the wanted rank and clears the histogram.  Once at most kGather keys
//    match, the next pass collects them and its last block ranks them; the
//    passes after that return at once (random energies: four passes, the last
//    of them collecting, where eight and as many launches to pick took eight
//    times two).  The result is the threshold key T and the number `need` of
//    groups with key T to take (the first `need` of them in flat order).
// 2. Per tile of kTile groups: how many keys are above T and equal to T; the
//    last block turns them into each tile's offset among the equal keys and
//    among the selected groups (a tile takes its equal keys while the running
//    count of equal keys is below `need`).
// 3. Per tile: block-local scans give each selected group its record
//    index, written to rec_index and gidx1, and the row pointers of the
//    rows whose first group lies in the tile.
// Up to kSmall groups one workgroup does all of it, with the keys in registers.
// kSmall is what they hold: the one workgroup is the faster at every size it
// takes (10 % of random energies, against the launches above, each some 2 us of
// launch and 5 of atomics' round trips: 4000 groups 26 and 55 us, 8192 27 and
// 58, 32768 34 and 60; with few distinct energies 39 and 61, 41 and 87, 53 and
// 88), so the cost steps up where it ends (32800 groups: 57 us).
// Counts are integers, so the result is deterministic and unique.

#include <mutex>

#include "tq_internal.h"

namespace tq {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;                  // groups per thread per tile
constexpr int kTile = kThreads * kItems;    // 4096 groups per tile

// Workspace layout: histogram, state, then four uint32 arrays over tiles.
constexpr size_t kHistBytes = 256 * sizeof(uint32_t);
struct SelState {
  uint64_t prefix;   // digits found so far (the threshold key T at the end)
  uint64_t mask;     // which bits of prefix are set
  uint64_t rank;     // wanted rank among keys matching prefix (1-based, from the top)
  uint32_t ticket;   // blocks of the running launch that have finished
  uint32_t phase;    // kCount, kCollect or kDone, + the collected keys << 2
};
constexpr uint32_t kCount = 0, kCollect = 1, kDone = 2;
constexpr int kGather = kThreads;           // keys ranked by one block, one per thread
constexpr int kSmallThreads = 1024;
constexpr int kSmallItems = 32;
constexpr int kSmall = kSmallThreads * kSmallItems;
constexpr size_t kStateOff = kHistBytes;
constexpr size_t kTilesOff = kStateOff + sizeof(SelState);

__host__ __device__ constexpr int64_t num_tiles(int64_t n) { return (n + kTile - 1) / kTile; }

constexpr size_t workspace_bytes_for(int64_t n) {
  return (kTilesOff + 4 * sizeof(uint32_t) * (size_t)num_tiles(n) + 255) & ~(size_t)255;
}

// Scratch of the allocation-free entry point: one copy per GPU, held until
// the process ends.  Host code never passes this name to a kernel; it uses
// the device address obtained for it below.
constexpr size_t kScratchBytes = workspace_bytes_for(TQ_SELECT_NOALLOC_MAX_GROUPS);
static __device__ __attribute__((aligned(256))) unsigned char scratch[kScratchBytes];

// Orderable key of an energy: larger energy, larger key; NaN is 0, below
// every number (-inf maps to 0x000FFFFFFFFFFFFF); both zeros map to the key
// of +0.
__device__ inline uint64_t energy_key(double e) {
  uint64_t b = __builtin_bit_cast(uint64_t, e);
  if ((b & 0x7FFFFFFFFFFFFFFFull) > 0x7FF0000000000000ull) return 0;   // NaN
  if ((b & 0x7FFFFFFFFFFFFFFFull) == 0) b = 0;                          // -0 -> +0
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// Exclusive scan of v over the block (blockDim.x a multiple of 64, at most
// 1024 threads); *total receives the block's sum.  Every thread must call.
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wsum[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t s = wsum[w];
    before += w < wave ? s : 0u;
    tot += s;
  }
  __syncthreads();   // wsum is reused by the next call
  *total = tot;
  return before + inc - v;
}

// Values that blocks of one launch hand to its last block: accesses that
// bypass the caches of the eight dies, so that no cache has to be written
// back (a device-wide fence costs more than a pass).
template <typename V>
__device__ inline V ld_dev(const V* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ inline void st_dev(V* p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether this block is the last of the launch: every block's stores and
// atomics have completed before it takes its ticket.
__device__ inline bool last_block(SelState* st) {
  __shared__ uint32_t mine;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    mine = __hip_atomic_fetch_add(&st->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (mine == gridDim.x - 1) st_dev(&st->ticket, 0u);
  }
  __syncthreads();
  return mine == gridDim.x - 1;
}

// One block of 256 threads: clear the histogram and set the state.
__global__ void __launch_bounds__(256) sel_init(uint32_t* hist, SelState* st, uint64_t rank) {
  hist[threadIdx.x] = 0u;
  if (threadIdx.x == 0) {
    st->prefix = 0;
    st->mask = 0;
    st->rank = rank;
    st->ticket = 0;
    st->phase = kCount;
  }
}

// Adds one to h[digit] for every lane with `match` (LDS); a wave whose
// matching lanes share a digit, as in the first passes, adds once.
__device__ inline void count_digit(uint32_t* h, uint32_t digit, bool match) {
  const uint64_t m = __ballot(match);
  if (m == 0) return;
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, __builtin_ctzll(m));
  if (__ballot(match && digit == d0) == m) {
    if (__lane_id() == 0) atomicAdd(&h[d0], (uint32_t)__builtin_popcountll(m));
  } else if (match) {
    atomicAdd(&h[digit], 1u);
  }
}

// The digit of 256 that holds rank (1-based, counting from the largest
// digit), the count of larger digits and the digit's own count; c is the
// count of digit 255 - threadIdx.x in the first 256 threads of the block.
struct Digit {
  uint32_t digit, above, count;
};
__device__ inline Digit pick_digit(uint32_t c, uint64_t rank) {
  __shared__ Digit found;
  uint32_t total;
  const uint32_t above = block_exclusive_scan(threadIdx.x < 256 ? c : 0u, &total);
  if (threadIdx.x < 256 && above < rank && rank <= (uint64_t)above + c) found = Digit{255u - threadIdx.x, above, c};
  __syncthreads();
  const Digit f = found;
  __syncthreads();   // (before the next call writes it)
  return f;
}

// One pass: the histogram of the digit at `shift` over the keys that match
// the digits found so far (LDS counts per block, then one global add per bin),
// or, with few keys left, their indexes in `list`; the last block finishes
// the pass.
__global__ void __launch_bounds__(kThreads) sel_pass(const double* __restrict__ energy, int64_t n, SelState* st,
                                                     uint32_t* hist, int32_t* list, int shift) {
  __shared__ uint32_t h[256];
  __shared__ uint64_t keys[kGather];
  const uint32_t phase = ld_dev(&st->phase) & 3u;
  if (phase == kDone) return;
  h[threadIdx.x] = 0u;
  __syncthreads();
  const uint64_t prefix = st->prefix, mask = st->mask;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t base = (int64_t)blockIdx.x * kThreads; base < n; base += stride) {
    const int64_t i = base + threadIdx.x;
    const uint64_t k = energy_key(energy[i < n ? i : n - 1]);
    const bool match = i < n && (k & mask) == prefix;
    if (phase == kCount) {
      count_digit(h, (uint32_t)(k >> shift) & 255u, match);
    } else if (match) {
      const uint32_t at = __hip_atomic_fetch_add(&st->phase, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 2;
      if (at < (uint32_t)kGather) st_dev(&list[at], (int32_t)i);
    }
  }
  __syncthreads();
  const uint32_t c = h[threadIdx.x];
  if (c) __hip_atomic_fetch_add(&hist[threadIdx.x], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!last_block(st)) return;
  const uint64_t rank = st->rank;
  if (phase == kCount) {
    const uint32_t bin = ld_dev(&hist[255 - threadIdx.x]);
    const Digit f = pick_digit(bin, rank);
    hist[255 - threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
      st->rank = rank - f.above;
      st->prefix = prefix | (uint64_t)f.digit << shift;
      st->mask = mask | 255ull << shift;
      if (f.count <= (uint32_t)kGather && shift > 0) st->phase = kCollect;
    }
  } else {
    // The rank-th largest of the collected keys: the one with fewer than
    // `rank` keys above it and at least `rank` at or above it.
    const uint32_t have = ld_dev(&st->phase) >> 2;
    const bool mine = threadIdx.x < have;
    const uint64_t k = mine ? energy_key(energy[ld_dev(&list[threadIdx.x])]) : 0ull;
    keys[threadIdx.x] = k;
    __syncthreads();
    uint32_t above = 0, equal = 0;
    for (uint32_t j = 0; j < have; ++j) {
      above += keys[j] > k ? 1u : 0u;
      equal += keys[j] == k ? 1u : 0u;
    }
    if (mine && above < rank && rank <= (uint64_t)above + equal) {   // (equal keys store the same values)
      st->prefix = k;
      st->rank = rank - above;
      st->phase = kDone;
    }
  }
}

// A tile's offsets among the equal keys and among the selected groups, for
// all tiles, in chunks of blockDim.x tiles with running carries (one block).
__device__ inline void tile_offsets(uint64_t need, const uint32_t* gt, const uint32_t* eq, uint32_t* eq_off,
                                    uint32_t* sel_off, int64_t ntiles) {
  uint64_t carry_eq = 0, carry_sel = 0;
  for (int64_t c0 = 0; c0 < ntiles; c0 += blockDim.x) {
    const int64_t b = c0 + threadIdx.x;
    const uint32_t e = b < ntiles ? ld_dev(&eq[b]) : 0u, g = b < ntiles ? ld_dev(&gt[b]) : 0u;
    uint32_t te, ts;
    const uint64_t eoff = carry_eq + block_exclusive_scan(e, &te);
    const uint64_t left = need > eoff ? need - eoff : 0;
    const uint32_t take = (uint32_t)(left < e ? left : e);
    const uint64_t soff = carry_sel + block_exclusive_scan(g + take, &ts);
    if (b < ntiles) {
      eq_off[b] = (uint32_t)eoff;
      sel_off[b] = (uint32_t)soff;
    }
    carry_eq += te;
    carry_sel += ts;
  }
}

// Per tile: keys above and equal to the threshold; the last block: offsets.
__global__ void __launch_bounds__(kThreads) sel_count(const double* __restrict__ energy, int64_t n, SelState* st,
                                                      uint32_t* gt, uint32_t* eq, uint32_t* eq_off, uint32_t* sel_off) {
  const uint64_t T = st->prefix;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  uint32_t cg = 0, ce = 0;
#pragma unroll 4
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = base + (int64_t)j * kThreads + threadIdx.x;
    if (i < n) {
      const uint64_t k = energy_key(energy[i]);
      cg += k > T ? 1u : 0u;
      ce += k == T ? 1u : 0u;
    }
  }
  uint32_t tg, te;
  block_exclusive_scan(cg, &tg);
  block_exclusive_scan(ce, &te);
  if (threadIdx.x == 0) {
    st_dev(&gt[blockIdx.x], tg);
    st_dev(&eq[blockIdx.x], te);
  }
  if (last_block(st)) tile_offsets(st->rank, gt, eq, eq_off, sel_off, gridDim.x);
}

// Everything for n <= kSmall in one block.  Item j of thread t is
// group 1024 j + t, so loads and stores are whole lines and a wave's ballot
// holds the flags of 64 consecutive groups, in which flat order is counted.
// The digits, of 12 bits, start at the first bit in which the largest and the
// smallest key differ: the bits above would count every key in a few bins,
// one after the other.
constexpr int kSmallBins = 4096;
__global__ void __launch_bounds__(kSmallThreads) sel_small(const double* __restrict__ energy, int n, int G,
                                                           uint32_t magic, int64_t n_out, int nnz, int32_t* rec_index,
                                                           int32_t* rowptr1, uint16_t* gidx1) {
  __shared__ uint32_t h[kSmallBins];
  __shared__ uint64_t eq_s[kSmall / 64], sel_s[kSmall / 64];   // sel_s: keys above the threshold, then the selected
  __shared__ uint32_t base_s[kSmall / 64], found[3];
  __shared__ uint64_t lo_s[kSmallThreads / 64], hi_s[kSmallThreads / 64];
  const int t = threadIdx.x, lane = t & 63;
  uint64_t key[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) key[j] = energy_key(energy[min(kSmallThreads * j + t, n - 1)]);
  uint64_t lo = key[0], hi = key[0];   // (groups past the end repeat the last one)
#pragma unroll
  for (int j = 1; j < kSmallItems; ++j) {
    lo = key[j] < lo ? key[j] : lo;
    hi = key[j] > hi ? key[j] : hi;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    const uint64_t l = __shfl_xor(lo, d), m = __shfl_xor(hi, d);
    lo = l < lo ? l : lo;
    hi = m > hi ? m : hi;
  }
  if (lane == 0) {
    lo_s[t >> 6] = lo;
    hi_s[t >> 6] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSmallThreads / 64; ++w) {
    lo = lo_s[w] < lo ? lo_s[w] : lo;
    hi = hi_s[w] > hi ? hi_s[w] : hi;
  }
  int left = lo == hi ? 0 : 64 - __builtin_clzll(lo ^ hi);   // bits still to find
  left = __builtin_amdgcn_readfirstlane(left);
  uint64_t mask = left == 64 ? 0ull : ~0ull << left;
  uint64_t prefix = hi & mask;
  uint32_t need = (uint32_t)nnz;
  while (left > 0) {
    const int shift = left > 12 ? left - 12 : 0;
    const uint32_t digits = (1u << (left - shift)) - 1u;
    for (int i = t; i < kSmallBins; i += kSmallThreads) h[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j)
      if (kSmallThreads * j + t < n && (key[j] & mask) == prefix) atomicAdd(&h[(uint32_t)(key[j] >> shift) & digits], 1u);
    __syncthreads();
    // Four bins a thread, the largest digits first.
    uint32_t c[4], sum = 0, total;
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += c[i] = h[kSmallBins - 1 - 4 * t - i];
    uint32_t above = block_exclusive_scan(sum, &total);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (above < need && need <= above + c[i]) {
        found[0] = (uint32_t)(kSmallBins - 1 - 4 * t - i);
        found[1] = above;
        found[2] = c[i];
      }
      above += c[i];
    }
    __syncthreads();
    need -= found[1];
    prefix |= (uint64_t)found[0] << shift;
    mask |= (uint64_t)digits << shift;
    left = found[2] == need ? 0 : shift;   // (every key that matches is taken)
    left = __builtin_amdgcn_readfirstlane(left);
    __syncthreads();
  }
  // Selected: keys above the matching ones, and the first `need` of these.
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int i = kSmallThreads * j + t;
    const uint64_t k = key[j] & mask;
    const uint64_t gt = __ballot(i < n && k > prefix), eq = __ballot(i < n && k == prefix);
    if (lane == 0) {
      eq_s[i >> 6] = eq;
      sel_s[i >> 6] = gt;
    }
  }
  __syncthreads();
  const bool word = t < kSmall / 64;
  uint64_t eq = word ? eq_s[t] : 0ull, sel = word ? sel_s[t] : 0ull;
  uint32_t total;
  const uint32_t before = block_exclusive_scan((uint32_t)__builtin_popcountll(eq), &total);
  if (before + (uint32_t)__builtin_popcountll(eq) <= need) {
    sel |= eq;
  } else {
    for (uint32_t r = before; r < need; ++r) {   // (one word at most starts below `need` and ends above)
      sel |= eq & (0ull - eq);
      eq &= eq - 1;
    }
  }
  const uint32_t rec0 = block_exclusive_scan((uint32_t)__builtin_popcountll(sel), &total);
  if (word) {
    sel_s[t] = sel;
    base_s[t] = rec0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int i = kSmallThreads * j + t;
    // The word of the wave's 64 groups, in scalar registers.
    const uint64_t w = sel_s[i >> 6];
    const uint32_t wl = __builtin_amdgcn_readfirstlane((uint32_t)w), wh = __builtin_amdgcn_readfirstlane((uint32_t)(w >> 32));
    const uint32_t base = __builtin_amdgcn_readfirstlane(base_s[i >> 6]);
    const uint32_t rec = __builtin_amdgcn_mbcnt_hi(wh, __builtin_amdgcn_mbcnt_lo(wl, base));
    if (i < n) {
      const bool s = ((lane < 32 ? wl : wh) >> (lane & 31)) & 1u;
      const int row = G == 1 ? i : (int)__umulhi((uint32_t)i, magic), g = i - row * G;   // exact for i < 2^16
      rec_index[i] = s ? (int32_t)rec : -1;
      if (s && rec < (uint32_t)nnz) gidx1[rec] = (uint16_t)g;
      if (g == 0) rowptr1[row] = (int32_t)rec;   // records before the row's first group
    }
  }
  if (t == 0) rowptr1[n_out] = nnz;
}

// Nothing to select (the steps above took three launches and, at 4.2 million
// groups, 71 us; this one takes 8).
__global__ void __launch_bounds__(kThreads) sel_none(int64_t n, int64_t n_out, int32_t* rec_index, int32_t* rowptr1) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
    rec_index[i] = -1;
    if (i <= n_out) rowptr1[i] = 0;
  }
  if (n == n_out && blockIdx.x == 0 && threadIdx.x == 0) rowptr1[n_out] = 0;
}

// Per tile: thread t takes the kItems consecutive groups base + kItems t ..,
// so block-local scans follow flat order.
__global__ void __launch_bounds__(kThreads) sel_write(const double* __restrict__ energy, int64_t n, int32_t G,
                                                      int64_t n_out, int64_t nnz, const SelState* st,
                                                      const uint32_t* eq_off, const uint32_t* sel_off,
                                                      int32_t* rec_index, int32_t* rowptr1, uint16_t* gidx1) {
  const uint64_t T = st->prefix, need = st->rank;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
  uint32_t gtm = 0, eqm = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = base + j;
    if (i < n) {
      const uint64_t k = energy_key(energy[i]);
      gtm |= (k > T ? 1u : 0u) << j;
      eqm |= (k == T ? 1u : 0u) << j;
    }
  }
  uint32_t total;
  uint64_t r = (uint64_t)eq_off[blockIdx.x] + block_exclusive_scan((uint32_t)__builtin_popcount(eqm), &total);
  uint32_t selm = gtm;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if ((eqm >> j) & 1u) {
      if (r < need) selm |= 1u << j;
      ++r;
    }
  }
  uint32_t rec = sel_off[blockIdx.x] + block_exclusive_scan((uint32_t)__builtin_popcount(selm), &total);
  uint32_t row = (uint32_t)base / (uint32_t)G, g = (uint32_t)base - row * (uint32_t)G;   // (n < 2^31)
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = base + j;
    if (i < n) {
      const bool s = (selm >> j) & 1u;
      rec_index[i] = s ? (int32_t)rec : -1;
      if (s && rec < (uint64_t)nnz) gidx1[rec] = (uint16_t)g;
      if (g == 0) rowptr1[row] = (int32_t)rec;   // records before the row's first group
      rec += s ? 1u : 0u;
      if (++g == (uint32_t)G) {
        g = 0;
        ++row;
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) rowptr1[n_out] = (int32_t)nnz;
}

}  // namespace

size_t select_workspace_bytes(int64_t n) { return workspace_bytes_for(n); }

hipError_t launch_select(const double* energy, int64_t n_out, int32_t G, int64_t nnz, int32_t* rec_index,
                         int32_t* rowptr1, uint16_t* gidx1, void* workspace, hipStream_t s) {
  const int64_t n = n_out * G;
  const int64_t nt = num_tiles(n);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws);
  SelState* st = reinterpret_cast<SelState*>(ws + kStateOff);
  uint32_t* gt = reinterpret_cast<uint32_t*>(ws + kTilesOff);
  uint32_t* eq = gt + nt;
  uint32_t* eq_off = eq + nt;
  uint32_t* sel_off = eq_off + nt;

  if (nnz == 0) {
    const int64_t b = (n + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(sel_none, dim3((unsigned)(b < 2048 ? b : 2048)), dim3(kThreads), 0, s, n, n_out, rec_index,
                       rowptr1);
    return hipGetLastError();
  }
  if (n <= kSmall) {
    hipLaunchKernelGGL(sel_small, dim3(1), dim3(kSmallThreads), 0, s, energy, (int)n, G,
                       (uint32_t)((0x100000000ull + G - 1) / G), n_out, (int)nnz, rec_index, rowptr1, gidx1);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(sel_init, dim3(1), dim3(256), 0, s, hist, st, (uint64_t)nnz);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // The candidates' list is kept in rec_index, which the last step writes
  // whole (n > kSmall holds them).
  const unsigned hb = (unsigned)(nt < 512 ? nt : 512);
  for (int shift = 56; shift >= 0; shift -= 8) {
    hipLaunchKernelGGL(sel_pass, dim3(hb), dim3(kThreads), 0, s, energy, n, st, hist, rec_index, shift);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(sel_count, dim3((unsigned)nt), dim3(kThreads), 0, s, energy, n, st, gt, eq, eq_off, sel_off);
  hipLaunchKernelGGL(sel_write, dim3((unsigned)nt), dim3(kThreads), 0, s, energy, n, G, n_out, nnz, st, eq_off,
                     sel_off, rec_index, rowptr1, gidx1);
  return hipGetLastError();
}

// Device address of `scratch` on the current GPU, looked up once per device
// (each GPU holds its own copy of the array at its own address).
static hipError_t scratch_address(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

hipError_t launch_select_noalloc(const double* energy, int64_t n_out, int32_t G, int64_t nnz, int32_t* rec_index,
                                 int32_t* rowptr1, uint16_t* gidx1, hipStream_t s) {
  if (n_out * G > TQ_SELECT_NOALLOC_MAX_GROUPS) return hipErrorInvalidValue;
  void* ws = nullptr;
  const hipError_t e = scratch_address(&ws);
  if (e != hipSuccess) return e;
  return launch_select(energy, n_out, G, nnz, rec_index, rowptr1, gidx1, ws, s);
}

}  // namespace tq
