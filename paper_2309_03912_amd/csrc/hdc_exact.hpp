// Exact sum of bfloat16 values: the real sum of the inputs, rounded once to
// fp64, whatever the summation order, tuning or grid -- bit-reproducible.
//
// Every finite bf16 value is m * 2^(E - 134) with an integer m < 2^8 and its
// biased exponent E in [0, 254] (m = 128 + the fraction for E >= 1; for
// subnormals, E = 0, m is twice the fraction).  Two exact ways to add one:
//  * the window: values whose exponents lie within 40 of each other are
//    integers below 2^47 in the unit of the lowest one, so 32 of them add up
//    exactly in fp64 registers (below 2^52);
//  * the digits, for any value: writing E = 32 d + r, the value is
//    (m << r) * 2^(32 d - 134), an integer below 2^39 added to digit d
//    (d in [0, 7]) of a fixed-point number whose digit j has the unit
//    2^(32 j - 134), kept as fp64 accumulators in LDS (integers below 2^53,
//    so every add is exact; no carries while folding).
// Lanes, wavefronts and blocks then add digit by digit as int64 (integer
// additions: exact and order-free), and the final combine propagates the
// carries into 32-bit digits and rounds the whole number to nearest-even fp64
// once.  Infinities and NaNs are tracked as flags with the IEEE outcome of
// their sum (NaN if a NaN or both infinities appear).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "hdc_device.hpp"
#include "hdc_functors.hpp"
#include "hdc_kernels.hpp"

namespace hdc {

constexpr int kExactDigits = 10;  // units 2^-134 .. 2^154: every sum of < 2^31 bf16 values
constexpr int kExactFoldDigits = 8;  // digits that receive terms directly

// Fold state: digits (carry-save) and the non-finite flags
// (bit 0: +inf seen, bit 1: -inf seen, bit 2: NaN seen).
struct Bf16Exact {
  int64_t d[kExactDigits];
  uint32_t nf;
  uint32_t pad;
  __device__ static Bf16Exact zero() {
    Bf16Exact z;
#pragma unroll
    for (int j = 0; j < kExactDigits; ++j) z.d[j] = 0;
    z.nf = 0;
    z.pad = 0;
    return z;
  }
  __device__ static Bf16Exact merge(Bf16Exact a, const Bf16Exact& b) {
#pragma unroll
    for (int j = 0; j < kExactDigits; ++j) a.d[j] += b.d[j];
    a.nf |= b.nf;
    return a;
  }
  // Carries into the next digit: digits 0 .. 8 end in [0, 2^32), the top one
  // keeps the sign (floor division, so negative digits borrow correctly).
  __device__ void normalize() {
#pragma unroll
    for (int j = 0; j + 1 < kExactDigits; ++j) {
      const int64_t c = d[j] >> 32;  // arithmetic shift: floor(d / 2^32)
      d[j] -= c * (int64_t(1) << 32);
      d[j + 1] += c;
    }
  }
  // The exact value rounded once to fp64 (nearest, ties to even).
  __device__ double value() const {
    if ((nf & 4u) || (nf & 3u) == 3u) return __builtin_nan("");
    if (nf & 1u) return __builtin_inf();
    if (nf & 2u) return -__builtin_inf();
    Bf16Exact t = *this;
    t.normalize();
    const bool neg = t.d[kExactDigits - 1] < 0;
    uint32_t g[kExactDigits];  // magnitude, 32-bit digits
    uint64_t borrow = 1;       // two's complement negation: ~digits + 1
#pragma unroll
    for (int j = 0; j < kExactDigits; ++j) {
      const uint32_t v = (uint32_t)t.d[j];
      if (neg) {
        const uint64_t s = (uint64_t)(uint32_t)~v + borrow;
        g[j] = (uint32_t)s;
        borrow = s >> 32;
      } else {
        g[j] = v;
      }
    }
    // The highest non-zero digit and the two below it (constant indices: the
    // digits stay in registers), and whether any lower digit is non-zero.
    uint32_t h = 0, m1 = 0, m0 = 0;
    int top = -1;
    bool rest = false;
#pragma unroll
    for (int j = kExactDigits - 1; j >= 0; --j) {
      if (top < 0) {
        if (g[j]) {
          top = j;
          h = g[j];
          m1 = j >= 1 ? g[j - 1] : 0;
          m0 = j >= 2 ? g[j - 2] : 0;
        }
      } else if (j < top - 2) {
        rest = rest || g[j] != 0;
      }
    }
    if (top < 0) return 0.0;
    const int lz = __builtin_clz(h);
    const uint64_t hi = ((uint64_t)h << 32) | m1;
    const uint64_t m = (hi << lz) | (lz ? (uint64_t)m0 >> (32 - lz) : 0);
    rest = rest || (uint32_t)(m0 << lz) != 0;
    const double r = round_top64(m, rest, 32 * (top - 1) - lz - 134);  // bit 0 has the value 2^-134
    return neg ? -r : r;
  }
};

// A block's total as it lies in the workspace: the normalized digits 0 .. 8,
// the flags, and the signed top digit as two words (the upper one biased by
// 2^31, so that all words add up unsigned) -- 48 bytes instead of the state's 88.
constexpr int kBf16Words = kExactDigits + 2;
struct alignas(8) Bf16Partial {
  uint32_t w[kBf16Words];
};

__device__ __forceinline__ Bf16Partial exact_pack(Bf16Exact s) {
  s.normalize();
  Bf16Partial p;
#pragma unroll
  for (int j = 0; j + 1 < kExactDigits; ++j) p.w[j] = (uint32_t)s.d[j];
  p.w[kExactDigits - 1] = s.nf;
  p.w[kExactDigits] = (uint32_t)s.d[kExactDigits - 1];
  p.w[kExactDigits + 1] = (uint32_t)(s.d[kExactDigits - 1] >> 32) + 0x80000000u;
  return p;
}

// Merge the g packed totals with one block and write the rounded sum (integer
// additions: any order gives the same digits).  The totals are read as one
// flat run of 8-byte words by a multiple of six threads, so every thread's
// words are the same two of a total; it adds them to two int64 sums (the
// flags by OR), and six threads then add up the threads' sums.  (One total
// per thread, merged as whole states across the wavefronts, took 4 us for
// 1024 of them, most of it the 22 words of every lane exchange.)
// `sums` (LDS) holds 2 * blockDim.x values.
template <class Load>
__device__ __forceinline__ void exact_bf16_fold_partials(Load load, int g, double* out, uint64_t* sums) {
  constexpr int P = kBf16Words / 2;  // 8-byte words per total
  static_assert(kBf16Words % 2 == 0);
  const int tid = threadIdx.x, nt = blockDim.x, used = nt / P * P;
  const int total = g * P;
  uint64_t s0 = 0, s1 = 0;
  uint32_t any = 0;
  const int col = tid % P;
  constexpr int kFlags = (kExactDigits - 1) / 2, kTop = kExactDigits / 2;  // the columns of flags and top digit
  static_assert((kExactDigits - 1) % 2 == 1);                              // the flags are a column's second word
  if (tid < used) {
    constexpr int kRound = 12;
    for (int base = tid; base < total; base += kRound * used) {
      uint64_t v[kRound];
#pragma unroll
      for (int u = 0; u < kRound; ++u) {
        const int i = base + u * used;
        v[u] = load(i < total ? i : tid);  // past the end: a word that exists, not added
      }
#pragma unroll
      for (int u = 0; u < kRound; ++u) {
        if (base + u * used >= total) v[u] = 0;
        s0 += (uint32_t)v[u];
        s1 += v[u] >> 32;
        any |= (uint32_t)(v[u] >> 32);
      }
    }
    if (col == kFlags) s1 = any;
    sums[tid] = s0;
    sums[nt + tid] = s1;
  }
  // the threads' sums in two rounds: rows of 42 threads, then rows of six
  auto gather = [&](int step, int end) {
    __syncthreads();
    if (tid < step) {
      for (int i = tid + step; i < end; i += step) {
        s0 += sums[i];
        s1 = col == kFlags ? s1 | sums[nt + i] : s1 + sums[nt + i];
      }
      sums[tid] = s0;
      sums[nt + tid] = s1;
    }
  };
  gather(7 * P, used);
  gather(P, 7 * P);
  __syncthreads();
  if (tid == 0) {
    Bf16Exact s = Bf16Exact::zero();
#pragma unroll
    for (int j = 0; j < kExactDigits - 1; ++j) s.d[j] = (int64_t)sums[(j & 1) * nt + j / 2];
    s.nf = (uint32_t)sums[nt + kFlags];
    s.d[kExactDigits - 1] = (int64_t)(sums[kTop] + ((sums[nt + kTop] - ((uint64_t)g << 31)) << 32));
    *out = s.value();
  }
}

// Merge the g partials get(0) ... get(g - 1) with one block and write the
// rounded sum.
template <class Acc, class Get>
__device__ __forceinline__ void exact_fold_partials(Get get, int g, double* out, Acc* lds) {
  Acc s = Acc::zero();
  for (int i = threadIdx.x; i < g; i += blockDim.x) s = Acc::merge(s, get(i));
  s = block_reduce(s, MergeOp<Acc>{}, lds);
  if (threadIdx.x == 0) *out = s.value();
}

// The end of a block of pass 1 in the one-launch form: thread 0 publishes the
// block's total and counts it on the ticket; true in every thread of the
// block that arrives last.
template <class Partial>
__device__ __forceinline__ bool exact_arrive(const Partial& p, Partial* partials, uint32_t* ticket) {
  __shared__ int last;
  if (threadIdx.x == 0) {
    publish_partial(partials, blockIdx.x, p);
    last = arrive_last(ticket, blockIdx.x, gridDim.x);
  }
  __syncthreads();
  return last;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Pass 1: every block folds its grid-stride share of 16-byte vectors (8
// values; head and tail elements by the last block) into one state.
//
// What bounds it: HBM, with the vector ALU close behind.  A wavefront takes
// its window from the first values it sees (4 exponents above their largest,
// 35 below) and checks every vector against it with packed 16-bit minima and
// maxima of the bit patterns (zeros pass: the minimum is taken of pattern - 1).
// A vector inside it costs five instructions per value (check two, unpack,
// widen, add); the chunk's sum is then split exactly in two by a magic
// constant and added to two fp64 totals, which take 2^25 such sums.  A vector
// with a value outside goes to the digits: the value scaled by
// 2^(134 - 32 d) in fp64 and one fp64 LDS add to the lane's accumulator of
// digit d by address (digit j of thread i at dig[j * blockDim + i], a ninth
// slot that is never read for infinities and NaNs, whose flags are taken on a
// rare path): nine instructions and an LDS atomic per value.  If half of a
// chunk's vectors do, the wavefront takes the digits without a check for
// kExactSkip chunks and then a new window, so data with no common window
// costs what the digits cost.  Whole call, every value through the digits ->
// windows: 2^27 N(0,1) values 64.7 -> 48.4 us, 2^28 108.8 -> 87.9 us (6.1
// TB/s); lognormal(0, 4) values, which share no window, 103.6 -> 101.9 us.
// The digit accumulators stay exact while a lane takes fewer than 2^14 terms,
// which the launch guarantees (at most 1024 vectors per lane,
// kExactVecsPerLane).
constexpr int64_t kExactVecsPerLane = 1024;  // 8192 terms (+2 head/tail) < 2^14
constexpr int kExactMaxBlock = 512;          // 9 slots x 8 bytes x 512 threads = 36 KiB of LDS
constexpr int kExactAbove = 4, kExactBelow = 35;  // the window: from 35 exponents below the largest to 4 above
constexpr int kExactSkip = 16;

template <int U>
__global__ __launch_bounds__(kExactMaxBlock) void exact_bf16_kernel(const uint16_t* __restrict__ x, Range r,
                                                                    Bf16Partial* partials, uint32_t* ticket,
                                                                    double* out) {
  extern __shared__ double dig[];  // (kExactFoldDigits + 1) * blockDim
  constexpr int V = 8;
  const int64_t B = blockDim.x, tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j <= kExactFoldDigits; ++j) dig[j * B + tid] = 0.0;
  // LDS byte address of this thread's slot of digit d: own + 8 B d, one
  // 24-bit multiply-add (d is bits 12-14 of the bf16 word, the top three bits
  // of E).
  using lds_f64 = __attribute__((address_space(3))) double;
  const uint32_t own = (uint32_t)(uintptr_t)(lds_f64*)(dig + tid), stride = 8u * (uint32_t)B;
  const uint32_t sink = own + stride * kExactFoldDigits;
  uint32_t nf = 0;
  auto fold = [&](const uint32_t (&u)[V]) {  // u: bf16 bits, 0 for no value
    bool special = false;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const uint32_t d = (u[i] >> 12) & 7u;  // E / 32
      // the value itself (bf16 is the top half of binary32; subnormals are kept),
      // scaled by 2^(134 - 32 d): the signed integer m 2^(E mod 32), exact in fp64
      const float v = __builtin_bit_cast(float, u[i] << 16);
      const bool fin = __builtin_isfinite(v);
      special = special || !fin;
      const double t = __builtin_ldexp((double)v, 134 - 32 * (int)d);
      const uint32_t at = fin ? own + d * stride : sink;
      __hip_atomic_fetch_add((lds_f64*)(uintptr_t)at, t, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (__builtin_amdgcn_ballot_w64(special) != 0) {  // rare: infinities and NaNs present
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (((u[i] >> 7) & 0xFFu) == 0xFFu) nf |= (u[i] & 0x7Fu) ? 4u : ((u[i] >> 15) ? 2u : 1u);
    }
  };
  auto fold_vec = [&](const u32x4& a) {
    uint32_t u[V];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      u[2 * k] = a[k] & 0xFFFFu;
      u[2 * k + 1] = a[k] >> 16;
    }
    fold(u);
  };
  // The window (uniform in the wavefront): exponents [low, top], at most 40, as
  // bounds of the patterns without the sign, both halves alike.  The totals:
  // integers in the unit 2^(low - 134), `hi` a multiple of 2^24 of them.
  int low = -1;  // no window yet
  uint32_t pmin1 = 0, pmax = 0;
  double magic = 0.0, hi = 0.0, lo = 0.0;
  // The integer q (|q| <= 2^38) in the unit 2^(at - 134), at < 224, to the
  // lane's digits: below 2^39 each, so at most 64 windows add less than 2^45.
  auto to_digits = [&](int64_t q, int at) {
    const int j = at >> 5, r = at & 31;
    const uint64_t part = (uint64_t)(uint32_t)q << r;
    dig[j * B + tid] += (double)(uint32_t)part;
    dig[(j + 1) * B + tid] += (double)((int64_t)(part >> 32) + (q >> 32) * (int64_t(1) << r));
  };
  auto close_window = [&]() {
    if (low < 0) return;
    const double scale = __builtin_ldexp(1.0, 134 - low);
    to_digits((int64_t)(hi * scale * 0x1p-24), low + 24);  // at most 1024 chunks of 2^52: below 2^38
    to_digits((int64_t)(lo * scale), low);                 // at most 1024 chunks of 2^23
    hi = lo = 0.0;
    low = -1;
    pmin1 = pmax = 0;  // admits zeros only
  };
  auto open_window = [&](const u32x4 (&a)[U]) {
    uint32_t m = 0;
#pragma unroll
    for (int w = 0; w < U; ++w)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t p = a[w][k] & 0x7FFFu, q = (a[w][k] >> 16) & 0x7FFFu;
        m = p < 0x7F80u && p > m ? p : m;
        m = q < 0x7F80u && q > m ? q : m;
      }
    m = wave_reduce(m, [](uint32_t p, uint32_t q) { return p > q ? p : q; });
    m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    if (m == 0) return;  // only zeros so far (or nothing finite)
    const int top = (int)(m >> 7) + kExactAbove;
    if (top > 238) return;  // from 2^112 on: digits only (low + 24 stays below digit 7)
    low = top - (kExactAbove + kExactBelow);
    low = low < 0 ? 0 : low;
    const uint32_t first = low > 0 ? (uint32_t)low << 7 : 1u, end = ((uint32_t)top << 7) | 0x7Fu;
    pmin1 = (first - 1) * 0x10001u;
    pmax = end * 0x10001u;
    magic = __builtin_ldexp(1.5, 52 + 24 + low - 134);
  };
  const uint16_t* xv = x + r.head;
  const int64_t cv = B * U;  // vectors per chunk
  const int64_t nchunk = (r.nvec + cv - 1) / cv;
  // The chunk's loads go through a raw buffer resource based at the chunk
  // and ending at its last vector (word 3 0x00020000: 32-bit data format, no
  // swizzle; cache policy 2: non-temporal): lane offsets stay fixed, and a
  // load past the end returns zeros, which add nothing.
  uint32_t vo[U];
#pragma unroll
  for (int w = 0; w < U; ++w) vo[w] = (uint32_t)(tid + w * B) * 16u;
  int skip = 0;
  for (int64_t c = blockIdx.x; c < nchunk; c += gridDim.x) {
    const int64_t v0 = c * cv;
    const int32_t bytes = (int32_t)((r.nvec - v0 < cv ? r.nvec - v0 : cv) * 16);
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void*)(xv + v0 * V), (short)0, bytes, 0x00020000);
    u32x4 a[U];
#pragma unroll
    for (int w = 0; w < U; ++w) a[w] = __builtin_amdgcn_raw_buffer_load_b128(rx, vo[w], 0, 2);
    if (skip == 0 && low < 0) open_window(a);
    int outside = 0;
    double c0 = 0.0, c1 = 0.0;
#pragma unroll
    for (int w = 0; w < U; ++w) {
      u16x2 mn = __builtin_bit_cast(u16x2, pmin1), mx = __builtin_bit_cast(u16x2, pmax);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u16x2 p = __builtin_bit_cast(u16x2, a[w][k] & 0x7FFF7FFFu);
        mx = __builtin_elementwise_max(mx, p);
        mn = __builtin_elementwise_min(mn, (u16x2)(p - (u16x2)1));
      }
      const bool bad = __builtin_bit_cast(uint32_t, mn) != pmin1 || __builtin_bit_cast(uint32_t, mx) != pmax;
      if (skip == 0 && __builtin_amdgcn_ballot_w64(bad) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          c0 += (double)__builtin_bit_cast(float, a[w][k] << 16);
          c1 += (double)__builtin_bit_cast(float, a[w][k] & 0xFFFF0000u);
        }
      } else {
        fold_vec(a[w]);
        ++outside;
      }
    }
    const double sum = c0 + c1;                 // 32 terms below 2^47: exact
    const double h = (sum + magic) - magic;     // the multiple of 2^24 nearest it
    hi += h;
    lo += sum - h;
    if (skip > 0) {
      --skip;
    } else if (2 * outside > U) {  // no common window here: digits for a while, then a new window
      close_window();
      skip = kExactSkip;
    }
  }
  if (blockIdx.x == gridDim.x - 1) {  // unaligned head and the tail, one element per lane
    uint32_t u[V] = {};
    if (tid < r.head) u[0] = x[tid];
    if (tid < r.tail) u[1] = x[r.tail_start + tid];
    fold(u);
  }
  close_window();
  // The block's digits: wavefront w adds up the lanes' accumulators of digits
  // w, w + waves, ... straight from LDS.  (Every lane converting and merging
  // its own eight digits, 22 words a lane exchange, cost ~1000 instructions a
  // wavefront: 7 us of a 12 us kernel at 2^24 values.)
  __shared__ int64_t total_sh[kExactFoldDigits];
  __shared__ uint32_t nf_sh;
  if (tid == 0) nf_sh = 0;
  __syncthreads();
  if (nf) atomicOr(&nf_sh, nf);
  const int lane = (int)tid & 63, nw = (int)(B >> 6);
  for (int j = (int)(tid >> 6); j < kExactFoldDigits; j += nw) {
    uint64_t t = 0;
    for (int i = lane; i < (int)B; i += 64) t += (uint64_t)(int64_t)dig[j * B + i];  // integers below 2^53: exact
    t = wave_reduce(t, AddU64{});
    if (lane == 0) total_sh[j] = (int64_t)t;
  }
  __syncthreads();
  Bf16Exact s = Bf16Exact::zero();
  if (tid == 0) {
#pragma unroll
    for (int j = 0; j < kExactFoldDigits; ++j) s.d[j] = total_sh[j];
    s.nf = nf_sh;
  }
  if (gridDim.x == 1) {
    if (tid == 0) *out = s.value();
    return;
  }
  const Bf16Partial p = exact_pack(s);  // thread 0's
  if (!ticket) {
    if (tid == 0) partials[blockIdx.x] = p;
    return;
  }
  if (exact_arrive(p, partials, ticket)) {
    const uint64_t* w = reinterpret_cast<const uint64_t*>(partials);
    exact_bf16_fold_partials(
        [&](int i) { return __hip_atomic_load(w + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, (int)gridDim.x,
        out, reinterpret_cast<uint64_t*>(dig));
  }
}

// Pass 2 (one block) of the two-launch form.
static __global__ __launch_bounds__(256) void exact_bf16_final_kernel(const Bf16Partial* partials, int g, double* out) {
  __shared__ uint64_t sums[2 * 256];
  const uint64_t* w = reinterpret_cast<const uint64_t*>(partials);
  exact_bf16_fold_partials([&](int i) { return w[i]; }, g, out, sums);
}

// ---------------------------------------------------------------------------
// Exact dot product of fp16 vectors.  The product p of two fp16 values is
// exact in fp32 (at most 22 significant bits, 2^-48 <= |p| < 2^32 unless 0)
// and is an integer multiple of 2^-48.  Split at 2^-8, p = h + l with
// h = trunc(p 2^8) 2^-8 (a multiple of 2^-8 below 2^32) and l = p - h (a
// multiple of 2^-48 below 2^-8); both steps are exact in fp32.  Each part
// spans at most 40 bits, so fp64 chains of up to 2^13 of them never round.
// Lanes flush their two chains once per grid-stride step into a 128-bit
// two's-complement integer in units of 2^-48 (h 2^8 and l 2^48 are integers
// below 2^53); the total, below 2^63 in magnitude for fewer than 2^31
// products, is rounded once to fp64.  A product with an infinite or NaN
// factor (inf * 0 is NaN) goes to the high chain only, and the non-finite
// chain values add by IEEE rules in `nf`.
// ---------------------------------------------------------------------------

struct F16DotExact {
  double dh;  // chain of high parts
  double dl;  // chain of low parts
  float nf;   // IEEE sum of the non-finite chains; 0 if none
  uint32_t pad;
  uint64_t lo, hi;  // 128-bit two's complement, units of 2^-48
  __device__ static F16DotExact zero() { return {0.0, 0.0, 0.0f, 0u, 0u, 0u}; }
  __device__ void add(float p) {
    const float h = __builtin_truncf(p * 256.0f) * 0.00390625f;
    const float l = __builtin_isfinite(p) ? p - h : 0.0f;
    dh += (double)h;
    dl += (double)l;
  }
  __device__ void add128(uint64_t low, uint64_t high) {
    const uint64_t s = lo + low;
    hi += high + (s < lo ? 1u : 0u);
    lo = s;
  }
  __device__ void flush() {
    if (!__builtin_isfinite(dh)) {
      nf += (float)dh;
    } else {
      const int64_t qh = (int64_t)(dh * 256.0);                // |.| < 2^53: exact
      const int64_t ql = (int64_t)(dl * 281474976710656.0);    // 2^48; |.| < 2^53: exact
      add128((uint64_t)ql, (uint64_t)(ql >> 63));
      add128((uint64_t)qh << 40, (uint64_t)(qh >> 24));     // qh 2^40 as 128 bits
    }
    dh = 0.0;
    dl = 0.0;
  }
  __device__ static F16DotExact merge(F16DotExact a, F16DotExact b) {
    a.flush();
    b.flush();
    a.nf += b.nf;
    a.add128(b.lo, b.hi);
    return a;
  }
  // The 128-bit integer rounded by the fp16 sum's rounding (units of 2^-24),
  // then scaled by 2^-24, which is exact for these magnitudes.
  __device__ double value() const {
    F16DotExact t = *this;
    t.flush();
    if (t.nf != 0.0f || t.nf != t.nf) return (double)t.nf;
    ExactAcc e = ExactAcc::zero();
    e.lo = t.lo;
    e.hi = t.hi;
    return __builtin_ldexp(e.value(), -24);
  }
};

__device__ __forceinline__ float f16_bits_to_f32(uint32_t u) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)u);
}

// Pass 1: every block folds its grid-stride share in 16-byte vectors of 8
// values aligned to x (the head and the tail by the last block).  kEven: z's
// vectors start on 4-byte boundaries, as buffer loads need, and are loaded
// through a buffer resource as x's are; otherwise they are loaded with global
// loads, which take any address.
template <int U, bool kEven>
__global__ __launch_bounds__(1024) void exact_f16_dot_kernel(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ z, Range r,
                                                             F16DotExact* partials, uint32_t* ticket,
                                                             double* out) {
  __shared__ F16DotExact lds[kMaxWaves];
  const int64_t B = blockDim.x, tid = threadIdx.x;
  F16DotExact acc = F16DotExact::zero();
  constexpr int V = 8;
  const uint16_t* xv = x + r.head;
  const uint16_t* zv = z + r.head;
  const int64_t cv = B * U;  // vectors per chunk
  const int64_t nchunk = (r.nvec + cv - 1) / cv;
  // Loads through raw buffer resources based at the chunk and ending at its
  // last vector, as in exact_bf16_kernel: zeros past the end (a product of
  // zeros adds nothing), fixed lane offsets.
  uint32_t vo[U];
#pragma unroll
  for (int u = 0; u < U; ++u) vo[u] = (uint32_t)(tid + u * B) * 16u;
  for (int64_t c = blockIdx.x; c < nchunk; c += gridDim.x) {
    const int64_t v0 = c * cv;
    const int32_t bytes = (int32_t)((r.nvec - v0 < cv ? r.nvec - v0 : cv) * 16);
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void*)(xv + v0 * V), (short)0, bytes, 0x00020000);
    u32x4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = __builtin_amdgcn_raw_buffer_load_b128(rx, vo[u], 0, 2);
    if constexpr (kEven) {
      const __amdgpu_buffer_rsrc_t rz =
          __builtin_amdgcn_make_buffer_rsrc((void*)(zv + v0 * V), (short)0, bytes, 0x00020000);
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = __builtin_amdgcn_raw_buffer_load_b128(rz, vo[u], 0, 2);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // past the end: the chunk's first vector again, replaced by zeros
        const int64_t v = v0 + tid + u * B;
        const Vec<F16> w = load16<F16>(reinterpret_cast<const _Float16*>(zv + (v < r.nvec ? v : v0) * V));
        __builtin_memcpy(&b[u], &w, 16);
        if (v >= r.nvec) b[u] = u32x4{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc.add(f16_bits_to_f32(a[u][k]) * f16_bits_to_f32(b[u][k]));          // exact in fp32
        acc.add(f16_bits_to_f32(a[u][k] >> 16) * f16_bits_to_f32(b[u][k] >> 16));
      }
    acc.flush();  // chains of at most 8 U terms
  }
  if (blockIdx.x == gridDim.x - 1) {  // unaligned head and the tail, one element per lane
    if (tid < r.head) acc.add(f16_bits_to_f32(x[tid]) * f16_bits_to_f32(z[tid]));
    if (tid < r.tail) acc.add(f16_bits_to_f32(x[r.tail_start + tid]) * f16_bits_to_f32(z[r.tail_start + tid]));
  }
  acc.flush();
  acc = block_reduce(acc, MergeOp<F16DotExact>{}, lds);
  if (gridDim.x == 1) {
    if (tid == 0) *out = acc.value();
  } else if (!ticket) {
    if (tid == 0) partials[blockIdx.x] = acc;
  } else if (exact_arrive(acc, partials, ticket)) {
    exact_fold_partials<F16DotExact>([&](int i) { return read_partial(partials, i); }, (int)gridDim.x, out, lds);
  }
}

static __global__ __launch_bounds__(256) void exact_f16_dot_final_kernel(const F16DotExact* partials, int g,
                                                                         double* out) {
  __shared__ F16DotExact lds[kMaxWaves];
  exact_fold_partials<F16DotExact>([&](int i) { return partials[i]; }, g, out, lds);
}

}  // namespace hdc
