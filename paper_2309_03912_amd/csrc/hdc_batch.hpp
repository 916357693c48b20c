// Grouped batch: many independent map + reduce calls of one class (same
// storage type, callables and fold) in one grouped launch and, where a call has
// more than 64 chunks or all have more than there are compute units, one
// combine launch.  The call table is a by-value kernel argument (no
// host-to-device copy, so the launches can be recorded into a graph as they are).
//
// Every call is cut into chunks of its `chunk_vecs` 16-byte vectors, which its
// own size and the tuning set; the global chunk index space is the concatenation of all calls' chunks.  A block takes
// chunks grid-stride, finds the call owning the chunk from the prefix table,
// maps and folds it, and writes one partial per chunk.  The combine launch
// folds each call's partials in chunk order, so results depend only on the
// data, the chunk size and the block: bit-reproducible, and the same whatever
// other calls the batch holds.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "hdc_device.hpp"
#include "hdc_functors.hpp"
#include "hdc_kernels.hpp"

namespace hdc {

constexpr int kBatchMax = 32;  // calls per grouped launch (keeps the table ~2.3 KB)

struct BatchCall {
  const void* x;
  void* y;  // nullptr: no map for this call
  void* out;
  Range r;  // the walk, aligned to y if the call maps, else to x; the other operand is read from wherever it starts
  int64_t chunk_vecs;  // 16-byte vectors per chunk
};

struct BatchTable {
  int32_t count;
  int64_t prefix[kBatchMax + 1];      // first global chunk of each call
  BatchCall call[kBatchMax];
};

// Fold chunk partials [lo, hi) of one call, as read by get(k), and write the
// call's result: the first kBatchFold threads stride over them in chunk order,
// then the fixed block reduction (the waves beyond add zero states, so the bits
// do not depend on the block).
constexpr int kBatchFold = 256;

template <class Acc>
using BatchFoldT = std::conditional_t<std::is_same_v<Acc, CompAcc>, double, Acc>;

template <class Acc, class Get>
__device__ __forceinline__ void batch_fold(Get get, int64_t lo, int64_t hi, void* out, BatchFoldT<Acc>* lds) {
  const bool mine = threadIdx.x < kBatchFold;
  if constexpr (std::is_same_v<Acc, CompAcc>) {
    double d = 0.0;
    for (int64_t k = lo + threadIdx.x; mine && k < hi; k += kBatchFold) {
      const CompAcc q = get(k);
      d += __builtin_isfinite(q.s) ? (double)q.s + (double)q.c : (double)q.s;
    }
    d = block_reduce(d, AddF64{}, lds);
    if (threadIdx.x == 0) *static_cast<double*>(out) = d;
  } else {
    Acc a = Acc::zero();
    for (int64_t k = lo + threadIdx.x; mine && k < hi; k += kBatchFold) a = Acc::merge(a, get(k));
    a = block_reduce(a, MergeOp<Acc>{}, lds);
    if (threadIdx.x == 0) {
      if constexpr (std::is_same_v<Acc, PlainAcc>)
        *static_cast<float*>(out) = a.s;
      else
        *static_cast<int64_t*>(out) = (int64_t)a.s;
    }
  }
}

// The result of a call without elements.
template <class Acc>
__device__ __forceinline__ void write_empty(void* out) {
  if constexpr (std::is_same_v<Acc, PlainAcc>)
    *static_cast<float*>(out) = 0.0f;
  else
    *static_cast<uint64_t*>(out) = 0;  // a double or an int64
}

// kOne: the grid is one block per chunk, and `ticket` has zero counters (left
// zero).  The chunks of a call are counted on the call's own counter and
// the block that arrives last folds them: no second launch.  A kernel of its
// own: as a run-time branch it cost the two-launch form 9% (32 calls of up to
// 2^24 int32: 97.9 -> 106.5 us).
static_assert(kBatchMax <= (int)kTicketCounters);

template <class FM, class F, class S, class Acc, int U, bool kOne>
  requires device_callable<F> && device_callable<FM>
__global__ __launch_bounds__(1024) void batch_kernel(FM fm, F f, BatchTable t, Acc* partials, uint32_t* ticket) {
  __shared__ Acc lds[kMaxWaves];
  const int64_t B = blockDim.x;
  const int64_t tid = threadIdx.x;
  constexpr int KV = S::kVec;
  constexpr int N = U * KV;
  const int64_t total = t.prefix[t.count];
  for (int64_t c = blockIdx.x; c < total; c += gridDim.x) {
    int i = 0;
    while (i + 1 < t.count && t.prefix[i + 1] <= c) ++i;  // uniform: the owning call
    const BatchCall& call = t.call[i];
    const elem_t<S>* x = static_cast<const elem_t<S>*>(call.x);
    elem_t<S>* y = static_cast<elem_t<S>*>(call.y);
    const Range& r = call.r;
    const int64_t lc = c - t.prefix[i];
    Acc acc[KV];
#pragma unroll
    for (int k = 0; k < KV; ++k) acc[k] = Acc::zero();
    const elem_t<S>* xv = x + r.head;
    const int64_t vend = (lc + 1) * call.chunk_vecs < r.nvec ? (lc + 1) * call.chunk_vecs : r.nvec;
    // Int32 calls (a quarter-rate multiply per element) load and store
    // through raw buffer resources based at the step and ending at the
    // chunk's last vector (word 3 0x00020000: 32-bit data format, no swizzle;
    // cache policy 2: non-temporal): fixed lane offsets instead of 64-bit
    // address arithmetic per access; past the end, loads return zeros (the
    // mask leaves them out) and stores are dropped.
    constexpr bool kBuf = std::is_same_v<S, I32>;
    auto step = [&](int64_t v0, auto full_c) {
      constexpr bool kFull = decltype(full_c)::value;
      const int64_t base = v0 + tid;
      const int32_t bytes = kBuf ? (int32_t)((vend - v0 < B * U ? vend - v0 : B * U) * 16) : 0;
      Vec<S> a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if constexpr (kBuf) {
          const __amdgpu_buffer_rsrc_t rx =
              __builtin_amdgcn_make_buffer_rsrc((void*)(xv + v0 * KV), (short)0, bytes, 0x00020000);
          const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rx, (uint32_t)(tid + u * B) * 16u, 0, 2);
          __builtin_memcpy(&a[u], &w, 16);
        } else if (kFull || base + u * B < vend) {
          a[u] = load16<S>(xv + (base + u * B) * KV);
        } else {
          a[u] = Vec<S>{};
        }
      }
      elem_t<S> v[N];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < KV; ++k) v[u * KV + k] = a[u].e[k];
      auto ok = [&](int q) { return kFull || base + (q / KV) * B < vend; };
      if constexpr (!std::is_same_v<S, I32>) {
        float tv[N];
#pragma unroll
        for (int q = 0; q < N; ++q) tv[q] = S::widen(v[q]);
        eval_batch(f, tv);
#pragma unroll
        for (int q = 0; q < N; ++q)
          if (ok(q)) acc[q % KV].add(tv[q]);
      } else {
#pragma unroll
        for (int q = 0; q < N; ++q)
          if (ok(q)) fold_elem<F, S>(acc[q % KV], f, v[q], v[q]);
      }
      if (y) {
        elem_t<S> o[N];
        map_batch<FM, S>(fm, v, o);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if constexpr (kBuf) {
            const __amdgpu_buffer_rsrc_t ry =
                __builtin_amdgcn_make_buffer_rsrc((void*)(y + r.head + v0 * KV), (short)0, bytes, 0x00020000);
            u32x4 w;
            __builtin_memcpy(&w, &o[u * KV], 16);
            __builtin_amdgcn_raw_buffer_store_b128(w, ry, (uint32_t)(tid + u * B) * 16u, 0, 2);
          } else if (kFull || base + u * B < vend) {
            Vec<S> ov;
#pragma unroll
            for (int k = 0; k < KV; ++k) ov.e[k] = o[u * KV + k];
            store16_nt<S>(y + r.head + (base + u * B) * KV, ov);
          }
        }
      }
    };
    int64_t v0 = lc * call.chunk_vecs;
    for (; v0 + B * U <= vend; v0 += B * U) step(v0, std::true_type{});
    if (v0 < vend) step(v0, std::false_type{});
    if (lc == 0) {  // the first chunk also takes the unaligned head and tail
      if (tid < r.head) {
        fold_elem<F, S>(acc[0], f, x[tid], x[tid]);
        if (y) y[tid] = map_elem<FM, S>(fm, x[tid]);
      }
      if (tid < r.tail) {
        const int64_t e = r.tail_start + tid;
        fold_elem<F, S>(acc[1 % KV], f, x[e], x[e]);
        if (y) y[e] = map_elem<FM, S>(fm, x[e]);
      }
    }
    Acc tt = acc[0];
#pragma unroll
    for (int k = 1; k < KV; ++k) tt = Acc::merge(tt, acc[k]);
    tt = block_reduce(tt, MergeOp<Acc>{}, lds);
    if constexpr (kOne) {
      const int64_t lo = t.prefix[i], chunks = t.prefix[i + 1] - lo;
      __shared__ int last;
      __shared__ BatchFoldT<Acc> fold_lds[kMaxWaves];
      if (tid == 0) {
        last = 1;
        if (chunks > 1) {
          publish_partial(partials, c, tt);
          last = arrive(ticket + i * kTicketStride, (uint32_t)chunks);
        }
      }
      __syncthreads();
      if (last)
        batch_fold<Acc>([&](int64_t k) { return chunks > 1 ? read_partial(partials, k) : tt; }, lo, lo + chunks,
                        call.out, fold_lds);
      if (c == 0 && tid < t.count && t.prefix[tid + 1] == t.prefix[tid]) write_empty<Acc>(t.call[tid].out);
      return;  // the block's only chunk
    } else {
      if (tid == 0) partials[c] = tt;
    }
  }
}

// One block per call folds that call's chunk partials.
template <class Acc>
__global__ __launch_bounds__(kBatchFold) void batch_combine_kernel(BatchTable t, const Acc* partials) {
  __shared__ BatchFoldT<Acc> lds[kMaxWaves];
  const int c = blockIdx.x;
  batch_fold<Acc>([&](int64_t k) { return partials[k]; }, t.prefix[c], t.prefix[c + 1], t.call[c].out, lds);
}

}  // namespace hdc
