// Launch templates of the kernel families: grid geometry and kernel-instance
// choice (unroll) for one concrete (callable, storage, fold) combination.
#pragma once

#include <type_traits>

#include "hdc_batch.hpp"
#include "hdc_exact.hpp"
#include "hdc_host.hpp"
#include "hdc_scan.hpp"

namespace hdc {

template <class F, class S>
hdc_status launch_map(const F& f, const void* x, void* y, int64_t n, const Tuning& t, hipStream_t st) {
  using T = typename S::T;
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  const bool vec = map_vectors(x, y, n);
  const Range r = vec ? make_range<S>(y, n) : Range{n, 0, 0, 0, 0};
  const int64_t units = vec ? r.nvec : n;
  const int64_t g = grid_for(units, (int64_t)t.block * t.unroll, cus, t);
  auto go = [&](auto U) {
    constexpr int kU = decltype(U)::value;
    if (vec)
      map_kernel<F, S, kU, true><<<dim3((unsigned)g), dim3(t.block), 0, st>>>(f, (const T*)x, (T*)y, r);
    else
      map_kernel<F, S, kU, false><<<dim3((unsigned)g), dim3(t.block), 0, st>>>(f, (const T*)x, (T*)y, r);
  };
  switch (t.unroll) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
  return check_launch("map kernel launch");
}

template <class Acc>
hdc_status launch_final(const Acc* partials, int64_t g, void* out, hipStream_t st) {
  reduce_final_kernel<Acc><<<dim3(1), dim3(kFoldThreads), 0, st>>>(partials, (int)g, out);
  return check_launch("final combine launch");
}

// `ticket`: kTicketCounters zero counters that no other work uses until this call
// completes; with it the reduction is one launch (its last block folds the
// partials), without it (NULL) two launches.  Both fold in the same order, so
// they give the same bits.
template <class F, class S, class Acc, class FM = Identity, bool kMap = false>
hdc_status launch_reduce(const F& f, const void* x, const void* z, int64_t n, void* out, void* ws,
                         uint32_t* ticket, const Tuning& t, hipStream_t st, const FM& fm = FM{},
                         void* y = nullptr) {
  using T = typename S::T;
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  const Range r = make_range<S>(kMap ? y : x, n);
  const int64_t g = grid_for(r.nvec, (int64_t)t.block * t.unroll, cus, t);
  Acc* partials = static_cast<Acc*>(ws);
  auto go = [&](auto U) {
    constexpr int kU = decltype(U)::value;
    reduce_kernel<F, S, Acc, kU, FM, kMap><<<dim3((unsigned)g), dim3(t.block), 0, st>>>(
        f, (const T*)x, (const T*)z, r, partials, ticket, out, fm, (T*)y);
  };
  switch (t.unroll) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
  HDC_TRY(check_launch("reduce kernel launch"));
  if (ticket || g == 1) return HDC_OK;
  return launch_final<Acc>(partials, g, out, st);
}


// Exact bf16 sum: pass 1 over t.block threads (at most kExactMaxBlock: the
// digit accumulators take 64 bytes of LDS per thread) x t.unroll vectors per
// step (1, 2 or 4), at most 4096 blocks (their 48-byte partials fit the
// reduce workspace), then the one-block final combine and rounding.
inline hdc_status launch_exact_bf16(const void* x, int64_t n, void* out, void* ws, uint32_t* ticket,
                                    const Tuning& tuned, hipStream_t st) {
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  Tuning t = tuned;
  if (t.block > kExactMaxBlock) t.block = kExactMaxBlock;
  const Range r = make_range<BF16>(x, n);
  const int u = t.unroll >= 4 ? 4 : t.unroll;
  int64_t g = grid_for(r.nvec, (int64_t)t.block * u, cus, t);
  if (g > 4096) g = 4096;
  // Enough lanes that none takes more than kExactVecsPerLane vectors (its
  // fp64 accumulators stay exact), within the partials the workspace holds.
  const int64_t lanes_needed = (r.nvec + kExactVecsPerLane - 1) / kExactVecsPerLane;
  const int64_t g_min = (lanes_needed + t.block - 1) / t.block;
  constexpr int64_t kMaxExactGrid = (int64_t)(kMaxGrid * kPartialBytes / sizeof(Bf16Partial));
  if (g_min > kMaxExactGrid)
    return fail(HDC_ERR_UNSUPPORTED, "n = %lld is too large for an exact bf16 sum at block %d", (long long)n, t.block);
  if (g < g_min) g = g_min;
  Bf16Partial* partials = static_cast<Bf16Partial*>(ws);
  const uint16_t* xp = static_cast<const uint16_t*>(x);
  double* o = static_cast<double*>(out);
  const dim3 grid((unsigned)g), block(t.block);
  const size_t lds = sizeof(double) * (kExactFoldDigits + 1) * (size_t)t.block;
  if (u == 1)
    exact_bf16_kernel<1><<<grid, block, lds, st>>>(xp, r, partials, ticket, o);
  else if (u == 2)
    exact_bf16_kernel<2><<<grid, block, lds, st>>>(xp, r, partials, ticket, o);
  else
    exact_bf16_kernel<4><<<grid, block, lds, st>>>(xp, r, partials, ticket, o);
  HDC_TRY(check_launch("exact bf16 launch"));
  if (ticket || g == 1) return HDC_OK;
  exact_bf16_final_kernel<<<dim3(1), dim3(256), 0, st>>>(partials, (int)g, o);
  return check_launch("exact bf16 final launch");
}

// Exact fp16 dot product, in vectors aligned to x.
inline hdc_status launch_exact_f16_dot(const void* x, const void* z, int64_t n, void* out, void* ws,
                                       uint32_t* ticket, const Tuning& t, hipStream_t st) {
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  const Range r = make_range<F16>(x, n);
  const bool even = ((uintptr_t)z - (uintptr_t)x) % 4 == 0;
  const int u = t.unroll >= 4 ? 4 : t.unroll;
  int64_t g = grid_for(r.nvec, (int64_t)t.block * u, cus, t);
  if (g > 4096) g = 4096;
  F16DotExact* partials = static_cast<F16DotExact*>(ws);
  const uint16_t* xp = static_cast<const uint16_t*>(x);
  double* o = static_cast<double*>(out);
  const uint16_t* zp = static_cast<const uint16_t*>(z);
  const dim3 grid((unsigned)g), block(t.block);
  auto go = [&](auto U) {
    constexpr int kU = decltype(U)::value;
    if (even)
      exact_f16_dot_kernel<kU, true><<<grid, block, 0, st>>>(xp, zp, r, partials, ticket, o);
    else
      exact_f16_dot_kernel<kU, false><<<grid, block, 0, st>>>(xp, zp, r, partials, ticket, o);
  };
  switch (u) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    default: go(std::integral_constant<int, 4>{}); break;
  }
  HDC_TRY(check_launch("exact fp16 dot launch"));
  if (ticket || g == 1) return HDC_OK;
  exact_f16_dot_final_kernel<<<dim3(1), dim3(256), 0, st>>>(partials, (int)g, o);
  return check_launch("exact fp16 dot final launch");
}

// Tiled schedule of the segmented reduce (t.passes == 1): the tile pass and
// the fold of segments that span tiles, by one block (in the same launch, if a
// ticket is left) when it can hold all tiles and the segments are not far more
// than the elements (their zeros take the wavefronts of the second launch, which
// are by the segments), else in a second one.  The workspace is counted in
// two halves of 32 bytes per tile.
//
// `total` bounds the elements (it comes with the workspace).  Few elements are
// cut into smaller tiles than the tuning's, down to kMinChunk elements, while
// there are fewer tiles than kMinTiles: with 4096 elements a tile, 300,000
// would occupy 73 of the chip's 1024 SIMDs.
constexpr int64_t kMinTiles = 512;
// Tiles of more than kLongTile elements, which pay where there are many, are
// halved below kMinLongTiles where the mean segment is shorter than such a
// tile.  8192 / 4096 elements a tile, us: 1.7e7 f32 in segments of 1340 29.9 /
// 24.5, of 48 53.1 / 40.1; bf16 compensated 35.7 / 29.0, 48.6 / 37.3; 5e7 f32
// in segments of 300 68.4 / 61.7.  Longer segments have more parts to fold:
// 3e7 f32 in segments of 30000 30.8 / 33.8.
constexpr int64_t kLongTile = 4096;
constexpr int64_t kMinLongTiles = 8192;
// Where segments are shorter than kShortMean on average, a tile's chunks with
// many ends one after another are a chain of 1.5 to 3 us each, and a tile costs
// a search: tiles are halved while there are fewer than one and a half per
// element of a tile.  (Lengths in rising order, so that the short ones share
// tiles, mean 500: 4e6 f32 plain 29.7 -> 18.8 us; in lognormal segments of 1000
// 6e6 bf16 would take 26.5 in place of 22.5.)
// Elements a tile 1024 / 2048 / 4096 / 8192, us a call, segments of 64 (f32
// plain; bf16 compensated in brackets): 4e6 14.4 / 17.7 / 28.4 / - (12.0 / 13.0
// / 18.2), 8e6 23.4 / 21.9 / 28.8 / - (18.2 / 17.7 / 20.6), 1.7e7 39.5 / 37.6 /
// 40.7 / - (31.7 / 29.8 / 31.6), 7e7 131 / 117 / 112 / 120 (105 / 90 / 87 / 92).
constexpr int64_t kShortMean = 768;
constexpr int64_t short_min_tiles(int64_t tile) { return tile + tile / 2; }

template <class F, class S, class Acc>
hdc_status launch_seg_tiles(const F& f, const void* x, const int64_t* off, int64_t nseg, int64_t total, void* out,
                            void* ws, size_t ws_bytes, uint32_t* ticket, const Tuning& t, hipStream_t st) {
  using T = typename S::T;
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  const size_t half = ws_bytes / 2 / 256 * 256;
  const int block = t.block < kTilesMaxBlock ? t.block : kTilesMaxBlock;
  int64_t tile = t.chunk;
  auto few = [&] {
    if (nseg * kShortMean > total) return short_min_tiles(tile);
    return tile > kLongTile && nseg > total / (2 * kLongTile) ? kMinLongTiles : kMinTiles;
  };
  while (tile > kMinChunk && total / tile < few()) tile /= 2;
  SegTiles tl;
  tl.cap = (int64_t)(half / kPartialBytes);
  tl.first = static_cast<uint64_t*>(ws);
  tl.last = reinterpret_cast<uint64_t*>(static_cast<char*>(ws) + half);
  tl.meta = tl.first + tl.cap;  // 8 of a slot's 32 bytes are its fold state
  tl.tile_vecs = tile / S::kVec;
  tl.crowded = tile / kCrowdedLen < kMostEnds ? (int32_t)(tile / kCrowdedLen) : kMostEnds;
  int64_t tiles = total / tile + 2;  // at most: the head joins the first tile, the tail the last
  if (tiles > tl.cap) tiles = tl.cap;
  // by the sizes alone, not by whether a ticket is left: the passes and folds that follow give other bits
  tl.one = tiles <= seg_last_tiles(block) && nseg <= kMinChunk * tiles;
  if (!tl.one) ticket = nullptr;
  // a range of more elements than the workspace is sized for must not exceed the block's tiles
  if (tl.one && tl.cap > seg_last_tiles(block)) tl.cap = seg_last_tiles(block);
  const int64_t wpb = block / 64;
  int64_t g = (int64_t)cus * t.grid_mult;
  const int64_t need = (tiles + wpb - 1) / wpb;  // never more wavefronts than tiles
  if (g > need) g = need;
  if (g < 1) g = 1;
  const bool dense = tl.one || nseg * kDenseVecs * S::kVec > total;
  auto go = [&](auto U) {
    constexpr int kU = decltype(U)::value;
    if (dense)
      seg_tiles_kernel<F, S, Acc, kU, true>
          <<<dim3((unsigned)g), dim3(block), sizeof(DenseLds<S, Acc>) * (size_t)wpb, st>>>(f, (const T*)x, off, nseg,
                                                                                         tl, ticket, out);
    else
      seg_tiles_kernel<F, S, Acc, kU, false><<<dim3((unsigned)g), dim3(block), 0, st>>>(f, (const T*)x, off, nseg, tl,
                                                                                       ticket, out);
  };
  switch (t.unroll) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
  HDC_TRY(check_launch("segmented tile launch"));
  if (ticket) return HDC_OK;
  if (tl.one) {
    seg_last_kernel<S, Acc><<<dim3(1), dim3(block), 0, st>>>((const T*)x, off, nseg, tl, out);
    return check_launch("segmented last-fold launch");
  }
  // Up to 8 wavefronts per compute unit, of at most 64 segments at a time: a
  // wavefront folds its wide segments one by one (100 segments of 500,000 bf16
  // in two wavefronts: 87 us a call, in a wavefront each 28).
  const int64_t waves = (int64_t)cus * 8;
  int32_t per = 1;
  while (per < 64 && per * waves < nseg) per *= 2;
  int64_t gc = ((nseg + per - 1) / per + 3) / 4;
  // Parts of a crowded tile: its chunks one after another are a chain of 1.5 to
  // 3 us each, a part costs three searches (~5 us).  As many as give the
  // wavefronts four parts each if all segments lie in crowded tiles, of two
  // chunks at least.
  int32_t lg = 0;
  if (!dense && nseg > tl.crowded) {
    if (gc < waves / 4) gc = waves / 4;
    while ((nseg / tl.crowded << (lg + 1)) <= 4 * waves && (tl.tile_vecs >> (lg + 1)) >= 128) ++lg;
  }
  if (gc > (int64_t)cus * 8) gc = (int64_t)cus * 8;
  const dim3 cgrid((unsigned)gc), cblock(256);
  if (dense)
    seg_tiles_combine_kernel<S, Acc><<<cgrid, cblock, 0, st>>>((const T*)x, off, nseg, per, tl, out);
  else
    seg_tiles_combine_crowded_kernel<F, S, Acc>
        <<<cgrid, cblock, 0, st>>>(f, (const T*)x, off, nseg, per, lg, tl, out);
  return check_launch("segmented tile combine launch");
}

template <class F, class S, class Acc>
hdc_status launch_segmented(const F& f, const void* x, const int64_t* off, int64_t nseg, int64_t total, void* out,
                            void* ws, size_t ws_bytes, uint32_t* ticket, const Tuning& t, hipStream_t st) {
  using T = typename S::T;
  if (t.passes == 1)
    return launch_seg_tiles<F, S, Acc>(f, x, off, nseg, total, out, ws, ws_bytes, ticket, t, st);
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  const int64_t cap = seg_capacity(ws_bytes, nseg);
  if (cap < 1) return fail(HDC_ERR_WORKSPACE, "workspace of %zu bytes is too small for %lld segments", ws_bytes,
                           (long long)nseg);
  const SegLayout l = seg_layout_cap(cap, nseg);
  char* base = static_cast<char*>(ws);
  SegPlan p;
  p.cnt = reinterpret_cast<SegCounters*>(base + l.cnt);
  p.block_tot = reinterpret_cast<SegCounters*>(base + l.block_tot);
  p.full_list = reinterpret_cast<SegPiece*>(base + l.full);
  p.part_list = reinterpret_cast<SegPiece*>(base + l.part);
  p.long_base = reinterpret_cast<int32_t*>(base + l.long_base);
  p.long_list = reinterpret_cast<int32_t*>(base + l.long_list);
  p.partials = base + l.partials;
  p.cap_full = l.cap_full;
  p.cap_part = l.cap_part;
  p.cap_partials = l.cap_partials;
  p.chunk = t.chunk;
  p.small_seg = t.small_seg;
  p.spw = t.seg_per_wave;

  seg_count_kernel<<<dim3((unsigned)l.plan_blocks), dim3(kPlanBlock), 0, st>>>(off, nseg, p);
  HDC_TRY(check_launch("segmented count launch"));
  seg_count_scan_kernel<<<dim3(1), dim3(1024), 0, st>>>(l.plan_blocks, p);
  HDC_TRY(check_launch("segmented count-scan launch"));
  seg_write_kernel<<<dim3((unsigned)l.plan_blocks), dim3(kPlanBlock), 0, st>>>(off, nseg, p);
  HDC_TRY(check_launch("segmented plan launch"));

  // Persistent grid: enough wavefronts to fill the chip, never more than the
  // largest possible item count needs.
  const int64_t wpb = t.block / 64;
  const int64_t max_items = l.cap_full + l.cap_part + (nseg + p.spw - 1) / p.spw;
  int64_t g = (int64_t)cus * t.grid_mult;
  const int64_t need = (max_items + wpb - 1) / wpb;
  if (g > need) g = need;
  if (g < 1) g = 1;
  auto go = [&](auto U) {
    constexpr int kU = decltype(U)::value;
    seg_items_kernel<F, S, Acc, kU><<<dim3((unsigned)g), dim3(t.block), 0, st>>>(f, (const T*)x, off, nseg, p,
                                                                                 out);
  };
  switch (t.unroll) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
  HDC_TRY(check_launch("segmented item launch"));
  int64_t gc = (nseg + 3) / 4;
  if (gc > (int64_t)cus * 8) gc = (int64_t)cus * 8;
  if (gc < 1) gc = 1;
  seg_combine_kernel<Acc><<<dim3((unsigned)gc), dim3(256), 0, st>>>(off, nseg, p, out);
  return check_launch("segmented combine launch");
}

template <class FM, class F, class S, class Acc>
hdc_status launch_batch(const FM& fm, bool maps, const F& f, const hdc_batch_call* calls, const int32_t* idx,
                        const int* chunk, int cnt, void* ws, size_t ws_bytes, uint32_t* ticket, const Tuning& t,
                        hipStream_t st) {
  int cus = 0;
  HDC_TRY(compute_units(&cus));
  BatchTable tab{};
  tab.count = cnt;
  int64_t acc_chunks = 0, most = 0;  // of all calls, of one call
  for (int q = 0; q < cnt; ++q) {
    const hdc_batch_call& c = calls[idx[q]];
    BatchCall& b = tab.call[q];
    b.x = c.x;
    b.y = maps ? c.y : nullptr;
    b.out = c.out;
    b.r = make_range<S>(b.y ? b.y : c.x, c.n);
    Tuning own = t;
    own.chunk = chunk[q];
    b.chunk_vecs = batch_chunk_vecs(own, S::kVec);
    tab.prefix[q] = acc_chunks;
    if (c.n > 0) {
      int64_t nc = (b.r.nvec + b.chunk_vecs - 1) / b.chunk_vecs;
      acc_chunks += nc > 0 ? nc : 1;
      if (nc > most) most = nc;
    }
  }
  tab.prefix[cnt] = acc_chunks;
  if ((size_t)acc_chunks * sizeof(Acc) > ws_bytes)
    return fail(HDC_ERR_WORKSPACE, "the batch needs %lld chunk partials (%zu bytes) but the workspace holds %zu bytes",
                (long long)acc_chunks, (size_t)acc_chunks * sizeof(Acc), ws_bytes);
  Acc* partials = static_cast<Acc*>(ws);
  if (acc_chunks > 0) {
    int64_t g = (int64_t)cus * t.grid_mult;
    // One launch where the chunks are no more than the compute units (a block
    // per chunk, so an arrival is paid once) and no call has more than 64: a
    // call's arrivals queue on its counter, ~27 ns each.  One call of up to 4096
    // elements 11.1 -> 7.5 us, 11 of them 15.8 -> 13.4, 32 28.4 -> 26.6; but 4
    // calls of up to 2^22 int32 (256 chunks in the largest) 13.2 against 14.7.
    if (acc_chunks > cus || most > 64 || t.block < kBatchFold) ticket = nullptr;
    if (g > acc_chunks) g = acc_chunks;
    auto go = [&](auto U) {
      constexpr int kU = decltype(U)::value;
      const dim3 grid((unsigned)g), block(t.block);
      if (ticket)
        batch_kernel<FM, F, S, Acc, kU, true><<<grid, block, 0, st>>>(fm, f, tab, partials, ticket);
      else
        batch_kernel<FM, F, S, Acc, kU, false><<<grid, block, 0, st>>>(fm, f, tab, partials, nullptr);
    };
    switch (t.unroll) {
      case 1: go(std::integral_constant<int, 1>{}); break;
      case 2: go(std::integral_constant<int, 2>{}); break;
      case 4: go(std::integral_constant<int, 4>{}); break;
      default: go(std::integral_constant<int, 8>{}); break;
    }
    HDC_TRY(check_launch("batch launch"));
    if (ticket) return HDC_OK;
  }
  batch_combine_kernel<Acc><<<dim3((unsigned)cnt), dim3(256), 0, st>>>(tab, partials);
  return check_launch("batch combine launch");
}

// Scan: t.unroll == 1 selects the three-pass schedule, any other value the
// single pass.  `seg` carries the segment offsets of a segmented scan (Acc a
// SegAcc), else nothing.  Workspace (scan_workspace_bytes):
//   three passes: 256-byte header (status) | tile sums | tile offsets, one
//                 fold state per tile each;
//   single pass:  256-byte header (ticket, status) | the tree nodes
//                 (tree_nodes(G), level by level), kWords 8-byte words each.
// `slot`: library memory for the look-back nodes of all the single pass's tiles
// (kScanSlotWords or kScanLongWords words), or NULL.
template <class F, class S, class Acc>
hdc_status launch_scan(const F& f, const void* x, void* y, int64_t n, int exclusive, SegSpec seg, void* ws,
                       uint64_t* slot, const Tuning& t, hipStream_t st) {
  using T = typename S::T;
  using OutT = typename ScanOut<Acc>::T;
  static_assert(sizeof(Acc) <= 24, "scan_workspace_bytes holds 24 bytes per tile and array");
  const int64_t narrow = (int64_t)t.block * kScanE;
  if ((n + narrow - 1) / narrow * t.block > (int64_t)UINT32_MAX)
    return fail(HDC_ERR_UNSUPPORTED, "n = %lld is too large for one scan", (long long)n);
  // 2-byte storage that does not start on 4-byte boundaries takes global loads
  const bool even = (uintptr_t)x % 4 == 0;
  const bool wide = ScanWide<Acc>::value && t.unroll != 1 && n >= kScanWideN && (sizeof(T) == 4 || even);
  const int64_t tile = wide ? 2 * narrow : narrow;
  const int64_t G = (n + tile - 1) / tile;
  const T* xp = static_cast<const T*>(x);
  OutT* yp = static_cast<OutT*>(y);
  const dim3 grid((unsigned)G), block(t.block);
  if (t.unroll != 1) {
    // The look-back nodes: none for one tile, a library slot, else the
    // workspace, cleared first.  (The clear is a launch of its own, ~4 us of the
    // host's time and ~2 us of the card's: 112,000 f32 12.3 -> 6.7 us without it,
    // 5e6 f32 17.2 -> 15.2, 1.34e8 209.2 -> 206.7.)
    uint64_t* w = static_cast<uint64_t*>(ws);
    uint32_t* const status = static_cast<uint32_t*>(ws) + 1;
    ScanLB lb{static_cast<uint32_t*>(ws), nullptr, status, w + 32, 1};
    if (G > 1 && slot) {
      lb.ticket64 = slot;
      lb.node = slot + 16;
    } else if (G > 1) {
      const int64_t nwords = 32 + (int64_t)ScanCarry<Acc>::kWords * tree_nodes(G);
      const int64_t cb = (nwords + 255) / 256;
      scan_lb_clear_kernel<<<dim3((unsigned)(cb < 1024 ? cb : 1024)), dim3(256), 0, st>>>(w, nwords);
      HDC_TRY(check_launch("scan look-back clear launch"));
    }
    if (wide) {
      if constexpr (ScanWide<Acc>::value)
        scan_onepass_kernel<F, S, Acc, 2 * kScanE, true><<<grid, block, 0, st>>>(f, xp, n, seg, lb, yp, exclusive);
    } else if (sizeof(T) == 4 || even) {
      scan_onepass_kernel<F, S, Acc, kScanE, true><<<grid, block, 0, st>>>(f, xp, n, seg, lb, yp, exclusive);
    } else if constexpr (sizeof(T) < 4) {
      scan_onepass_kernel<F, S, Acc, kScanE, false><<<grid, block, 0, st>>>(f, xp, n, seg, lb, yp, exclusive);
    }
    return check_launch("scan single-pass launch");
  }
  // three passes: the same 256-byte header (its status word cleared by the
  // offsets pass), then the tile sums and the tile offsets
  Acc* sums = reinterpret_cast<Acc*>(static_cast<char*>(ws) + 256);
  Acc* offsets = reinterpret_cast<Acc*>(static_cast<char*>(ws) + 256 + round_up((size_t)G * sizeof(Acc), 256));
  if (sizeof(T) == 4 || even)
    scan_tile_sums_kernel<F, S, Acc, true><<<grid, block, 0, st>>>(f, xp, n, seg, sums);
  else if constexpr (sizeof(T) < 4)
    scan_tile_sums_kernel<F, S, Acc, false><<<grid, block, 0, st>>>(f, xp, n, seg, sums);
  HDC_TRY(check_launch("scan tile-sum launch"));
  scan_offsets_kernel<Acc><<<dim3(1), dim3(1024), 0, st>>>(sums, G, offsets, static_cast<uint32_t*>(ws) + 1);
  HDC_TRY(check_launch("scan offset launch"));
  if (sizeof(T) == 4 || even)
    scan_tiles_kernel<F, S, Acc, true><<<grid, block, 0, st>>>(f, xp, n, seg, offsets, yp, exclusive);
  else if constexpr (sizeof(T) < 4)
    scan_tiles_kernel<F, S, Acc, false><<<grid, block, 0, st>>>(f, xp, n, seg, offsets, yp, exclusive);
  return check_launch("scan tile launch");
}

}  // namespace hdc
