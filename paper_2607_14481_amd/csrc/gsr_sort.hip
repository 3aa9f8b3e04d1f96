// gsr_sort.hip -- binning stages of the rasterizer on gfx950:
//   A2 scans: visible-item compaction and per-item pair offsets (exclusive
//      scans in u32 with saturating adds, reduce-then-scan, no spin waits)
//   A3-A5 binning: the (depth bits, item) entries of each tile's list, grouped
//      by tile in no particular order, and each list's [start, end)
//   A4c per-tile depth order: each tile's list sorted by (depth bits, item)
//
// Order of work.  The pairs must end up sorted by (tile, depth bits, item).
// The tiles of one view are few enough for one counter each in a workgroup's
// LDS, so the grouping by tile is one counting sort with a digit per tile: a
// pass that counts (k_bin_count), a column scan (k_bin_scan) and a pass that
// places every pair (k_bin_place); the pairs are generated from the items'
// tile boxes in both passes and never stored unsorted.  One workgroup per tile
// then sorts its short list by (depth bits, item) in LDS: the result is the
// (tile, depth, item) order exactly, whatever order a tile's list had before.
//
// Every kernel reads its element count from the workspace header, so the
// launch grid can be sized for a capacity and the call needs no host
// synchronisation (graph capture).
#include <algorithm>

#include "gsr_internal.h"

namespace gsr {

__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) {
    const uint32_t s = a + b;
    return s < a ? 0xffffffffu : s;
}

// Block-wide exclusive scan of one value per thread (256 threads), saturating.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t *lds /* [4] */, uint32_t &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(x, sat_add);
    if (lane == 63) lds[w] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int k = 0; k < w; ++k) before = sat_add(before, lds[k]);
    total = sat_add(sat_add(lds[0], lds[1]), sat_add(lds[2], lds[3]));
    __syncthreads();
    return sat_add(before, inc - x);
}

// ---------------------------------------------------------------------------
// Ordered compaction of byte flags, reduce-then-scan: out_idx receives, in
// ascending order, the indices i < n with flags[i] != 0; their number goes to
// *out_count.  Phase 1 counts each block of kScanTile flags; phase 2 writes a
// block's indices from the sum of the blocks before it, which each block adds
// up itself while they are few (kFlagFewBlocks) and a launch between scans
// otherwise: 4.6 M flags, 4,464 blocks, take 14.6 us with the one and 20.6 us with
// the other.
// ---------------------------------------------------------------------------
constexpr uint32_t kFlagFewBlocks = 8192;

// The flags of items [base, base + 4) (base a multiple of 4, flags aligned) as
// bits; none past n.
__device__ __forceinline__ uint32_t four_flags(const uint8_t *__restrict__ flags, uint64_t base, uint64_t n) {
    static_assert(kScanItems == 4, "a thread's flags are one word");
    uint32_t bits = 0;
    if (base + 4 <= n) {
        const uint32_t w = *reinterpret_cast<const uint32_t *>(flags + base);
#pragma unroll
        for (int k = 0; k < 4; ++k) bits |= ((w >> (8 * k) & 0xffu) ? 1u : 0u) << k;
    } else {
        for (int k = 0; k < 4; ++k) bits |= (base + k < n && flags[base + k] ? 1u : 0u) << k;
    }
    return bits;
}

__global__ __launch_bounds__(kScanThreads) void k_flag_count(const uint8_t *__restrict__ flags, uint64_t n,
                                                             uint32_t *__restrict__ block_sums) {
    __shared__ uint32_t lds[4];
    uint32_t total;
    block_exclusive_scan(
        (uint32_t)__popc(four_flags(flags, (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems, n)),
        lds, total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// Single workgroup: exclusive scan of nb block sums in place.
__global__ __launch_bounds__(1024) void k_scan_blocks(uint32_t *__restrict__ block_sums, uint32_t nb) {
    __shared__ uint32_t lds[16];
    __shared__ uint32_t carry;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < nb; base += 1024) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < nb ? block_sums[i] : 0u;
        const uint32_t inc = wave_inclusive_scan(x, sat_add);
        if (lane == 63) lds[w] = inc;
        __syncthreads();
        uint32_t before = carry;
        for (int k = 0; k < w; ++k) before = sat_add(before, lds[k]);
        if (i < nb) block_sums[i] = sat_add(before, inc - x);
        __syncthreads();
        if (threadIdx.x == 1023) carry = sat_add(before, inc);
        __syncthreads();
    }
}

// scanned: block_sums holds the sums of the blocks before, not the blocks' own.
__global__ __launch_bounds__(kScanThreads) void k_flag_compact_apply(const uint8_t *__restrict__ flags, uint64_t n,
                                                                     const uint32_t *__restrict__ block_sums,
                                                                     int scanned, uint32_t *__restrict__ out_idx,
                                                                     uint32_t *__restrict__ out_count) {
    __shared__ uint32_t lds[4], s_before[4];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    const uint32_t bits = four_flags(flags, base, n);
    uint32_t before = 0;
    if (scanned) {
        before = block_sums[blockIdx.x];
    } else {
        for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kScanThreads) before += block_sums[j];
        before = wave_reduce(before, 0u, sat_add);
        if ((threadIdx.x & 63) == 0) s_before[threadIdx.x >> 6] = before;
        __syncthreads();
        before = s_before[0] + s_before[1] + s_before[2] + s_before[3];
    }
    uint32_t total;
    uint32_t pos = before + block_exclusive_scan((uint32_t)__popc(bits), lds, total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (bits & (1u << k)) out_idx[pos++] = (uint32_t)(base + k);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *out_count = before + total;
}

void launch_compact_flags(const uint8_t *flags, uint64_t n, uint32_t *out_idx, uint32_t *block_tmp,
                          uint32_t *out_count, hipStream_t st) {
    const uint32_t nb = (uint32_t)((n + kScanTile - 1) / kScanTile);
    if (nb == 0) return;
    const bool few = nb <= kFlagFewBlocks;
    hipLaunchKernelGGL(k_flag_count, dim3(nb), dim3(kScanThreads), 0, st, flags, n, block_tmp);
    if (!few) hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, st, block_tmp, nb);
    hipLaunchKernelGGL(k_flag_compact_apply, dim3(nb), dim3(kScanThreads), 0, st, flags, n, block_tmp, few ? 0 : 1,
                       out_idx, out_count);
}

// ---------------------------------------------------------------------------
// A2 in one reduce-then-scan over the items, with two values per item: visible
// (tiles touched > 0) and its tile count.  An invisible item counts zero tiles,
// so the pair offset of the k-th visible item is the prefix of the counts over
// all items before it.  Phase 1 sums each block of kScanTile items; phase 2
// gives each block the sums of the blocks before it (each block adds them up
// itself: at most a few thousand L2-resident values, no extra launch) and
// writes the k-th visible item's id, pair offset and box and, for each
// chunk of kChunkPairs pair slots whose first pair the item holds, k; each
// view's first visible index too.  The last block writes the visible and pair
// counts and the overflow decision (pairs > capacity).
//
// It moves 44 bytes per visible item and 4 per item (8 with phase 1), with every
// access contiguous except for the gaps of the invisible ones: the projection leaves the box words in an
// array of their own and the pair offset by item goes to another.  (Read from
// and written into the records themselves, 48 bytes apart, both touched every
// line of theirs for one word: 132 us for 8 views of 1 M items, 63 us now.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kScanThreads) void k_vis_reduce(const uint32_t *__restrict__ count, uint64_t n,
                                                             uint32_t *__restrict__ block_vis,
                                                             uint32_t *__restrict__ block_pairs) {
    __shared__ uint32_t lds[4];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    uint32_t nv = 0, np = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t c = base + k < n ? count[base + k] : 0u;
        nv += c > 0u ? 1u : 0u;
        np = sat_add(np, c);
    }
    uint32_t tv, tp;
    block_exclusive_scan(nv, lds, tv);
    block_exclusive_scan(np, lds, tp);
    if (threadIdx.x == 0) {
        block_vis[blockIdx.x] = tv;
        block_pairs[blockIdx.x] = tp;
    }
}

// Blocks up to which phase 2 reads the counts of the blocks before it itself,
// which saves phase 1's launch (2 us in a trace of 1,000 items); with 16 blocks
// (16,000 items) a forward was 1.5 us slower so.
constexpr uint32_t kScanFewBlocks = 8;

__global__ __launch_bounds__(kScanThreads) void k_vis_apply(ViewTable vt, uint64_t n_view,
                                                            const uint32_t *__restrict__ count,
                                                            const uint4 *__restrict__ box, uint64_t n,
                                                            const uint32_t *__restrict__ block_vis,
                                                            const uint32_t *__restrict__ block_pairs,
                                                            uint32_t *__restrict__ vis, uint32_t *__restrict__ poff,
                                                            uint32_t *__restrict__ ioff,
                                                            uint4 *__restrict__ item_box,
                                                            uint32_t *__restrict__ chunk_item, uint64_t chunks_cap,
                                                            uint32_t *__restrict__ view_seg,
                                                            WsHeader *__restrict__ hdr) {
    // The block's kScanTile items in kScanItems rounds of kScanThreads
    // consecutive ones (round k, thread t: item base + k kScanThreads + t), so
    // that every load and store of a round is row-contiguous across the wave.
    // Per wave and round: the inclusive totals of the visible flags and the
    // pair counts; last, the wave's part of the sums of the blocks before.
    constexpr int kV = kScanItems * 2;
    __shared__ uint32_t s_w[4][kV + 2];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t c[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint64_t it = base + (uint64_t)k * kScanThreads + tid;
        c[k] = it < n ? count[it] : 0u;
    }
    // the visible items' boxes, all requested before the scans (the others ask for
    // the block's first: under a branch the four loads waited for each other, 27
    // against 23 us for 4 views of 700 k)
    uint4 bw[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) bw[k] = box[c[k] > 0u ? base + (uint64_t)k * kScanThreads + tid : base];
    // the sums of the blocks before this one, from phase 1 or, without it, from
    // their counts
    uint32_t bv = 0, bp = 0;
    if (block_vis) {
        for (uint32_t j = tid; j < blockIdx.x; j += kScanThreads) {
            bv += block_vis[j];
            bp = sat_add(bp, block_pairs[j]);
        }
    } else {
        const uint4 *c4 = reinterpret_cast<const uint4 *>(count);
        for (uint32_t j = 0; j < blockIdx.x; ++j) {  // (kScanTile items are kScanThreads words)
            const uint4 x = c4[(size_t)j * kScanThreads + tid];
            bv += (x.x > 0u ? 1u : 0u) + (x.y > 0u ? 1u : 0u) + (x.z > 0u ? 1u : 0u) + (x.w > 0u ? 1u : 0u);
            bp = sat_add(bp, sat_add(sat_add(x.x, x.y), sat_add(x.z, x.w)));
        }
    }
    bv = wave_reduce(bv, 0u, sat_add);
    bp = wave_reduce(bp, 0u, sat_add);
    uint32_t fv[kScanItems], fp[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        fv[k] = wave_inclusive_scan(c[k] > 0u ? 1u : 0u, sat_add);
        fp[k] = wave_inclusive_scan(c[k], sat_add);
    }
    if (lane == kWave - 1) {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) s_w[w][k] = fv[k], s_w[w][kScanItems + k] = fp[k];
        s_w[w][kV] = bv;
        s_w[w][kV + 1] = bp;
    }
    __syncthreads();
    uint32_t v0 = 0, p0 = 0;  // visible items and pairs before the current round
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) v0 = sat_add(v0, s_w[ww][kV]), p0 = sat_add(p0, s_w[ww][kV + 1]);
    uint32_t kv[kScanItems], run[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        uint32_t ov = 0, op = 0, tv = 0, tp = 0;  // waves before this one; the whole round
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            if (ww < w) ov = sat_add(ov, s_w[ww][k]), op = sat_add(op, s_w[ww][kScanItems + k]);
            tv = sat_add(tv, s_w[ww][k]);
            tp = sat_add(tp, s_w[ww][kScanItems + k]);
        }
        kv[k] = sat_add(sat_add(v0, ov), fv[k] - (c[k] > 0u ? 1u : 0u));
        run[k] = sat_add(sat_add(p0, op), fp[k] - c[k]);
        v0 = sat_add(v0, tv);
        p0 = sat_add(p0, tp);
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        hdr->n_visible = v0;
        hdr->n_pairs = p0;
        hdr->overflow = p0 > hdr->pair_capacity ? 1u : 0u;
        view_seg[vt.n_views] = v0;
        view_seg[GSR_MAX_VIEWS + 1 + vt.n_views] = p0;
    }
    // the first visible index and the first pair of each view that starts here
    for (uint64_t v = (base + n_view - 1) / n_view; v * n_view < min(base + kScanTile, n); ++v) {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + (uint64_t)k * kScanThreads + tid == v * n_view) {
                view_seg[v] = kv[k];
                view_seg[GSR_MAX_VIEWS + 1 + v] = run[k];
            }
    }
    uint32_t infinite = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (c[k] > 0u) {
            const uint32_t item = (uint32_t)(base + (uint64_t)k * kScanThreads + tid);
            vis[kv[k]] = item;
            poff[kv[k]] = run[k];
            ioff[item] = run[k];
            item_box[kv[k]] = make_uint4(bw[k].x, bw[k].y, bw[k].z, item);
            infinite |= bw[k].w;
            // chunks whose first pair lies in [run, run + c)
            const uint32_t end = sat_add(run[k], c[k]);
            for (uint64_t ch = chunk_count(run[k]); ch < chunks_cap && ch * kChunkPairs < end; ++ch)
                chunk_item[ch] = kv[k];
        }
    }
    if (infinite) hdr->infinite = 1u;  // (whoever writes it writes the same)
}

void launch_visible_offsets(const ViewTable &vt, uint64_t n, const uint32_t *count, const uint4 *box, uint64_t items,
                            uint32_t *vis, uint32_t *poff, uint32_t *ioff, uint4 *item_box, uint32_t *chunk_item,
                            uint64_t chunks_cap, uint32_t *block_tmp, uint32_t *view_seg, WsHeader *hdr,
                            hipStream_t st) {
    const uint32_t nb = (uint32_t)((items + kScanTile - 1) / kScanTile);
    if (nb == 0) {
        launch_fill_u32(view_seg, 0u, 2 * (GSR_MAX_VIEWS + 1), st);
        return;
    }
    static_assert(kScanItems == 4, "a block's counts are one uint4 a thread");
    uint32_t *bv = block_tmp, *bp = block_tmp + nb;
    if (nb <= kScanFewBlocks)
        bv = bp = nullptr;
    else
        hipLaunchKernelGGL(k_vis_reduce, dim3(nb), dim3(kScanThreads), 0, st, count, items, bv, bp);
    hipLaunchKernelGGL(k_vis_apply, dim3(nb), dim3(kScanThreads), 0, st, vt, n, count, box, items, bv, bp, vis, poff,
                       ioff, item_box, chunk_item, chunks_cap, view_seg, hdr);
}

__global__ __launch_bounds__(256) void k_export_items(const uint32_t *__restrict__ poff,
                                                      const uint4 *__restrict__ item_box,
                                                      const Rec *__restrict__ rec, const WsHeader *__restrict__ hdr,
                                                      uint64_t items, float *__restrict__ records,
                                                      float *__restrict__ centre_lo,
                                                      uint32_t *__restrict__ depth_keys) {
    const uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= min((uint64_t)hdr->n_visible, items)) return;
    const uint4 bw = item_box[k];
    const Rec r = rec[bw.w];
    if (records) {
        const auto colour = [](float c) { return c == kColourMax ? __builtin_inff() : c; };
        const float w[kExportWords] = {r.r0.x, r.r0.y, r.r0.z, r.r0.w, r.r1.x, r.r1.y, colour(r.r1.z), colour(r.r1.w),
                                       colour(r.r2.x), r.r2.y, r.r2.z, __uint_as_float(poff[k])};
        for (int c = 0; c < kExportWords; ++c) records[(size_t)bw.w * kExportWords + c] = w[c];
    }
    if (centre_lo) centre_lo[2 * (size_t)bw.w] = r.r3.x, centre_lo[2 * (size_t)bw.w + 1] = r.r3.y;
    if (depth_keys) depth_keys[bw.w] = bw.z;
}

void launch_export_items(const uint32_t *poff, const uint4 *item_box, const Rec *rec, const WsHeader *hdr,
                         uint64_t items, float *records, float *centre_lo, uint32_t *depth_keys, hipStream_t st) {
    if (items == 0 || (!records && !centre_lo && !depth_keys)) return;
    if (depth_keys) launch_fill_u32(depth_keys, kCulledKey, items, st);
    hipLaunchKernelGGL(k_export_items, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, poff, item_box, rec, hdr,
                       items, records, centre_lo, depth_keys);
}

// ---------------------------------------------------------------------------
// A3-A5: the counting sort by tile.  A view's visible items are cut into G
// shares (groups of kBinGroup consecutive items, dealt round robin, so that the
// shares get about as many pairs each) and its rows of tiles into bands; a
// workgroup takes one share in one band.
//   k_bin_count  counts the share's pairs per tile of the band and writes them
//                into row g of the count matrix.  A tile's count is a 2-D
//                prefix sum: an item adds four corners of its box to a
//                difference array in LDS, however many tiles it covers;
//   k_bin_scan   per tile: the exclusive scan over the rows in place, and the
//                tile's total;
//   k_bin_place  scans the view's tile totals (every workgroup itself: no
//                launch between), adds its row, and places its pairs with LDS
//                counters as cursors (the pairs come from the items' boxes, a
//                lane per item while the item has at most kBinLaneTiles tiles
//                in the band and a wave per item beyond); the first share also
//                writes the tiles' ranges and lists the long ones.
// A view's pairs start where its first visible item's do, so a workgroup
// needs only its own view's totals.
//
// What bounds the placing is its scattered 8-byte stores: a tile's list is
// filled by all shares at once, so every cache line of the output stays
// partly written until the end.  Hence the bands, taken one after the other
// (the workgroups of a band fill the chip): a band's output is small enough
// for the XCDs' L2s to hold its lines until they are full, and each XCD takes
// consecutive shares, whose parts of a list lie side by side.
// A view of 341 k visible items and 5.4 M pairs (capacity 7.0 M; 1920x1080, 8,160
// tiles): 84 us in one band, 43 us in three; at 1.0, 1.7, 2.6 and 4.0 M pairs a
// band 54, 49, 46 and 52 us, and smaller calls lose with more bands than one
// (each band walks all the share's boxes again).  Counting, scanning and placing
// take 57 us there in all, where emitting the pairs unsorted, a two-pass radix sort by
// tile and the search for the tiles' ranges took 96 us; with 8 views
// (2.9 M visible items, 15.3 M pairs, 14,720 tiles) 123 us against 285 us.
// ---------------------------------------------------------------------------
constexpr int kBinThreads = 1024;
constexpr uint32_t kBinLaneTiles = 48;
// The one launch: its bands, items of a view and pairs of capacity per band at
// most.  Forwards of three launches and of one: 1,000 items 37.8 / 30.4 us
// (128x128) and 169 / 131 us (1920x1080 in 32,400 tiles), 8,000 items 46.5 / 41.5
// us (640x480) and 169 / 164 us (1920x1080, capacity 520 k); of 16,000 items 55.5 /
// 57.8 us and 78 / 92 us, each band walking all of them.
constexpr uint32_t kBinSmallBands = 32;
constexpr uint64_t kBinSmallItems = 8192, kBinSmallPairs = 32768;
constexpr uint64_t kBinBandPairs = 2600000;  // pairs (of the capacity) a band of a view is meant to hold
constexpr uint32_t kBinGroup = 16;  // 256 contiguous bytes of box words

// Visible index of the q-th item of share g of G of the view whose visible
// indices start at s0.
__device__ __forceinline__ uint32_t bin_item(uint32_t s0, uint32_t q, uint32_t g, uint32_t G) {
    return s0 + (q / kBinGroup * G + g) * kBinGroup + q % kBinGroup;
}

// A visible item's box, clipped to the tile rows [r0, r1) of its view.
struct BinBox {
    uint32_t x0, y0, w, h;  // first column and (clipped) row, width and (clipped) height
    uint32_t z, item;
};
__device__ __forceinline__ BinBox bin_box(const uint4 &bw, uint32_t r0, uint32_t r1) {
    const uint32_t y = bw.x >> 16, y1 = min(y + (bw.y >> 16), r1);
    BinBox b;
    b.x0 = bw.x & 0xffffu;
    b.w = bw.y & 0xffffu;
    b.y0 = max(y, r0);
    b.h = y1 > b.y0 ? y1 - b.y0 : 0u;
    b.z = bw.z;
    b.item = bw.w;
    return b;
}

// Adds a box to the difference array of the band that starts at row r0 (rows of
// P words).
__device__ __forceinline__ void bin_add_corners(uint32_t *s_tile, uint32_t P, const BinBox &b, uint32_t r0) {
    if (!b.h) return;
    uint32_t *at = s_tile + (b.y0 - r0) * P + b.x0;
    atomicAdd(at, 1u);
    atomicAdd(at + b.w, 0xffffffffu);
    atomicAdd(at + b.h * P, 0xffffffffu);
    atomicAdd(at + b.h * P + b.w, 1u);
}

// Sums along the rows of a difference array of ny rows of nx tiles, a wave each.
__device__ __forceinline__ void bin_row_sums(uint32_t *s_tile, uint32_t nx, uint32_t ny) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, P = nx + 1;
    const auto add = [](uint32_t a, uint32_t b) { return a + b; };
    for (uint32_t y = wave; y < ny; y += kBinThreads / kWave) {
        uint32_t carry = 0;
        for (uint32_t x0 = 0; x0 < nx; x0 += kWave) {
            const uint32_t x = x0 + lane;
            const uint32_t inc = wave_inclusive_scan(x < nx ? s_tile[y * P + x] : 0u, add) + carry;
            if (x < nx) s_tile[y * P + x] = inc;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
    }
}

// Clears the slots' "moments written" flags, set by the backward compositing,
// and the schedule's counters, filled by the forward; the grid shares the work.
__device__ __forceinline__ void bin_clear(uint32_t m, uint32_t *__restrict__ pflag, uint32_t *__restrict__ tile_order) {
    const uint64_t words = ((uint64_t)m + 3) / 4, nb = gridDim.x, w1 = words * (blockIdx.x + 1) / nb;
    for (uint64_t i = words * blockIdx.x / nb + threadIdx.x; i < w1; i += kBinThreads) pflag[i] = 0u;
    if (blockIdx.x == 0 && threadIdx.x < kCostBuckets) tile_order[threadIdx.x] = 0u;
}

// (share, view, tile rows) of a workgroup: views and bands one after the
// other, and within one, consecutive shares on each XCD.
struct BinTurn {
    uint32_t g, v, r0, r1;
};
__device__ __forceinline__ BinTurn bin_turn(const ViewTable &vt, uint32_t G, uint32_t bands) {
    BinTurn b;
    const uint32_t turn = blockIdx.x / G;
    b.g = xcd_contiguous(blockIdx.x - turn * G, G);
    b.v = turn / bands;
    const uint32_t band = turn - b.v * bands, rows = (uint32_t)vt.v[b.v].tiles_y;
    const uint32_t per = (rows + bands - 1) / bands;
    b.r0 = min(band * per, rows);
    b.r1 = min(b.r0 + per, rows);
    return b;
}

__global__ __launch_bounds__(kBinThreads) void k_bin_count(ViewTable vt, uint32_t G, uint32_t bands,
                                                           const uint32_t *__restrict__ seg,
                                                           const uint4 *__restrict__ item_box,
                                                           uint32_t *__restrict__ counts,
                                                           const WsHeader *__restrict__ hdr) {
    extern __shared__ uint32_t s_tile[];  // rows + 1 of tiles_x + 1
    const BinTurn bt = bin_turn(vt, G, bands);
    if (bt.r0 >= bt.r1) return;  // uniform
    const uint32_t nx = (uint32_t)vt.v[bt.v].tiles_x, ny = bt.r1 - bt.r0, P = nx + 1, off = vt.v[bt.v].tile_off;
    const uint32_t tid = threadIdx.x;
    for (uint32_t t = tid; t < P * (ny + 1); t += kBinThreads) s_tile[t] = 0u;
    __syncthreads();
    if (!hdr->overflow) {
        const uint32_t s0 = seg[bt.v], s1 = seg[bt.v + 1];
        for (uint32_t q = tid;; q += kBinThreads) {
            const uint32_t k = bin_item(s0, q, bt.g, G);
            if (k >= s1) break;
            bin_add_corners(s_tile, P, bin_box(item_box[k], bt.r0, bt.r1), bt.r0);
        }
    }
    __syncthreads();
    bin_row_sums(s_tile, nx, ny);  // then down the columns (a thread each)
    __syncthreads();
    uint32_t *out = counts + (size_t)bt.g * vt.total_tiles + off + bt.r0 * nx;
    for (uint32_t x = tid; x < nx; x += kBinThreads) {
        uint32_t run = 0, y = 0;
        for (; y + 8 <= ny; y += 8) {  // eight loads in flight
            uint32_t c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = s_tile[(y + u) * P + x];
#pragma unroll
            for (int u = 0; u < 8; ++u) out[(y + u) * nx + x] = run += c[u];
        }
        for (; y < ny; ++y) out[y * nx + x] = run += s_tile[y * P + x];
    }
}

// 64 tiles per workgroup, each of its 16 waves holding up to 16 rows of them in
// registers: the matrix is read once, all loads in flight, and written once.
__global__ __launch_bounds__(kBinThreads) void k_bin_scan(uint32_t *__restrict__ counts, uint32_t G,
                                                          uint32_t total_tiles, uint32_t *__restrict__ totals) {
    constexpr int kWaves = kBinThreads / kWave, kRows = kBinMaxRows / kWaves;
    __shared__ uint32_t part[kWaves][kWave];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t t = blockIdx.x * kWave + lane, g0 = w * kRows;
    const bool ok = t < total_tiles;
    uint32_t c[kRows], sum = 0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) c[r] = ok && g0 + r < G ? counts[(size_t)(g0 + r) * total_tiles + t] : 0u;
#pragma unroll
    for (int r = 0; r < kRows; ++r) sum += c[r];
    part[w][lane] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (uint32_t q = 0; q < w; ++q) run += part[q][lane];
    if (!ok) return;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (g0 + r < G) counts[(size_t)(g0 + r) * total_tiles + t] = run;
        run += c[r];
    }
    if (w == kWaves - 1) totals[t] = run;
}

// A list longer than kGroupSortMax: registered for the multi-workgroup sort.
__device__ __forceinline__ void register_long(uint32_t tile, uint32_t len, uint32_t *__restrict__ long_tiles,
                                              WsHeader *__restrict__ hdr) {
    const uint32_t k = atomicAdd(&hdr->n_long, 1u);
    if (k < kMaxLongTiles) long_tiles[k] = tile;
    atomicAdd(&hdr->long_pairs, len);
    atomicMax(&hdr->max_long, len);
}

// Places the pairs of share g of G of the visible indices [s0, s1) in the tile
// rows [r0, r1): s_tile holds each tile's next free entry, a row of the band
// every `pitch` words.
__device__ __forceinline__ void bin_place_items(uint32_t *s_tile, uint32_t pitch, uint32_t r0, uint32_t r1,
                                                uint32_t s0, uint32_t s1, uint32_t g, uint32_t G,
                                                const uint4 *__restrict__ item_box,
                                                unsigned long long *__restrict__ entries) {
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const auto place = [&](uint32_t t, uint32_t z, uint32_t item) {
        entries[atomicAdd(&s_tile[t], 1u)] = ((unsigned long long)z << 32) | item;
    };
    for (uint32_t q = w * kWave; bin_item(s0, q, g, G) < s1; q += kBinThreads) {  // the wave's first item: uniform
        const uint32_t k = bin_item(s0, q + lane, g, G);
        BinBox b{};
        b.w = 1u;
        if (k < s1) b = bin_box(item_box[k], r0, r1);
        const uint32_t c = b.w * b.h, t_first = (b.y0 - r0) * pitch + b.x0;
        const bool big = c > kBinLaneTiles;
        uint32_t left = big ? 0u : c, col = 0, t = t_first;
        while (__ballot(left > 0u)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (left > 0u) {
                    place(t, b.z, b.item);
                    --left;
                    ++t;
                    if (++col == b.w) col = 0, t += pitch - b.w;
                }
            }
        }
        unsigned long long mb = __ballot(big);
        while (mb) {
            const int j = __builtin_ctzll(mb);
            mb &= mb - 1ull;
            const uint32_t tj = __builtin_amdgcn_readlane(t_first, j), wj = __builtin_amdgcn_readlane(b.w, j);
            const uint32_t zj = __builtin_amdgcn_readlane(b.z, j), ij = __builtin_amdgcn_readlane(b.item, j);
            const uint32_t nj = __builtin_amdgcn_readlane(c, j);
            for (uint32_t q = lane; q < nj; q += kWave) {
                const uint32_t y = q / wj;
                place(tj + y * pitch + (q - y * wj), zj, ij);
            }
        }
    }
}

__global__ __launch_bounds__(kBinThreads) void k_bin_place(ViewTable vt, uint32_t G, uint32_t bands,
                                                           const uint32_t *__restrict__ seg,
                                                           const uint4 *__restrict__ item_box,
                                                           const uint32_t *__restrict__ counts,
                                                           const uint32_t *__restrict__ totals,
                                                           uint2 *__restrict__ ranges, uint32_t *__restrict__ long_tiles,
                                                           uint32_t *__restrict__ tile_order,
                                                           unsigned long long *__restrict__ entries,
                                                           uint32_t *__restrict__ pflag, WsHeader *hdr) {
    extern __shared__ uint32_t s_tile[];
    __shared__ uint32_t s_wave[2][kBinThreads / kWave];
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool overflow = hdr->overflow != 0u;
    const uint32_t m = overflow ? 0u : hdr->n_pairs;
    bin_clear(m, pflag, tile_order);
    const BinTurn bt = bin_turn(vt, G, bands);
    if (bt.r0 >= bt.r1) return;  // uniform
    const uint32_t nx = (uint32_t)vt.v[bt.v].tiles_x, off = vt.v[bt.v].tile_off;
    const uint32_t before = bt.r0 * nx, T = (bt.r1 - bt.r0) * nx, band0 = off + before;
    const uint32_t s0 = seg[bt.v], s1 = overflow ? s0 : seg[bt.v + 1];
    const uint32_t first = overflow ? 0u : seg[GSR_MAX_VIEWS + 1 + bt.v];
    // the band's tile starts: the totals of the view's tiles before it summed,
    // its own staged in LDS, each thread's run of consecutive tiles scanned
    const auto add = [](uint32_t a, uint32_t b) { return a + b; };
    // (eight loads in flight: with many tiles and few items these loops count)
    uint32_t early = 0;
#pragma unroll 8
    for (uint32_t t = tid; t < before; t += kBinThreads) early += totals[off + t];
#pragma unroll 8
    for (uint32_t t = tid; t < T; t += kBinThreads) s_tile[t] = totals[band0 + t];
    early = wave_reduce(early, 0u, add);
    if (lane == 0) s_wave[0][w] = early;
    __syncthreads();
    // (runs of an odd length: the lanes' starts then lie in different banks; 100 k items
    // in 129,600 tiles: 158 us with even runs and a load at a time above, 79 us)
    const uint32_t per = (T + kBinThreads - 1) / kBinThreads | 1u, t0 = min(tid * per, T), t1 = min(t0 + per, T);
    uint32_t sum = 0;
    for (uint32_t t = t0; t < t1; ++t) sum += s_tile[t];
    const uint32_t inc = wave_inclusive_scan(sum, add);
    if (lane == 63) s_wave[1][w] = inc;
    __syncthreads();
    uint32_t run = first + inc - sum;
    for (uint32_t q = 0; q < kBinThreads / kWave; ++q) run += s_wave[0][q] + (q < w ? s_wave[1][q] : 0u);
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t n = s_tile[t];
        s_tile[t] = run;
        if (bt.g == 0) {
            ranges[band0 + t] = make_uint2(run, run + n);
            if (n > (uint32_t)kGroupSortMax) register_long(band0 + t, n, long_tiles, hdr);
        }
        run += n;
    }
    __syncthreads();
    const uint32_t *row = counts + (size_t)bt.g * vt.total_tiles + band0;
#pragma unroll 8
    for (uint32_t t = tid; t < T; t += kBinThreads) s_tile[t] += row[t];
    __syncthreads();
    bin_place_items(s_tile, nx, bt.r0, bt.r1, s0, s1, bt.g, G, item_box, entries);
}

// All three in one launch, for calls of few items: a workgroup takes a band of
// tile rows of a view and all of the view's items, so that its counters are the
// tiles' totals; the pairs of the rows above come from the items' boxes.
__global__ __launch_bounds__(kBinThreads) void k_bin_small(ViewTable vt, uint32_t bands,
                                                           const uint32_t *__restrict__ seg,
                                                           const uint4 *__restrict__ item_box,
                                                           uint2 *__restrict__ ranges, uint32_t *__restrict__ long_tiles,
                                                           uint32_t *__restrict__ tile_order,
                                                           unsigned long long *__restrict__ entries,
                                                           uint32_t *__restrict__ pflag, WsHeader *hdr) {
    extern __shared__ uint32_t s_tile[];  // rows + 1 of tiles_x + 1
    __shared__ uint32_t s_wave[2][kBinThreads / kWave];
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool overflow = hdr->overflow != 0u;
    bin_clear(overflow ? 0u : hdr->n_pairs, pflag, tile_order);
    const BinTurn bt = bin_turn(vt, 1, bands);
    if (bt.r0 >= bt.r1) return;  // uniform
    const uint32_t nx = (uint32_t)vt.v[bt.v].tiles_x, ny = bt.r1 - bt.r0, P = nx + 1, T = nx * ny;
    const uint32_t band0 = vt.v[bt.v].tile_off + bt.r0 * nx;
    const uint32_t s0 = seg[bt.v], s1 = overflow ? s0 : seg[bt.v + 1];
    for (uint32_t t = tid; t < P * (ny + 1); t += kBinThreads) s_tile[t] = 0u;
    __syncthreads();
    const auto add = [](uint32_t a, uint32_t b) { return a + b; };
    uint32_t early = 0;  // pairs in the rows above
    for (uint32_t k = s0 + tid; k < s1; k += kBinThreads) {
        const uint4 bw = item_box[k];
        const uint32_t y = bw.x >> 16, above = min(y + (bw.y >> 16), bt.r0);
        if (above > y) early += (above - y) * (bw.y & 0xffffu);
        bin_add_corners(s_tile, P, bin_box(bw, bt.r0, bt.r1), bt.r0);
    }
    early = wave_reduce(early, 0u, add);
    if (lane == 0) s_wave[0][w] = early;
    __syncthreads();
    bin_row_sums(s_tile, nx, ny);
    __syncthreads();
    for (uint32_t x = tid; x < nx; x += kBinThreads) {
        uint32_t run = 0;
        for (uint32_t y = 0; y < ny; ++y) s_tile[y * P + x] = run += s_tile[y * P + x];
    }
    __syncthreads();
    // counts to starts, each thread a run of consecutive tiles
    const uint32_t per = (T + kBinThreads - 1) / kBinThreads | 1u, t0 = min(tid * per, T), t1 = min(t0 + per, T);
    uint32_t sum = 0;
    for (uint32_t t = t0, at = t0 / nx * P + t0 % nx, x = t0 % nx; t < t1; ++t) {
        sum += s_tile[at++];
        if (++x == nx) x = 0, ++at;
    }
    const uint32_t inc = wave_inclusive_scan(sum, add);
    if (lane == 63) s_wave[1][w] = inc;
    __syncthreads();
    uint32_t run = (overflow ? 0u : seg[GSR_MAX_VIEWS + 1 + bt.v]) + inc - sum;
    for (uint32_t q = 0; q < kBinThreads / kWave; ++q) run += s_wave[0][q] + (q < w ? s_wave[1][q] : 0u);
    for (uint32_t t = t0, at = t0 / nx * P + t0 % nx, x = t0 % nx; t < t1; ++t) {
        const uint32_t n = s_tile[at];
        s_tile[at++] = run;
        ranges[band0 + t] = make_uint2(run, run + n);
        if (n > (uint32_t)kGroupSortMax) register_long(band0 + t, n, long_tiles, hdr);
        run += n;
        if (++x == nx) x = 0, ++at;
    }
    __syncthreads();
    bin_place_items(s_tile, P, bt.r0, bt.r1, s0, s1, 0, 1, item_box, entries);
}

hipError_t bin_allow_lds(size_t bytes) {
    if (bytes <= 65536) return hipSuccess;  // up to 64 KB of LDS need no leave
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bin_count),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBinMaxLds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bin_place), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kBinMaxLds);
}

BinPlan bin_plan(const ViewTable &vt, uint64_t n, uint64_t cap) {
    const uint64_t V = (uint64_t)vt.n_views;
    const auto lds = [&](uint32_t bands) {
        size_t most = 0;
        for (int v = 0; v < vt.n_views; ++v) {
            const size_t rows = ((size_t)vt.v[v].tiles_y + bands - 1) / bands;
            most = std::max(most, 4 * (rows + 1) * ((size_t)vt.v[v].tiles_x + 1));
        }
        return most;
    };
    BinPlan p{};
    // one launch: few items and no more pairs than its bands, a row of tiles each
    // at least, place in a few us
    uint32_t rows = 1;
    for (int v = 0; v < vt.n_views; ++v) rows = std::max(rows, (uint32_t)vt.v[v].tiles_y);
    const uint32_t bands = std::min(rows, kBinSmallBands);
    if (n <= kBinSmallItems && cap <= V * bands * kBinSmallPairs && lds(bands) <= 65536) {
        p.small_bands = bands;
        p.lds_place = lds(bands);
        return p;
    }
    // (a row of the widest view, 4,096 tiles, and the one after it always fit)
    p.count_bands = 1;
    while (lds(p.count_bands) > kBinMaxLds) ++p.count_bands;
    const uint64_t want = std::min<uint64_t>((cap + V * kBinBandPairs - 1) / (V * kBinBandPairs), 64);
    p.place_bands = std::max(p.count_bands, (uint32_t)std::max<uint64_t>(want, 1));
    p.lds_count = lds(p.count_bands);
    p.lds_place = lds(p.place_bands);
    return p;
}

void launch_bin_pairs(const ViewTable &vt, const BinPlan &plan, uint32_t G, const uint32_t *seg,
                      const uint4 *item_box, uint32_t *counts, uint32_t *totals, uint2 *ranges, uint32_t *long_tiles,
                      uint32_t *tile_order, unsigned long long *entries, uint32_t *pflag, WsHeader *hdr,
                      hipStream_t st) {
    const uint32_t V = (uint32_t)vt.n_views;
    if (plan.small_bands) {
        hipLaunchKernelGGL(k_bin_small, dim3(V * plan.small_bands), dim3(kBinThreads), plan.lds_place, st, vt,
                           plan.small_bands, seg, item_box, ranges, long_tiles, tile_order, entries, pflag, hdr);
        return;
    }
    hipLaunchKernelGGL(k_bin_count, dim3(G * V * plan.count_bands), dim3(kBinThreads), plan.lds_count, st, vt, G,
                       plan.count_bands, seg, item_box, counts, hdr);
    hipLaunchKernelGGL(k_bin_scan, dim3((vt.total_tiles + kWave - 1) / kWave), dim3(kBinThreads), 0, st, counts, G, vt.total_tiles,
                       totals);
    hipLaunchKernelGGL(k_bin_place, dim3(G * V * plan.place_bands), dim3(kBinThreads), plan.lds_place, st, vt, G,
                       plan.place_bands, seg, item_box, counts, totals, ranges, long_tiles, tile_order,
                       entries, pflag, hdr);
}

// ---------------------------------------------------------------------------
// A4c: per-tile depth order.  The binning leaves each tile's items in no
// particular order; they are sorted here by the 64-bit key
// (depth key << 32 | item), the unique order of the compositing definition.
// The binning leaves those keys as the lists' entries, so a list is one
// contiguous read; its sorted item ids go to pval.
//
// The network is bitonic with every comparator oriented low-to-high: each
// merge starts with a "flip" that pairs mirrored positions, then half-cleaners
// at halving distances.  Lists are padded to a power of two with keys above
// every real key, which the network leaves at the end.
//
// A workgroup of four waves takes one tile.  A list of up to kBlockBucketMax
// entries is sorted by a bucket pass (below) when the depths allow, else by the
// network in registers.  There each lane holds E (1..16) consecutive entries,
// so comparators closer than E are register operations and the others pair
// lane l with lane l ^ m, fetched with DPP or ds_swizzle (within 32 lanes) or
// ds_bpermute, or, across waves, exchanged through LDS; a flip also mirrors
// the register index.  Lists up to 4096 entries take the network with 16
// entries per lane; longer lists run the multi-workgroup path (below) or, when
// it is off, the same network over global memory, one comparator per thread
// and step.
// ---------------------------------------------------------------------------
typedef unsigned long long u64;
constexpr u64 kPadKey = ~0ull;
// Bucket path: four waves, up to 8 entries per lane.  (With up to 4, half
// of the lists of the dense views, about 1,000 entries on average, fell to the
// 4096-entry network: sorting 8 views of 1 M items took 307 us, 4 views of 700 k
// 130 us; with 8, and the entries in one array, 81 us and 53 us.)
constexpr int kBlockBucketMax = 2048;

// v from lane (lane ^ M)
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
    if constexpr (M == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
    else if constexpr (M == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);  // quad_perm 2,3,0,1
    else if constexpr (M == 3) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x1B, 0xF, 0xF, false);  // quad_perm 3,2,1,0
    else if constexpr (M == 7) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false); // row_half_mirror
    else if constexpr (M == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false); // row_ror 8
    else if constexpr (M == 15) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false); // row_mirror
    else if constexpr (M < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (M << 10));  // xor in 32 lanes
    else return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ M) << 2, (int)v);
}

template <int M>
__device__ __forceinline__ u64 lane_xor64(u64 v, int lane) {
    const uint32_t lo = lane_xor<M>((uint32_t)v, lane), hi = lane_xor<M>((uint32_t)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ void order_regs(u64 &a, u64 &b) {
    const u64 x = a, y = b;
    a = x < y ? x : y;
    b = x < y ? y : x;
}

// keep the smaller of (mine, other) when `low`, else the larger
__device__ __forceinline__ u64 keep(u64 mine, u64 other, bool low) { return (other < mine) == low ? other : mine; }

// One comparator step of the network over P = 64 * E * W keys: merge size K,
// distance J (J == K / 2 is the flip).  key[r] of lane `lane` in wave `wave`
// is entry wave * 64E + lane * E + r.  W > 1 exchanges across waves through
// `xs` (64 * E * W words) and requires every thread of the W waves.
template <int E, int W, int K, int J>
__device__ __forceinline__ void bitonic_step(u64 (&key)[E], int lane, int wave, uint32_t *xs) {
    constexpr bool kFlip = J == K / 2;
    if constexpr (J < E) {  // both entries in this lane's registers
#pragma unroll
        for (int r = 0; r < E; ++r) {
            if constexpr (kFlip) {
                if ((r ^ (K - 1)) > r) order_regs(key[r], key[r ^ (K - 1)]);
            } else {
                if (!(r & J)) order_regs(key[r], key[r + J]);
            }
        }
    } else if constexpr (J < 64 * E) {  // another lane of this wave
        if constexpr (kFlip) {
            const bool low = !(lane & (K / (2 * E)));
            u64 o[E];
#pragma unroll
            for (int r = 0; r < E; ++r) o[r] = lane_xor64<K / E - 1>(key[E - 1 - r], lane);
#pragma unroll
            for (int r = 0; r < E; ++r) key[r] = keep(key[r], o[r], low);
        } else {
            const bool low = !(lane & (J / E));
#pragma unroll
            for (int r = 0; r < E; ++r) key[r] = keep(key[r], lane_xor64<J / E>(key[r], lane), low);
        }
    } else {  // another wave: through LDS, one 32-bit half at a time
        static_assert(W > 1, "cross-wave steps need several waves");
        constexpr int M = kFlip ? K / (64 * E) - 1 : J / (64 * E);
        const bool low = !(wave & (kFlip ? K / (128 * E) : M));
        const int pw = wave ^ M, pl = kFlip ? lane ^ 63 : lane;
        uint32_t half[2][E];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int r = 0; r < E; ++r) xs[(r * W + wave) * 64 + lane] = (uint32_t)(key[r] >> (32 * h));
            __syncthreads();
#pragma unroll
            for (int r = 0; r < E; ++r) half[h][r] = xs[((kFlip ? E - 1 - r : r) * W + pw) * 64 + pl];
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < E; ++r) key[r] = keep(key[r], ((u64)half[1][r] << 32) | half[0][r], low);
    }
}

template <int E, int W, int K, int J>
__device__ __forceinline__ void bitonic_merge(u64 (&key)[E], int lane, int wave, uint32_t *xs) {
    bitonic_step<E, W, K, J>(key, lane, wave, xs);
    if constexpr (J > 1) bitonic_merge<E, W, K, J / 2>(key, lane, wave, xs);
}

template <int E, int W, int K = 2>
__device__ __forceinline__ void register_bitonic(u64 (&key)[E], int lane, int wave, uint32_t *xs) {
    bitonic_merge<E, W, K, K / 2>(key, lane, wave, xs);
    if constexpr (K < 64 * E * W) register_bitonic<E, W, 2 * K>(key, lane, wave, xs);
}

// Sort list[0, len) of keys; the caller's threads are `W` whole waves and
// 64 * E * W >= len.  The items go to out, or, with out null, the keys back to
// list (every entry is in registers before the first is written).
template <int E, int W>
__device__ __forceinline__ void sort_list_regs(u64 *__restrict__ list, uint32_t len, uint32_t *__restrict__ out,
                                               int lane, int wave, uint32_t *xs) {
    u64 key[E];
    const uint32_t base = (uint32_t)(wave * 64 + lane) * E;
#pragma unroll
    for (int r = 0; r < E; ++r) key[r] = base + r < len ? list[base + r] : kPadKey;
    register_bitonic<E, W>(key, lane, wave, xs);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (base + r < len) {
            if (out) out[base + r] = (uint32_t)key[r];
            else list[base + r] = key[r];
        }
    }
}

// Fast path: a counting sort on a bucket index that is a monotone function of
// the depth key, b = floor((z - zmin) * NB / (zmax - zmin + 1)) in FP32
// (conversion, product and truncation are all non-decreasing, so bucket order
// never contradicts key order).  Entries are dropped into their bucket in
// arrival order; each then counts the bucket-mates with a smaller 64-bit key
// and stores itself at bucket start + that count.  For depths spread over the
// tile's range a bucket holds about one entry, so the ranking costs a read or
// two per entry, all independent.  Returns false, having written nothing, when
// some bucket holds more than kMaxBucket entries (clustered depths): the
// caller then sorts with the network, whose cost does not depend on the keys.
// Runs on the whole workgroup (256 threads, E entries each: NB = 256 E).
constexpr uint32_t kMaxBucket = 16;

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    return wave_reduce(v, 0xffffffffu, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    return wave_reduce(v, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
}

template <int E>
__device__ bool bucket_sort_block(const u64 *__restrict__ list, uint32_t len, uint32_t *__restrict__ out, u64 *buf,
                                  uint32_t *cnt, uint32_t *red /* [8] */) {
    constexpr uint32_t NB = 256 * E;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int r = 0; r < E; ++r) cnt[r * 256 + tid] = 0u;
    u64 key[E];
    uint32_t zmin = 0xffffffffu, zmax = 0u;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t i = (uint32_t)r * 256 + tid;
        key[r] = i < len ? list[i] : 0ull;
        const uint32_t z = (uint32_t)(key[r] >> 32);
        if (i < len) zmin = min(zmin, z), zmax = max(zmax, z);
    }
    zmin = wave_min_u32(zmin);
    zmax = wave_max_u32(zmax);
    if (lane == 0) red[wave] = zmin, red[4 + wave] = zmax;
    __syncthreads();
    zmin = min(min(red[0], red[1]), min(red[2], red[3]));
    zmax = max(max(red[4], red[5]), max(red[6], red[7]));
    const float scale = (float)NB / ((float)(zmax - zmin) + 1.0f);
    uint32_t bk[E], slot[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if ((uint32_t)r * 256 + tid < len) {
            const uint32_t z = (uint32_t)(key[r] >> 32);
            bk[r] = min(NB - 1, (uint32_t)((float)(z - zmin) * scale));
            slot[r] = atomicAdd(&cnt[bk[r]], 1u);
        }
    }
    __syncthreads();
    // thread owns buckets [tid * E, tid * E + E): their exclusive starts
    uint32_t c[E], run = 0, big = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        c[j] = cnt[tid * E + j];
        run += c[j];
        big = max(big, c[j]);
    }
    big = wave_max_u32(big);
    if (lane == 0) red[wave] = big;  // (red was last read before the barrier above)
    uint32_t total;
    uint32_t st = block_exclusive_scan(run, red + 4, total);  // ends with a barrier
    big = max(max(red[0], red[1]), max(red[2], red[3]));
    if (big > kMaxBucket) return false;  // uniform
#pragma unroll
    for (int j = 0; j < E; ++j) {
        cnt[tid * E + j] = (st << 16) | c[j];  // start < 2^16, count <= kMaxBucket
        st += c[j];
    }
    __syncthreads();
    uint32_t sc[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if ((uint32_t)r * 256 + tid < len) {
            sc[r] = cnt[bk[r]];
            buf[(sc[r] >> 16) + slot[r]] = key[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if ((uint32_t)r * 256 + tid < len) {
            const uint32_t s0 = sc[r] >> 16, n = sc[r] & 0xffffu;
            uint32_t rank = 0;
            for (uint32_t q = 0; q < n; ++q) rank += buf[s0 + q] < key[r] ? 1u : 0u;
            out[s0 + rank] = (uint32_t)key[r];
        }
    }
    return true;
}

template <int E>
__device__ __forceinline__ void sort_list_block(u64 *__restrict__ list, uint32_t len, uint32_t *__restrict__ out,
                                                u64 *buf, uint32_t *cnt, uint32_t *red, uint32_t *xs) {
    if (!bucket_sort_block<E>(list, len, out, buf, cnt, red)) {
        __syncthreads();  // the network reuses the exchange area
        sort_list_regs<E, 4>(list, len, out, threadIdx.x & 63, threadIdx.x >> 6, xs);
    }
}

// The same network over global memory, for lists beyond kGroupSortMax
// (comparators with an entry past the end are skipped: those entries act as
// +infinity).  Runs on the whole workgroup.
__device__ void sort_list_global(u64 *__restrict__ list, uint32_t len, uint32_t *__restrict__ out) {
    uint32_t p2 = 1;
    while (p2 < len) p2 <<= 1;
    for (uint32_t k = 2; k <= p2; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t c = threadIdx.x; c < p2 / 2; c += blockDim.x) {
                const uint32_t a = ((c & ~(j - 1)) << 1) | (c & (j - 1));
                const uint32_t b = j == (k >> 1) ? (a ^ (k - 1)) : (a + j);
                if (b < len) {
                    const u64 x = list[a], y = list[b];
                    if (x > y) list[a] = y, list[b] = x;
                }
            }
            __syncthreads();
        }
    }
    for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) out[i] = (uint32_t)list[i];
    __syncthreads();
}

// Lists longer than kGroupSortMax, when the multi-workgroup path takes them:
// every listed long tile of at most kLongWindow << passes entries (all of them
// once they fit the list).  k_long_windows numbers their windows (of
// kLongWindow entries for the run sort, of kMergeWindow outputs for the merge
// passes) in list order once per forward; a workgroup then finds its window
// among those offsets.
__device__ __forceinline__ bool long_path_on(const WsHeader *hdr, int passes) {
    return passes > 0 && passes <= kMaxLongPasses && hdr->n_long <= kMaxLongTiles;
}

__global__ __launch_bounds__(256) void k_long_windows(const uint2 *__restrict__ ranges,
                                                      uint32_t *__restrict__ long_tiles, int passes,
                                                      const WsHeader *__restrict__ hdr) {
    constexpr int kPer = kMaxLongTiles / 256;
    __shared__ uint32_t lds[4];
    if (hdr->overflow || !long_path_on(hdr, passes)) return;  // uniform
    const uint32_t n_long = hdr->n_long;
    const uint64_t cover = (uint64_t)kLongWindow << passes;
    uint32_t na[kPer], nm[kPer], sa = 0, sm = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t k = threadIdx.x * kPer + j;
        na[j] = nm[j] = 0;
        if (k < n_long) {
            const uint2 rg = ranges[long_tiles[k]];
            const uint32_t len = rg.y - rg.x;
            if ((uint64_t)len <= cover) {
                na[j] = (len + kLongWindow - 1) / kLongWindow;
                nm[j] = (len + kMergeWindow - 1) / kMergeWindow;
            }
        }
        sa += na[j];
        sm += nm[j];
    }
    uint32_t ta, tm;
    uint32_t ea = block_exclusive_scan(sa, lds, ta);
    uint32_t em = block_exclusive_scan(sm, lds, tm);
    uint32_t *wa = long_tiles + kMaxLongTiles, *wm = wa + kMaxLongTiles + 1;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t k = threadIdx.x * kPer + j;
        if (k < n_long) wa[k] = ea, wm[k] = em;
        ea += na[j];
        em += nm[j];
    }
    if (threadIdx.x == 0) wa[n_long] = ta, wm[n_long] = tm;
}

void launch_long_windows(const uint2 *ranges, uint32_t *long_tiles, int long_passes, const WsHeader *hdr,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_long_windows, dim3(1), dim3(256), 0, st, ranges, long_tiles, long_passes, hdr);
}

// Window e of all the long lists' windows (offsets `first`: one of the two
// tables above) as (tile, window within its list); false past the last.  Every
// lane of the wave calls it: the lists that start at or before e are counted, so
// that the offsets are one round of independent loads, not a chain.
__device__ __forceinline__ bool long_tile_window(const uint32_t *__restrict__ long_tiles,
                                                 const uint32_t *__restrict__ first, uint32_t n_long, uint32_t e,
                                                 uint32_t &tile, uint32_t &w) {
    if (n_long == 0) return false;
    const uint32_t lane = threadIdx.x & 63, total = first[n_long];
    uint32_t before = 0;
#pragma unroll 4
    for (uint32_t c = 0; c < n_long; c += kWave)
        before += (uint32_t)__popcll(__ballot(c + lane < n_long && first[min(c + lane, n_long)] <= e));
    if (e >= total) return false;
    // the last of them has the window (the next offset, or the total, is above e)
    tile = long_tiles[before - 1];
    w = e - first[before - 1];
    return true;
}

// The fused compositing's schedule, filed by one workgroup: every tile in the
// bucket of min(its list length, cost_hint[t]).  Each bucket has room for
// every tile, so filing needs only a slot counter per bucket, kept in LDS
// (`slots`): returning atomics on global counters serialise across the chip
// when most tiles share a few buckets, as they do, while LDS atomics resolve
// the lanes that collide within one instruction.  kSched tiles per thread are
// loaded together.
constexpr int kSched = 16;
__device__ void file_schedule(const uint2 *__restrict__ ranges, const uint32_t *__restrict__ cost_hint,
                              uint32_t total_tiles, uint32_t *__restrict__ order, uint32_t *slots) {
    const int tid = threadIdx.x, nt = blockDim.x;
    if (tid < (int)kCostBuckets) slots[tid] = 0u;
    __syncthreads();
    for (uint32_t base = 0; base < total_tiles; base += (uint32_t)(nt * kSched)) {
        uint32_t b[kSched];
#pragma unroll
        for (int q = 0; q < kSched; ++q) {
            const uint32_t t = base + (uint32_t)(q * nt + tid);
            b[q] = kCostBuckets;  // none
            if (t < total_tiles) {
                const uint2 rg = ranges[t];
                b[q] = cost_bucket(min(rg.y - rg.x, cost_hint[t]));
            }
        }
#pragma unroll
        for (int q = 0; q < kSched; ++q) {
            if (b[q] < kCostBuckets) {
                const uint32_t slot = atomicAdd(&slots[b[q]], 1u);
                order[kCostBuckets + (size_t)b[q] * total_tiles + slot] = base + (uint32_t)(q * nt + tid);
            }
        }
    }
    __syncthreads();
    if (tid < (int)kCostBuckets) order[tid] = slots[tid];
}

__global__ __launch_bounds__(256) void k_tile_depth_sort(const uint2 *__restrict__ ranges, uint32_t total_tiles,
                                                         u64 *__restrict__ entries, uint32_t *__restrict__ pval,
                                                         const uint32_t *__restrict__ long_tiles, int passes,
                                                         uint32_t *__restrict__ sched,
                                                         const uint32_t *__restrict__ cost_hint,
                                                         const WsHeader *__restrict__ hdr) {
    __shared__ u64 s_buf[kBlockBucketMax];  // bucket entries; the network's exchange area (16 KB)
    __shared__ uint32_t s_cnt[kBlockBucketMax];
    __shared__ uint32_t s_red[8];
    if (hdr->overflow) return;  // uniform (no schedule either: the fused compositing falls back to tile order)
    uint32_t *xs = reinterpret_cast<uint32_t *>(s_buf);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool multi = long_path_on(hdr, passes);
    // with a schedule to file, workgroup 0 files it (overlapping the sorts)
    // and the tiles start at workgroup 1
    if (sched && blockIdx.x == 0) {
        file_schedule(ranges, cost_hint, total_tiles, sched, s_cnt);
        return;
    }
    const uint32_t bid = blockIdx.x - (sched ? 1u : 0u);
    if (bid >= total_tiles) {
        // a window of a long list, sorted in place into a run of the first merge pass's input
        if (!multi) return;
        uint32_t t, w;
        if (!long_tile_window(long_tiles, long_tiles + kMaxLongTiles, hdr->n_long, bid - total_tiles, t, w))
            return;
        const uint2 rg = ranges[t];
        const uint32_t off = rg.x + w * kLongWindow;
        const uint32_t n = min(kLongWindow, rg.y - off);
        sort_list_regs<16, 4>(entries + off, n, nullptr, lane, wave, xs);
        return;
    }
    const uint32_t t = bid;
    const uint2 rg = ranges[t];
    const uint32_t len = rg.y - rg.x;
    u64 *list = entries + rg.x;
    uint32_t *out = pval + rg.x;
    if (len <= 1) {
        if (len == 1 && threadIdx.x == 0) out[0] = (uint32_t)list[0];
        return;
    }
    if (len <= 256)
        sort_list_block<1>(list, len, out, s_buf, s_cnt, s_red, xs);
    else if (len <= 512)
        sort_list_block<2>(list, len, out, s_buf, s_cnt, s_red, xs);
    else if (len <= 1024)
        sort_list_block<4>(list, len, out, s_buf, s_cnt, s_red, xs);
    else if (len <= (uint32_t)kBlockBucketMax)
        sort_list_block<8>(list, len, out, s_buf, s_cnt, s_red, xs);
    else if (len <= (uint32_t)kGroupSortMax)
        sort_list_regs<16, 4>(list, len, out, lane, wave, xs);
    else if (!multi || (uint64_t)len > ((uint64_t)kLongWindow << passes))
        sort_list_global(list, len, out);
    // else: the window workgroups and the merge passes sort it
}

void launch_tile_depth_sort(const uint2 *ranges, uint32_t total_tiles, unsigned long long *entries, uint32_t *pval,
                            const uint32_t *long_tiles, int long_passes, uint32_t chunk_wgs, uint32_t *sched,
                            const uint32_t *cost_hint, const WsHeader *hdr, hipStream_t st) {
    if (total_tiles == 0) return;
    const uint32_t grid = total_tiles + (long_passes > 0 ? chunk_wgs : 0u) + (sched ? 1u : 0u);
    hipLaunchKernelGGL(k_tile_depth_sort, dim3(grid), dim3(256), 0, st, ranges, total_tiles, entries, pval, long_tiles,
                       long_passes, sched, cost_hint, hdr);
}

// ---------------------------------------------------------------------------
// A4d: merge passes over the long lists' sorted runs.  Pass p merges runs of
// kLongWindow << p pairwise; a workgroup makes kMergeWindow consecutive
// outputs of one merge.  Its inputs start where the merge path crosses its
// first and last output (found by one wave each, 64 probes per round), are
// staged in LDS, and each thread merges 8 outputs from its own crossing.
// Keys are unique, so every split is unambiguous.  A pass moves little and is
// bound by the chain of dependent accesses before its stores: five passes over
// 84 lists (the longest 124 k) take 75 us, 89 us with a binary search for the
// workgroup's list and stores straight from the merging threads.
// ---------------------------------------------------------------------------
// Number of elements of A among the first d outputs of merge(A, B): the
// smallest a in [max(0, d - nB), min(d, nA)] with not (A[a] < B[d - 1 - a]).
// One whole wave calls it.
__device__ uint32_t wave_merge_split(const u64 *a, uint32_t nA, const u64 *b, uint32_t nB, uint32_t d, int lane) {
    uint32_t lo = d > nB ? d - nB : 0u, hi = min(d, nA);
    while (lo < hi) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint32_t m = lo + (uint32_t)lane * step;
        const bool probe = m < hi;
        const bool before = probe && a[m] < b[d - 1 - m];
        const uint32_t c = (uint32_t)__popcll(__ballot(before));  // probes before the split: a prefix of the lanes
        const uint32_t nlo = c > 0 ? lo + (c - 1) * step + 1 : lo;
        const uint32_t nhi = min(hi, lo + c * step);
        lo = nlo;
        hi = nhi;
    }
    return lo;
}

__global__ __launch_bounds__(256) void k_long_merge(const uint2 *__restrict__ ranges,
                                                    const uint32_t *__restrict__ long_tiles,
                                                    const WsHeader *__restrict__ hdr, int p, int passes,
                                                    const u64 *__restrict__ src, u64 *__restrict__ dst,
                                                    uint32_t *__restrict__ pval) {
    __shared__ u64 sA[kMergeWindow], sB[kMergeWindow];
    __shared__ uint32_t s_split[2];
    if (hdr->overflow || !long_path_on(hdr, passes)) return;  // uniform
    uint32_t t, w;
    if (!long_tile_window(long_tiles, long_tiles + 2 * kMaxLongTiles + 1, hdr->n_long, blockIdx.x, t, w)) return;
    const uint2 rg = ranges[t];
    const uint32_t L = rg.y - rg.x;
    const uint32_t o0 = w * kMergeWindow, o1 = min(o0 + kMergeWindow, L);
    const uint64_t R64 = (uint64_t)kLongWindow << p;  // p < kMaxLongPasses: R < 2^29
    const uint32_t R = (uint32_t)R64;
    const uint32_t base = (uint32_t)((o0 / (2 * R64)) * (2 * R64));
    const uint32_t nA = min(R, L - base), nB = L - base > R ? min(R, L - base - R) : 0u;
    const u64 *pa = src + rg.x + base, *pb = pa + R;
    const bool last = p == passes - 1;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t d0 = o0 - base, d1 = o1 - base;
    if (wave < 2) {
        const uint32_t a = wave_merge_split(pa, nA, pb, nB, wave == 0 ? d0 : d1, (int)lane);
        if (lane == 0) s_split[wave] = a;
    }
    __syncthreads();
    const uint32_t a0 = s_split[0], a1 = s_split[1], b0 = d0 - a0, b1 = d1 - a1;
    const uint32_t na = a1 - a0, nb = b1 - b0;
    for (uint32_t k = tid; k < na; k += 256) sA[k] = pa[a0 + k];
    for (uint32_t k = tid; k < nb; k += 256) sB[k] = pb[b0 + k];
    __syncthreads();
    constexpr uint32_t kPer = kMergeWindow / 256;
    const uint32_t q = tid * kPer;
    // this thread's crossing of the staged merge (threads past the end take the end)
    uint32_t lo = q > nb ? min(q - nb, na) : 0u, hi = min(q, na);
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (sA[mid] < sB[q - 1 - mid]) lo = mid + 1;
        else hi = mid;
    }
    uint32_t i = lo, j = q - lo;
    const uint32_t all = na + nb, nq = min(kPer, all - min(q, all));
    u64 v[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        if (k >= nq) continue;
        const bool take_b = i >= na || (j < nb && sB[j] < sA[i]);
        v[k] = take_b ? sB[j] : sA[i];
        i += take_b ? 0u : 1u;
        j += take_b ? 1u : 0u;
    }
    __syncthreads();
    // through LDS, so that the stores are contiguous across the lanes
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (k < nq) sA[q + k] = v[k];
    __syncthreads();
    const uint32_t out = rg.x + o0;
    for (uint32_t k = tid; k < all; k += 256) {
        if (last)
            pval[out + k] = (uint32_t)sA[k];
        else
            dst[out + k] = sA[k];
    }
}

void launch_long_merge(const uint2 *ranges, const uint32_t *long_tiles, const WsHeader *hdr, int p, int long_passes,
                       const unsigned long long *src, unsigned long long *dst, uint32_t *pval, uint32_t merge_wgs,
                       hipStream_t st) {
    if (merge_wgs == 0) return;
    hipLaunchKernelGGL(k_long_merge, dim3(merge_wgs), dim3(256), 0, st, ranges, long_tiles, hdr, p, long_passes,
                       src, dst, pval);
}

// Tile id at every position of the sorted pairs (the export of the lists).
__global__ __launch_bounds__(256) void k_expand_ranges(const uint2 *__restrict__ ranges, uint32_t total_tiles,
                                                       uint32_t *__restrict__ pair_tiles,
                                                       const WsHeader *__restrict__ hdr) {
    const uint32_t t = blockIdx.x;
    if (t >= total_tiles || hdr->overflow) return;
    const uint2 rg = ranges[t];
    for (uint32_t i = rg.x + threadIdx.x; i < rg.y; i += 256) pair_tiles[i] = t;
}

void launch_expand_ranges(const uint2 *ranges, uint32_t total_tiles, uint32_t *pair_tiles, const WsHeader *hdr,
                          hipStream_t st) {
    if (total_tiles == 0) return;
    hipLaunchKernelGGL(k_expand_ranges, dim3(total_tiles), dim3(256), 0, st, ranges, total_tiles, pair_tiles, hdr);
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *__restrict__ p, uint32_t value, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) p[i] = value;
}

void launch_fill_u32(uint32_t *p, uint32_t value, uint64_t n, hipStream_t st) {
    if (n == 0) return;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, value, n);
}

__global__ void k_reset_header(WsHeader *h, uint32_t cap) {
    const uint32_t t = threadIdx.x;
    uint32_t *w = reinterpret_cast<uint32_t *>(h);
    if (t < sizeof(WsHeader) / 4) w[t] = 0u;
    __syncthreads();
    if (t == 0) h->pair_capacity = cap;
}

void launch_reset_header(WsHeader *h, uint32_t cap, hipStream_t st) {
    hipLaunchKernelGGL(k_reset_header, dim3(1), dim3(64), 0, st, h, cap);
}

// Start of a backward pass: its work queue.
__global__ void k_reset_queue(WsHeader *h, int which) { h->queue[which] = 0u; }

void launch_reset_queue(WsHeader *h, int which, hipStream_t st) {
    hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(1), 0, st, h, which);
}

}  // namespace gsr
