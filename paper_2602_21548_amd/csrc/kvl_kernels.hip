// Launchers of the copy kernels and the entry points built on them (pack, unpack, move,
// storage layout, plain copy).  The kernels themselves are in kvl_copy_kernels.h.
#include <algorithm>
#include <cstdio>

#include <hip/hip_ext.h>

#include "kvl_copy_kernels.h"

namespace kvl {

// Every plane of a pool must be device-addressable memory of the pool's full size.
int check_pool(const kvl_plan_t *plan, const void *const *planes, uint64_t pool_blocks) {
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p) {
        if (!planes[p]) return KVL_EINVAL;
        const uint64_t bytes = pool_blocks * plan->layout.block_tokens * (uint64_t)plan->layout.row_bytes[p];
        int rc = check_buffer(plan, planes[p], bytes, false);
        if (rc != KVL_OK) return rc;
    }
    return KVL_OK;
}

// The descriptors live on the device that was current when the plan was made.
int check_device(const kvl_plan_t *plan) {
    int dev = -1;
    KVL_HIP(hipGetDevice(&dev));
    return dev == plan->device ? KVL_OK : KVL_EINVAL;
}

// Where a kernel goes, and the event that is to fire when it has finished (or null).  The event rides on the
// dispatch itself: recorded on its own behind it, it costs another packet for the host to write and the queue to
// wait for (launches of a 3 us kernel in a row: 7.5 us each recorded, 4.5 us riding, 2.8 us without; host 8 / 2.5).
struct On {
    hipStream_t stream;
    DefaultStreamEvent *passes = nullptr;       // (made by the making of `done`)
    hipEvent_t done;
    bool ok = false;
    On(const kvl_plan_t *plan, hipStream_t s) : stream(s), done(launch_event(plan, s, &passes)) {}
    ~On() {
        if (passes) launched(passes, ok);
    }
    On(const On &) = delete;
    On &operator=(const On &) = delete;
    // the launches' result, once all have been made
    int made() {
        KVL_HIP(hipGetLastError());
        ok = true;
        return KVL_OK;
    }
};
#define KVL_LAUNCH(kernel, grid, block, on, ...)                                                                  \
    do {                                                                                                          \
        if ((on).done) hipExtLaunchKernelGGL(kernel, grid, block, 0, (on).stream, nullptr, (on).done, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(kernel, grid, block, 0, (on).stream, __VA_ARGS__);                                \
    } while (0)

template <bool PACK, bool WAVE, int U, bool NTL, int SP>
static void launch_one(dim3 grid, dim3 block, const On &s, const CopyArgs &a) {
    if (PACK) KVL_LAUNCH((kvl_pack_kernel<WAVE, U, NTL, SP>), grid, block, s, a);
    else KVL_LAUNCH((kvl_unpack_kernel<WAVE, U, NTL, SP>), grid, block, s, a);
}

template <bool PACK, bool WAVE, int U, bool NTL>
static void launch_sp(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a) {
    switch ((v >> 3) & 3u) {
        case 0: launch_one<PACK, WAVE, U, NTL, 0>(g, b, s, a); break;
        case 1: launch_one<PACK, WAVE, U, NTL, 1>(g, b, s, a); break;
        case 2: launch_one<PACK, WAVE, U, NTL, 2>(g, b, s, a); break;
        default: launch_one<PACK, WAVE, U, NTL, 3>(g, b, s, a); break;
    }
}

template <bool PACK, bool WAVE, int U>
static void launch_nt(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a) {
    if (v & 4u) launch_sp<PACK, WAVE, U, true>(v, g, b, s, a);
    else launch_sp<PACK, WAVE, U, false>(v, g, b, s, a);
}

template <bool PACK>
static void launch_span_variant(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a) {
    const bool wave = (v & 3u) == 1u, deep = (v & 32u) != 0;
    if (wave) {
        if (deep) launch_nt<PACK, true, 8>(v, g, b, s, a);
        else launch_nt<PACK, true, 4>(v, g, b, s, a);
    } else {
        if (deep) launch_nt<PACK, false, 8>(v, g, b, s, a);
        else launch_nt<PACK, false, 4>(v, g, b, s, a);
    }
}

// The descriptor of workgroup b is (b * magic >> 32) >> shift, exactly, for every b below 2^31: with l = ceil(log2 d) the
// number m = ceil(2^(31+l) / d) fits 32 bits and exceeds 2^(31+l) / d by less than 2^l / d, which b / 2^(31+l) makes less than
// 1 / d.  (d == 1: magic 0, the workgroup's own number.)
struct TileDivisor {
    uint32_t magic = 0, shift = 0;
    explicit TileDivisor(uint32_t d) {
        if (d < 2) return;
        uint32_t l = 1;
        while ((1ull << l) < d) ++l;
        magic = (uint32_t)(((1ull << (31 + l)) + d - 1) / d);
        shift = l - 1;
    }
};

// How a launch's workgroups take its tiles (see tile_number).
static uint32_t tile_order(uint64_t tiles, uint64_t tile_bytes, uint64_t run_bytes) {
    if (run_bytes == 0) return 0;
    uint32_t shift = 1;
    while (shift < 12 && (tile_bytes << shift) < run_bytes) ++shift;
    return (uint32_t)(std::min<uint64_t>(tiles, INT32_MAX) >> (shift + 3) << (shift + 3)) | shift;
}

static TileMore more_planes(const CopyArgs &a, uint32_t planes) {
    TileMore more{};
    for (uint32_t q = 1; q < planes; ++q) {
        more.pool[q - 1] = a.pool[a.plane_begin + q];
        more.xfer[q - 1] = a.xfer[a.plane_begin + q];
    }
    return more;
}

// n_tiles != 0: the launch has fewer workgroups than tiles and they walk over them
template <bool PACK, int VPT, bool NTL, int SP>
static void launch_tile_one(dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t tpu, uint32_t al,
                            uint32_t n_tiles, uint64_t run_bytes) {
    if (n_tiles) {
        KVL_LAUNCH((kvl_tile_walk_kernel<PACK, VPT, NTL, SP>), g, b, s, a, tpu, al, n_tiles);
        return;
    }
    const TileDivisor d(tpu);
    const uint32_t p = a.plane_begin, how = d.shift << 1 | al;
    const uint32_t order = tile_order(g.x, 16ull * VPT * b.x, run_bytes);
    const TileMore more = more_planes(a, g.y);
    const kvl_unit_t *units = a.units + a.unit_begin;
    if (PACK) KVL_LAUNCH((kvl_pack_quick_tile_kernel<VPT, NTL, SP>), g, b, s, units, a.pool[p], a.xfer[p], a.row_elems[p], tpu, d.magic, how, b.x, order, more);
    else KVL_LAUNCH((kvl_unpack_quick_tile_kernel<VPT, NTL, SP>), g, b, s, units, a.pool[p], a.xfer[p], a.row_elems[p], tpu, d.magic, how, b.x, order, more);
}

template <bool PACK, int VPT, bool NTL>
static void launch_tile_sp(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t tpu,
                           uint32_t al, uint32_t n_tiles, uint64_t run_bytes) {
    switch ((v >> 3) & 3u) {
        case 0: launch_tile_one<PACK, VPT, NTL, 0>(g, b, s, a, tpu, al, n_tiles, run_bytes); break;
        case 1: launch_tile_one<PACK, VPT, NTL, 1>(g, b, s, a, tpu, al, n_tiles, run_bytes); break;
        case 2: launch_tile_one<PACK, VPT, NTL, 2>(g, b, s, a, tpu, al, n_tiles, run_bytes); break;
        default: launch_tile_one<PACK, VPT, NTL, 3>(g, b, s, a, tpu, al, n_tiles, run_bytes); break;
    }
}

template <bool PACK, int VPT>
static void launch_tile_variant(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t tpu,
                                uint32_t al, uint32_t n_tiles, uint64_t run_bytes) {
    if (v & 4u) launch_tile_sp<PACK, VPT, true>(v, g, b, s, a, tpu, al, n_tiles, run_bytes);
    else launch_tile_sp<PACK, VPT, false>(v, g, b, s, a, tpu, al, n_tiles, run_bytes);
}

template <bool PACK, bool NTL>
static void launch_pipe_sp(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t tpu, uint32_t al,
                           uint32_t n_tiles) {
    switch ((v >> 3) & 3u) {
        case 0: KVL_LAUNCH((kvl_tile_pipe_kernel<PACK, NTL, 0>), g, b, s, a, tpu, al, n_tiles); break;
        case 1: KVL_LAUNCH((kvl_tile_pipe_kernel<PACK, NTL, 1>), g, b, s, a, tpu, al, n_tiles); break;
        case 2: KVL_LAUNCH((kvl_tile_pipe_kernel<PACK, NTL, 2>), g, b, s, a, tpu, al, n_tiles); break;
        default: KVL_LAUNCH((kvl_tile_pipe_kernel<PACK, NTL, 3>), g, b, s, a, tpu, al, n_tiles); break;
    }
}

template <bool PACK>
static void launch_pipe_variant(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t tpu,
                                uint32_t al, uint32_t n_tiles) {
    if (v & 4u) launch_pipe_sp<PACK, true>(v, g, b, s, a, tpu, al, n_tiles);
    else launch_pipe_sp<PACK, false>(v, g, b, s, a, tpu, al, n_tiles);
}

// Compute units of a device (asked once per device).
static int compute_units(int device) {
    static int cached[64] = {};
    if (device < 0 || device >= 64) return 256;
    if (cached[device] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 256;
        }
        cached[device] = n;
    }
    return cached[device];
}

template <bool PACK, bool NTL, int SP>
static void launch_flat_one(dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t m) {
    const uint32_t p = a.plane_begin;
    const TileDivisor d(m);
    const kvl_unit_t *units = a.units + a.unit_begin;
    const TileMore more = more_planes(a, g.y);
#define KVL_FLAT(KERNEL) KVL_LAUNCH((KERNEL<PACK, NTL, SP>), g, b, s, units, a.pool[p], a.xfer[p], a.row_elems[p], a.n_units, m, d.magic, d.shift, b.x, more)
    if (m < kFlatShort) KVL_FLAT(kvl_flat_kernel_short);
    else KVL_FLAT(kvl_flat_kernel);
#undef KVL_FLAT
}

template <bool PACK, bool NTL>
static void launch_flat_sp(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t m) {
    switch ((v >> 3) & 3u) {
        case 0: launch_flat_one<PACK, NTL, 0>(g, b, s, a, m); break;
        case 1: launch_flat_one<PACK, NTL, 1>(g, b, s, a, m); break;
        case 2: launch_flat_one<PACK, NTL, 2>(g, b, s, a, m); break;
        default: launch_flat_one<PACK, NTL, 3>(g, b, s, a, m); break;
    }
}

template <bool PACK>
static void launch_flat_variant(uint32_t v, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t m) {
    if (v & 4u) launch_flat_sp<PACK, true>(v, g, b, s, a, m);
    else launch_flat_sp<PACK, false>(v, g, b, s, a, m);
}

template <bool PACK, bool NTL, int SP>
static void launch_rows(dim3 g, dim3 b, const On &s, const CopyArgs &a, const uint32_t *map, uint32_t row_begin,
                        uint32_t n_vecs, uint64_t run_bytes) {
    const uint32_t p = a.plane_begin, row = a.row_elems[p];
    const TileMore more = more_planes(a, g.y);
    const uint32_t order = tile_order(g.x, 16ull * b.x, run_bytes);
#define KVL_ROWS(K) KVL_LAUNCH((kvl_rows_kernel<PACK, NTL, SP, K>), g, b, s, map, a.pool[p], row_begin, n_vecs, a.xfer[p], row, b.x, order, more)
    if (row >= 64) KVL_ROWS(2);
    else if (row >= 32) KVL_ROWS(3);
    else if (row >= 16) KVL_ROWS(5);
    else KVL_ROWS(0);
#undef KVL_ROWS
}

template <bool PACK, bool NTL, int SP, bool SRC>
static void launch_any_one(bool flat, bool walk, dim3 g, dim3 b, const On &s, const CopyArgs &a, uint32_t x, uint32_t n_tiles,
                           uint64_t run_bytes) {
    const uint32_t order = tile_order(g.x, 16ull * b.x, run_bytes);
    const TileDivisor d(x);
    const uint32_t p = a.plane_begin;
    const kvl_unit_t *units = a.units + a.unit_begin;
    const TileMore more = more_planes(a, g.y);
#define KVL_ANY_FLAT(KERNEL) KVL_LAUNCH((KERNEL<PACK, NTL, SP>), g, b, s, units, a.pool[p], a.xfer[p], a.row_elems[p], a.n_units, x, d.magic, d.shift, b.x, order, more)
    if (flat && x < kFlatShort) KVL_ANY_FLAT(kvl_any_flat_kernel_short);
    else if (flat) KVL_ANY_FLAT(kvl_any_flat_kernel);
    else if (walk) KVL_LAUNCH((kvl_any_walk_kernel<PACK, NTL, SP, SRC>), g, b, s, a, x, n_tiles, n_tiles > g.x ? 0u : order);
    else KVL_LAUNCH((kvl_any_tile_kernel<PACK, NTL, SP, SRC>), g, b, s, units, a.pool[p], a.xfer[p], a.row_elems[p], x, d.magic, d.shift << 1, b.x, order, more);
#undef KVL_ANY_FLAT
}

// Rows or addresses that are not multiples of 16 bytes (the planes of a launch have one row size).
//   cache policy and lines of the tiles, by the payload.  Up to kCachedLayerBytes the on-die cache holds a layer from the
//     gather to the scatter: the gather writes with sc1 stores and the scatter reads with plain loads.  Up to kReadOnceBytes
//     both lay their tiles on the source's lines, so that the scatter's non-temporal loads take each line out of the cache
//     once (see kvl_any_tile_kernel), and the scatter stores with nt.  Larger layers pass the cache by, both ways, and the
//     scatter's tiles lie on the destination's lines.  The gather's lie on its source's, but across the host link.  Hops, three layers in
//     turn, us, passing by / read once / kept (gather on the destination's lines): 1026-byte rows by 64, 77 MB 56 / 50 / 50,
//     100 MB 72 / 64 / 74, 242 MB 167 / 148 / 170, 494 MB 342 / 332 / 355, 666 MB 461 / 456 / 477, 924 MB 636 / 642 / -;
//     333 by 64, 85 MB 69 / 61 / 60, 206 MB 161 / 143 / 156, 655 MB 519 / 490 / 540.  With one layer again and again the
//     kept form would be 2-5 % ahead up to 240 MB, with four it is 15 % behind from 77 MB.  Kept, the gather on its
//     source's lines: 333 by 64, 39 MB, 29.2 -> 27.5; 99 by 64, 22 MB, 21.3 -> 19.3.
//     Across the host link as kept (741-byte rows, 80 MB in and out, 2857 us against 2987 passing by).
//     Several planes of blocks of whole lines, none of which is nearly all of the layer: read once up to kReadOnceManyBytes, by
//     the scatter up to kScatterOnceManyBytes where the descriptors are single blocks or two (hops, random tables, before the
//     source's lines / on them / so: 132 and 132 by 64, 493 MB 356 / 367 / 346, 663 MB 484 / 506 / 473; 132 and 260 by 64, 592
//     MB 430 / 449 / 432; 72 and 72 by 128, 607 MB 436 / 466 / 433); past the cache their gather starts late from
//     kLateTileBytes on (516 and 516 by 64, 867 MB 623 / 647 / 626; in one plane the early start is 1 % ahead).
//   flat or tiled: a descriptor of up to kAnyFlatWindows vectors leaves too much of its last tile idle (150 MB hops, flat /
//     tiled: 300-byte rows by 8, 151 windows, 111 / 114; 90 by 32, 181 windows, 119 / 107; 153 by 24, 231 windows, 117 / 104).
//     Blocks of whole lines go better flat, once they are not kept (200 by 16, 201 windows, 31 MB 27 / 25, 147 MB 108 / 113; 70 by 64,
//     281 windows, 142 MB, 111 / 104).
//     Where the largest is more than half again the average, most tiles' workgroups would find nothing to do, and narrow ones
//     are many: flat up to kAnyFlatPastWindows (104 by 16, a chance pair merged here and there, 209 windows, 348 MB, gather
//     157 flat, 210 tiled).  A flat workgroup has 1024 lanes (1026-byte rows by 1: 361 us at 256, 329 at 512, 324).
//   lanes of a tile: a gather's 64, which idle least (132 by 64, 275 MB, 103 us with 256, 99 with 128, 94 with 64; 333 by 64,
//     196 MB, 69 / 64 / 63; 1026 by 64, 181 MB, 57 / 58 / 58); a scatter's 256, whose wavefronts share fewer lines at the
//     ends of tiles, or 128 where that leaves an eighth of the lanes fewer without work (256 / 128: 132 by 64 107 / 103, 333
//     by 16 54 / 49, 47 by 128 46 / 42; but 333 by 64, 8 % fewer, 73 / 77, 1115 by 16 45 / 48), up to kHalveBytes (scatter of 132
//     by 64, 306 MB 115 / 112, 541 MB 211 / 226; 72 by 128, 323 MB 123.5 / 123.1, 476 MB 184 / 203).  Past the cache 256 or, for
//     short descriptors, by the same rule (gather of 153 by 24, 948 MB, 256 / 128: 348 / 385).  Under a cap on the workgroups
//     they are widened until kCappedLanes are at work, which is what keeps the memory busy (gather with 64 / 256: 132 by 64,
//     254 MB, 512 workgroups 384 / 157, 4096 85 / 110; 333 by 64, 50 MB, 1024 42.4 / 20.4, 4096 19.6 / 20.8), and where 256
//     lanes are not enough descriptors go flat, in workgroups of 1024, up to kAnyFlatPastWindows (hops, flat / tiled with 256:
//     1026 by 4, 24 MB, 64 workgroups 140 / 251, 512 32.9 / 40.8, 1024 28.4 / 28.2).
//   order (tile_number): in runs, so that wavefronts that share a line have one L2.  Moves in runs of 256 KiB, flat hops too, from
//     kFlatOrderBytes, tiled ones above kOddOrderBytes of 512 KiB, or 128 where the layer is a little more than the on-die cache holds.
//     Hops, three layers in turn, us, in order / runs of 64, 128, 256, 512 KiB: 132 by 64, 70 MB 45.7 / 44.0 / 44.0 / 43.7 / 43.3, 199 MB
//     136 / 123 / 121 / 121 / 119, 340 MB 236 / 236 / 238 / 238 / 238, 1.4 GB 1048 / 1010 / 1001 / 993 / 988; 333 by 64, 340 MB 232 / 220 /
//     222 / 225 / 226, 793 MB 626 / 573 / 565 / 566 / 566; 1026 by 64, 279 MB 171 / 168 / 168 / 171 / 175; flat, 200 by 16, 401 MB 295 / 291 / 289 /
//     288 / 289, 21 by 64, 75 MB 74.0 / 74.1 / 74.4 / 74.1 / 75.4.  Short blocks of whole lines in one plane just beyond the cache,
//     where a plan serves every layer of a batch / each layer has one of its own, whose descriptors come from the memory then (in order, runs of
//     32, of 128 KiB): 132 by 64, 280 MB 192.1, 177.1, 170.4 / 190.6, 190.8, 195.0, 330 MB 233.9, 218.1, 209.7 / 229.1, 226.3, 230.2, 390 MB 273.0,
//     265.1, 254.7 / 274.7, 271.3, 275.6; 72 by 64, 285 MB 197.0, 179.2, 173.1 / 202.6, 203.0, 204.3; 132 by 128, 280 MB 181.8, 173.4, 167.5 / 182.3,
//     178.9, 182.8; 200 by 64, 330 MB 231.5, 221.0, 208.1 / 231.6, 226.0, 231.3; 260 by 64, 279 MB 181.3, 172.0, 165.7 / 182.8, 179.4, 183.1; 260 by
//     32, 355 MB 245.9, 238.6, 229.6 / 252.8, 249.7, 254.1.  In order stay small layers (132 by
//     64, 30 MB, one transfer buffer, 23.5 / 23.6 / 24.9 / 25.9 / 27.7).  Moves: 333 by 64, 206 MB 74.1 / 69.4 / 69.1 / 68.9 / 69.2, 132 by 64, 1.9 GB
//     663 / 640 / 632 / 626 / 624, 292 MB 96.0 / 96.4 / 96.1 / 95.8 / 95.9.
//   moves (150 MB of 90-byte rows by 32: flat 54, tiled with 256 / 128 lanes 53 / 59) and the host link: flat up to
//     kAnyFlatPastWindows, tiles of 256 lanes, 128 below two such tiles (1026 by 4: 377 us at 256, 286 at 128).
//   across the host link: tiles on few workgroups (kHostSideGroups); a flat launch has as many as ever, since few of them
//     would not keep the link busy with small descriptors (in / out, flat and tiled: 132 by 1, 8 MB, 149 / 153 and 684 /
//     255; 36 by 2, 40 MB, 716 / 743 and 6870 / 3109; 132 by 16, 40 MB, 726 / 736 and 793 / 750).
static void launch_any(const kvl_plan_t *plan, bool pack, const CopyArgs &a, uint32_t planes, bool far_host,
                       const On &on) {
    const uint64_t unit_bytes = (uint64_t)plan->max_unit_rows * a.row_elems[a.plane_begin];
    const uint64_t windows = (unit_bytes + 30) / 16;       // 16-byte windows a span of that size can touch
    const bool hop = !plan->paired && !far_host;
    const bool alike = 2ull * plan->max_unit_rows * plan->units.size() <= 3 * plan->hit_tokens;
    const bool lines = (uint64_t)plan->layout.block_tokens * a.row_elems[a.plane_begin] % 128 == 0 && plan->payload_bytes > kCachedFlatBytes;
    const bool thin = plan->tuning.max_groups && plan->tuning.max_groups < kCappedLanes / 256;
    const bool flat = windows <= (!hop || !alike || thin ? kAnyFlatPastWindows : lines ? kAnyFlatLinesWindows : kAnyFlatWindows);
    const bool kept = far_host || (!plan->paired && plan->payload_bytes <= (flat ? kCachedFlatBytes : kCachedLayerBytes));
    // the widest plane's share of the layer, where blocks are of whole lines
    uint64_t row_bytes = 0, widest_row = 0;
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p) {
        row_bytes += plan->layout.row_bytes[p];
        widest_row = std::max<uint64_t>(widest_row, plan->layout.row_bytes[p]);
    }
    const double share = lines ? (double)widest_row / (double)row_bytes : 1.0;
    const bool of_blocks = plan->max_unit_rows <= 2ull * plan->layout.block_tokens && unit_bytes < (64u << 10);
    const bool small = hop && !flat && plan->payload_bytes <= kSmallOffLinesBytes;
    const bool once = hop && !kept && plan->payload_bytes <= (share < 0.875 ? kReadOnceManyBytes : kReadOnceBytes);
    const bool scatter_once = once && !(share < 0.8 && of_blocks && plan->payload_bytes > kScatterOnceManyBytes);
    const bool late = hop && !kept && !once && share < 0.8 && of_blocks && unit_bytes >= kLateTileBytes;
    const uint64_t spanned = unit_bytes + 127;              // with the lanes before its first byte on the line
    auto tiles_of = [spanned](uint64_t lanes) { return (spanned + 16 * lanes - 1) / (16 * lanes); };
    uint64_t cap = plan->tuning.max_groups;
    if (!cap && far_host) cap = 2 * kHostSideGroups;       // (one vector per lane: see kHostSideGroups)
    uint32_t threads = plan->tuning.block_threads;
    if (!plan->threads_chosen) {
        const bool is_short = spanned <= 2 * 256 * 16;
        const double busy_128 = (double)spanned / (2048.0 * (double)tiles_of(128)), busy_256 = (double)spanned / (4096.0 * (double)tiles_of(256));
        const bool halve = busy_128 - busy_256 > 0.125;
        if (flat) threads = 1024;
        else if (!hop) threads = is_short ? 128 : 256;
        else if (small) threads = 128;
        else if (pack && (kept || once)) threads = 64;
        else threads = halve && (is_short || kept || (scatter_once && plan->payload_bytes <= kHalveBytes)) ? 128 : 256;
        if (hop && cap && a.n_units * tiles_of(threads) > cap)
            while (threads < 256 && cap * threads < kCappedLanes) threads *= 2;
    }
    uint64_t run_bytes = 0;
    if (plan->paired) {
        run_bytes = 256u << 10;
    } else if (!far_host && (small || plan->payload_bytes > (flat ? kFlatOrderBytes : kOddOrderBytes))) {
        const bool beyond = plan->payload_bytes > kOnDieBytes;
        if (flat) run_bytes = 256u << 10;
        else if (!beyond || plan->payload_bytes > kWaveTileBytes) run_bytes = 512u << 10;
        else run_bytes = 128u << 10;
    }
    const uint64_t per_unit = tiles_of(threads);
    uint64_t per_launch = flat ? ((1ull << 31) - threads) / windows : (uint64_t)INT32_MAX / per_unit;
    if (flat && plan->tuning.max_groups)
        per_launch = std::min<uint64_t>(per_launch, (uint64_t)plan->tuning.max_groups * threads / windows);
    per_launch = std::max<uint64_t>(1, per_launch);
    for (uint64_t first = 0; first < a.n_units; first += per_launch) {
        CopyArgs part = a;
        part.unit_begin = a.unit_begin + (uint32_t)first;
        part.n_units = (uint32_t)std::min<uint64_t>(per_launch, a.n_units - first);
        const uint64_t tiles = part.n_units * per_unit;
        bool walk = false;
        const uint32_t groups = flat ? (uint32_t)((part.n_units * windows + threads - 1) / threads)
                                     : launch_groups(tiles, threads, (uint32_t)cap, &walk);
        walk = walk || (late && !flat);         // (one tile to a workgroup all the same)
        const uint32_t x = (uint32_t)(flat ? windows : per_unit), n_tiles = (uint32_t)tiles;
        dim3 grid(groups, planes), block(threads);
        if (pack) {
            if (small && gather_stays(false, plan->payload_bytes, on.done != nullptr)) launch_any_one<true, true, 0, true>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
            else if (far_host) launch_any_one<true, true, 2, false>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
            else if (kept || (once && !flat)) launch_any_one<true, true, 2, true>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
            else launch_any_one<true, true, 1, true>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
        } else {
            if (kept) launch_any_one<false, false, 3, false>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
            else if (scatter_once) launch_any_one<false, true, 1, true>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
            else launch_any_one<false, true, 1, false>(flat, walk, grid, block, on, part, x, n_tiles, run_bytes);
        }
    }
}

// Planes of unlike rows in one launch: 16-byte vectors on this device, in layers of up to kPlanesAtOnceBytes.  All planes by
// the row map where one of them would take it (made, and not awaited by a stream under capture), else all by tiles, of
// whose lanes no plane may idle half.  False: they go apart.
//   lanes of the tiles: a gather's and a scatter's as the widest plane has them; a move's 64 where the descriptors are alike
//     and begin on lines, else 128 where that leaves clearly fewer idle over all planes (moves, us, 256 / 128: 656- and
//     336-byte rows by 40 in runs, 199 MB, 75.0 / 67.7; 272 and 144 by 48, 205 MB, 73.4 / 69.5; 656 and 128 by 16 at random,
//     20 MB, 10.9 / 8.5).
//   in larger layers a plane's own lanes are worth more than the launch.  Where the descriptors are alike (kPlanesAlikeBytes) a
//     hop's planes go apart if the common lanes are more in all (hops, together / apart: 256 and 128 by 100, 150 MB 92.3 /
//     90.5, 333 MB 220 / 213; 656 and 336 by 64, 91 MB 61.5 / 63.6, 302 MB 189 / 184), a move's if one would have another
//     width (160 and 320 by 16, 84 MB 31.5 / 32, 181 MB 66.9 / 63; 320 and 640 by 8, 132 MB 49.2 / 47); so do both where they
//     are not alike (kPlanesUnlikeBytes; moves in runs: 512 and 256 by 4, 45 MB 21.7 / 22.2, 64 MB 30.0 / 29.0, 299 MB 134 /
//     120; 256 and 128 by 16, 60 MB 25.1 / 26.6, 200 MB 80.0 / 76.6).
static bool launch_planes(const kvl_plan_t *plan, bool pack, const CopyArgs &a, uint32_t plane_end, const On &on) {
    const uint32_t begin = a.plane_begin;
    if (plan->tuning.variant || plan->tuning.max_groups || plan->threads_chosen || plan->payload_bytes > kPlanesAtOnceBytes)
        return false;
    const double average = (double)plan->hit_tokens / (double)plan->units.size();
    bool lines = true, by_rows = false, askew = false;
    uint32_t widest = 0, threads = 0;
    for (uint32_t p = begin; p < plane_end; ++p) {
        lines = lines && plan->layout.row_bytes[p] % 128 == 0;
        by_rows = by_rows || takes_row_map(plan, plan->layout.row_bytes[p], pack);
        widest = std::max(widest, a.row_elems[p]);
        askew = askew || (a.row_elems[p] >= 16 && a.row_elems[p] < 64 && a.row_elems[p] % 8 != 0);
    }
    if (by_rows) {
        if (!plan->d_row_map || !row_map_ready(plan, on.stream)) return false;
        threads = kDefaultBlockThreads;
    } else {
        auto lanes = [&](uint32_t p, uint64_t t) { return (plan->max_unit_rows * (uint64_t)a.row_elems[p] + t - 1) / t * t; };
        auto apart = [&](uint32_t p) {          // the lanes that the plane would have by itself
            return plan->paired ? move_threads(plan, plan->layout.row_bytes[p]) : tile_threads((uint64_t)plan->max_unit_rows * a.row_elems[p]);
        };
        const bool alike = 2ull * plan->max_unit_rows * plan->units.size() <= 3 * plan->hit_tokens;
        if (!plan->paired) {
            threads = tile_threads((uint64_t)plan->max_unit_rows * widest);
        } else {
            double vectors = 0, of_256 = 0, of_128 = 0;
            for (uint32_t p = begin; p < plane_end; ++p) {
                vectors += (double)plan->max_unit_rows * a.row_elems[p];
                of_256 += (double)lanes(p, 256);
                of_128 += (double)lanes(p, 128);
            }
            threads = lines && alike ? 64 : vectors / of_128 - vectors / of_256 > 0.07 ? 128 : kDefaultBlockThreads;
        }
        if (plan->payload_bytes > (alike ? kPlanesAlikeBytes : kPlanesUnlikeBytes)) {
            double shared = 0, own = 0;
            bool same = true;
            for (uint32_t p = begin; p < plane_end; ++p) {
                shared += (double)lanes(p, threads);
                own += (double)lanes(p, apart(p));
                same = same && apart(p) == threads;
            }
            if (alike && !plan->paired ? shared > 1.03 * own : !same) return false;
        }
    }
    const kvl_unit_t &first = plan->units[a.unit_begin], &last = plan->units[a.unit_begin + a.n_units - 1];
    PlanesArgs pl{};
    pl.row_begin = first.xfer_row;
    pl.n_rows = by_rows ? last.xfer_row + last.n_rows - first.xfer_row : 0;
    uint64_t groups = 0;
    for (uint32_t p = 0; p < KVL_MAX_PLANES; ++p) {
        pl.group_end[p] = UINT32_MAX;
        if (p < begin || p >= plane_end) continue;
        const uint64_t row = a.row_elems[p];
        const bool dst_lines = plan->layout.row_bytes[p] % 128 == 0 && (pack ? a.xfer[p] : a.pool[p]) % 128 == 0;
        pl.align_dst[p] = dst_lines ? 0u : 1u;
        const uint64_t tiles = (plan->max_unit_rows * row + (dst_lines ? 0 : 7) + threads - 1) / threads;
        if (!by_rows && average * (double)row < 0.5 * (double)(tiles * threads)) return false;
        pl.per_unit[p] = (uint32_t)tiles;
        pl.plain[p] = plan->layout.row_bytes[p] % 128 != 0 && plan->payload_bytes <= kPlainReadBackBytes ? 1u : 0u;
        groups += by_rows ? (pl.n_rows * row + 7 + threads - 1) / threads : a.n_units * tiles;
        if (groups > kMaxLanesPerLaunch / threads || groups > (uint64_t)INT32_MAX) return false;
        pl.group_end[p] = (uint32_t)groups;
    }
    const dim3 grid((uint32_t)groups), block(threads);
    const uint32_t *map = plan->d_row_map;
    if (plan->paired && move_nt(plan->payload_bytes)) KVL_LAUNCH((kvl_planes_kernel<true, 1, 0>), grid, block, on, a, pl, map);
    else if (plan->paired) KVL_LAUNCH((kvl_planes_kernel<true, 3, 0>), grid, block, on, a, pl, map);
    else if (pack && by_rows) KVL_LAUNCH((kvl_planes_kernel<true, 2, 1>), grid, block, on, a, pl, map);
    else if (pack) KVL_LAUNCH((kvl_planes_kernel<true, 2, 0>), grid, block, on, a, pl, map);
    else if (by_rows && plan->payload_bytes > (askew ? kPlainReadBackBytes : kPlanesCachedBytes)) KVL_LAUNCH((kvl_planes_kernel<false, 3, 2>), grid, block, on, a, pl, map);
    else if (by_rows) KVL_LAUNCH((kvl_planes_kernel<false, 3, 1>), grid, block, on, a, pl, map);
    else KVL_LAUNCH((kvl_planes_kernel<false, 3, 0>), grid, block, on, a, pl, map);
    return true;
}

int launch_units(const kvl_plan_t *plan, bool pack, uint32_t unit_begin, uint32_t unit_end,
                 uint32_t plane_begin, uint32_t plane_end,
                 void *const *pool_planes, const uintptr_t *xfer_plane, hipStream_t stream, bool far_host) {
    if (unit_end <= unit_begin || plane_end <= plane_begin) return KVL_OK;
    if (!plan->d_units || unit_end > plan->units.size() || plane_end > plan->layout.n_planes)
        return KVL_EINVAL;
    int rc_dev = check_device(plan);
    if (rc_dev != KVL_OK) return rc_dev;
    CopyArgs a{};
    a.units = plan->d_units;
    a.unit_begin = unit_begin;
    a.n_units = unit_end - unit_begin;
    a.plane_begin = plane_begin;
    bool vec = plan->vec16, unlike = false;
    for (uint32_t p = plane_begin; p < plane_end; ++p) {
        if (!pool_planes[p]) return KVL_EINVAL;
        a.pool[p] = reinterpret_cast<uintptr_t>(pool_planes[p]);
        a.xfer[p] = xfer_plane[p];
        vec = vec && (a.pool[p] % 16 == 0) && (a.xfer[p] % 16 == 0);
        unlike = unlike || plan->layout.row_bytes[p] != plan->layout.row_bytes[plane_begin];
    }
    for (uint32_t p = plane_begin; p < plane_end; ++p)
        a.row_elems[p] = vec ? plan->layout.row_bytes[p] / 16 : plan->layout.row_bytes[p];
    // Planes of different row sizes share a launch in which each has its own number of workgroups, or go in launches of
    // their own: with the tile count of the widest for every plane a narrow plane's workgroups would mostly find nothing
    // to do (K/V-style planes of 1024 and 128 bytes that way: 2.8 TB/s; apart: 6 TB/s and more).
    if (unlike) {
        if (vec && !far_host) {
            On on(plan, stream);
            if (launch_planes(plan, pack, a, plane_end, on)) return on.made();
        }
        for (uint32_t q = plane_begin; q < plane_end;) {
            uint32_t e = q + 1;
            while (e < plane_end && plan->layout.row_bytes[e] == plan->layout.row_bytes[q]) ++e;
            int rc = launch_units(plan, pack, unit_begin, unit_end, q, e, pool_planes, xfer_plane, stream, far_host);
            if (rc != KVL_OK) return rc;
            q = e;
        }
        return KVL_OK;
    }

    On on(plan, stream);
    uint32_t threads = plan->tuning.block_threads;
    // default: tiled, one vector per lane; cache policies as measured (see the top of kvl_copy_kernels.h)
    uint32_t v;
    if (plan->tuning.variant) {
        v = plan->tuning.variant - 1;
    } else {
        bool rows_128 = true;       // every span starts on a 128-byte line of the transfer buffer
        for (uint32_t p = plane_begin; p < plane_end; ++p)
            rows_128 = rows_128 && plan->layout.row_bytes[p] % 128 == 0;
        const uint64_t payload = far_host ? std::max(plan->payload_bytes, kNtScatterBytes + 1) : plan->payload_bytes;
        v = plan->paired ? (move_nt(payload) ? kNtMoveCode : kMoveCode) : default_tile_code(pack, rows_128, payload, on.done != nullptr);
        // across the host link: two vectors per lane, so that the few workgroups of the thin
        // form (kHostSideGroups) keep enough bytes in flight
        if (far_host) v |= 3u;
    }
    if (v & 256u) v = (v & ~(3u | 32u | 128u)) | 2u;      // the pipelined form is a tiled one, one vector per lane
    uint32_t widest = 0;        // vectors of the largest descriptor, over the planes of this launch
    for (uint32_t p = plane_begin; p < plane_end; ++p) widest = std::max(widest, a.row_elems[p]);
    const uint64_t unit_vecs = (uint64_t)plan->max_unit_rows * widest;
    const uint32_t row_bytes = plan->layout.row_bytes[plane_begin];
    // (explicit variants take their tiles in order, so that they differ in their form alone)
    const uint64_t run_bytes = far_host || plan->tuning.variant ? 0 : tile_run_bytes(shape_of(plan), row_bytes);
    if (vec && !plan->threads_chosen && !plan->tuning.variant) {
        threads = plan->paired ? move_threads(plan, row_bytes) : far_host ? tile_threads(unit_vecs) : hop_threads(shape_of(plan), row_bytes);
    }
    // descriptors that fill less than half a workgroup: deal the lanes out without tiles
    if (vec && !plan->tuning.variant && unit_vecs * 2 <= plan->tuning.block_threads) {
        v = plan->paired ? kFlatMoveCode : pack ? kFlatPackCode : kFlatUnpackCode;
        threads = plan->paired && !plan->threads_chosen ? 1024u : plan->tuning.block_threads;
    }
    dim3 block(threads);
    const kvl_unit_t &u_first = plan->units[unit_begin], &u_last = plan->units[unit_end - 1];
    if (vec && !plan->tuning.variant && !plan->tuning.max_groups && !far_host && plan->d_row_map &&
        rows_ahead(plan, row_bytes, pack) && row_map_ready(plan, stream)) {
        // the launch is laid out over the transfer rows of these descriptors; its lanes are numbered with 32 bits
        if (!plan->threads_chosen) threads = kDefaultBlockThreads;
        const uint64_t rows = (uint64_t)u_last.xfer_row + u_last.n_rows - u_first.xfer_row;
        const uint64_t per_launch = std::max<uint64_t>(1, ((1ull << 32) - threads - 8) / widest);
        const bool lines = row_bytes % 128 == 0;
        const uint64_t rows_run = run_bytes && !(lines && plan->payload_bytes > kOnDieBytes) ? kRowsRunBytes : 0;
        for (uint64_t first = 0; first < rows; first += per_launch) {
            const uint32_t n = (uint32_t)(std::min<uint64_t>(per_launch, rows - first) * widest);
            const uint32_t row_begin = (uint32_t)(u_first.xfer_row + first);
            dim3 grid((uint32_t)(((uint64_t)n + 7 + threads - 1) / threads), plane_end - plane_begin);
            if (pack && gather_stays(lines, plan->payload_bytes, on.done != nullptr)) launch_rows<true, true, 0>(grid, dim3(threads), on, a, plan->d_row_map, row_begin, n, rows_run);
            else if (pack) launch_rows<true, true, 2>(grid, dim3(threads), on, a, plan->d_row_map, row_begin, n, rows_run);
            else if (lines && !scatter_nt(lines, plan->payload_bytes)) launch_rows<false, true, 3>(grid, dim3(threads), on, a, plan->d_row_map, row_begin, n, rows_run);
            else launch_rows<false, true, 1>(grid, dim3(threads), on, a, plan->d_row_map, row_begin, n, rows_run);
        }
    } else if (!vec) {
        launch_any(plan, pack, a, plane_end - plane_begin, far_host, on);
    } else if (v & 128u) {
        // lane indices are 31 bits (TileDivisor): split the descriptors over launches where they would not fit
        // (tuning.max_groups, if given, lowers the workgroups per launch further)
        uint64_t lanes_per_launch = (1ull << 31) - threads;
        if (plan->tuning.max_groups)
            lanes_per_launch = std::min<uint64_t>(lanes_per_launch, (uint64_t)plan->tuning.max_groups * threads);
        const uint64_t per_launch = std::max<uint64_t>(1, lanes_per_launch / std::max<uint64_t>(1, unit_vecs));
        for (uint64_t first = 0; first < a.n_units; first += per_launch) {
            CopyArgs part = a;
            part.unit_begin = a.unit_begin + (uint32_t)first;
            part.n_units = (uint32_t)std::min<uint64_t>(per_launch, a.n_units - first);
            const uint64_t lanes = (uint64_t)part.n_units * unit_vecs;
            dim3 grid((uint32_t)((lanes + threads - 1) / threads), plane_end - plane_begin);
            if (pack) launch_flat_variant<true>(v, grid, block, on, part, (uint32_t)unit_vecs);
            else launch_flat_variant<false>(v, grid, block, on, part, (uint32_t)unit_vecs);
        }
    } else if ((v & 3u) >= 2u) {
        const uint32_t vpt = (v & 3u) == 3u ? 2 : 1;
        uint32_t max_row = 0;
        for (uint32_t p = plane_begin; p < plane_end; ++p) max_row = std::max(max_row, a.row_elems[p]);
        const uint64_t per_tile = (uint64_t)threads * vpt;
        // destination spans start on 128-byte lines by themselves when the rows and the base do
        bool dst_lines = true;
        for (uint32_t p = plane_begin; p < plane_end; ++p)
            dst_lines = dst_lines && plan->layout.row_bytes[p] % 128 == 0 &&
                        (pack ? a.xfer[p] : a.pool[p]) % 128 == 0;
        const uint32_t al = (dst_lines || (v & 64u)) ? 0u : 1u;
        const uint64_t tpu = ((uint64_t)plan->max_unit_rows * max_row + (al ? 7 : 0) + per_tile - 1) / per_tile;
        const uint64_t blocks = (uint64_t)a.n_units * tpu;
        if (tpu == 0 || blocks > (uint64_t)INT32_MAX) return KVL_ERANGE;
        // fewer workgroups than tiles, each walking over several: on request, or because the
        // far side is host memory
        const uint32_t cap = plan->tuning.max_groups ? plan->tuning.max_groups : (far_host ? kHostSideGroups : 0u);
        if (v & 256u) {
            // pipelined walk: as many workgroups as the machine holds at once (32 wavefronts per compute
            // unit), shared among the planes of the launch
            const uint64_t resident = (uint64_t)compute_units(plan->device) * (2048u / threads);
            uint64_t groups = cap ? cap : std::max<uint64_t>(1, resident / (plane_end - plane_begin));
            groups = std::min<uint64_t>(groups, blocks);
            dim3 grid((uint32_t)groups, plane_end - plane_begin);
            if (pack) launch_pipe_variant<true>(v, grid, block, on, a, (uint32_t)tpu, al, (uint32_t)blocks);
            else launch_pipe_variant<false>(v, grid, block, on, a, (uint32_t)tpu, al, (uint32_t)blocks);
            return on.made();
        }
        // one workgroup per tile, unless a cap was asked for or the launch would not fit
        bool walk = false;
        const uint32_t groups = launch_groups(blocks, threads, cap, &walk);
        const uint32_t n_tiles = walk ? (uint32_t)blocks : 0u;
        dim3 grid(groups, plane_end - plane_begin);
        if (pack) {
            if (vpt == 2) launch_tile_variant<true, 2>(v, grid, block, on, a, (uint32_t)tpu, al, n_tiles, run_bytes);
            else launch_tile_variant<true, 1>(v, grid, block, on, a, (uint32_t)tpu, al, n_tiles, run_bytes);
        } else {
            if (vpt == 2) launch_tile_variant<false, 2>(v, grid, block, on, a, (uint32_t)tpu, al, n_tiles, run_bytes);
            else launch_tile_variant<false, 1>(v, grid, block, on, a, (uint32_t)tpu, al, n_tiles, run_bytes);
        }
    } else {
        const uint32_t per_wg = (v & 3u) == 1u ? threads / 64 : 1;
        if ((uint64_t)((a.n_units + per_wg - 1) / per_wg) * threads > kMaxLanesPerLaunch) return KVL_ERANGE;
        dim3 grid((a.n_units + per_wg - 1) / per_wg, plane_end - plane_begin);
        if (pack) launch_span_variant<true>(v, grid, block, on, a);
        else launch_span_variant<false>(v, grid, block, on, a);
    }
    return on.made();
}

// Launch the layout-converting kernel on descriptors [unit_begin, unit_end).  A
// descriptor of block index k finds its rows at
//   base + k * block_pitch + layer_off + (plane span, row) inside the Layer Block;
// for a buffer of Full Blocks block_pitch is the Full-Block size and layer_off the
// layer's offset in it, for a staging area of Layer Blocks block_pitch is the
// Layer-Block size and layer_off is 0 (base may then lie before the area).
int fullblock_launch(const kvl_plan_t *plan, bool to_pool, uintptr_t base, uint64_t block_pitch,
                     uint64_t layer_off, uint32_t unit_begin, uint32_t unit_end,
                     void *const *pool_planes, hipStream_t stream, bool far_host) {
    if (unit_end <= unit_begin) return KVL_OK;
    if (!plan->d_units || unit_end > plan->units.size()) return KVL_EINVAL;
    const uint32_t P = plan->layout.n_planes;
    const uint64_t bs = plan->layout.block_tokens;
    bool vec = plan->vec16 && base % 16 == 0 && block_pitch % 16 == 0 && layer_off % 16 == 0;
    for (uint32_t p = 0; p < P; ++p) {
        if (!pool_planes[p]) return KVL_EINVAL;
        vec = vec && reinterpret_cast<uintptr_t>(pool_planes[p]) % 16 == 0;
    }
    const uint64_t e = vec ? 16 : 1;          // element size
    FullBlockArgs a{};
    a.units = plan->d_units + unit_begin;
    a.n_units = unit_end - unit_begin;
    a.block_tokens = plan->layout.block_tokens;
    a.blocks = base;
    a.fb_elems = block_pitch / e;
    uint64_t plane_off = 0;
    for (uint32_t p = 0; p < P; ++p) {
        a.row_elems[p] = (uint32_t)(plan->layout.row_bytes[p] / e);
        a.pool[p] = reinterpret_cast<uintptr_t>(pool_planes[p]);
        a.layer_plane_off[p] = (layer_off + plane_off) / e;
        plane_off += bs * plan->layout.row_bytes[p];
    }
    // across the host link: two vectors per lane on few workgroups (as the copy kernels do, see launch_units)
    const uint32_t vpt = far_host && vec ? 2 : 1;
    // vectors of a descriptor's plane, with those before it on its first line (none where every descriptor begins on a line:
    // whole blocks of whole lines, or rows of whole lines)
    const bool whole = !(plan->flags & KVL_TOKENS_APPEND) && plan->units.size() == plan->blocks_touched;
    bool lines = base % 128 == 0 && block_pitch % 128 == 0 && layer_off % 128 == 0, level = lines;
    for (uint32_t p = 0; p < P; ++p) {
        const uint64_t row = plan->layout.row_bytes[p];
        level = level && reinterpret_cast<uintptr_t>(pool_planes[p]) % 128 == 0 && bs * row % 128 == 0;
        lines = lines && reinterpret_cast<uintptr_t>(pool_planes[p]) % 128 == 0 && (row % 128 == 0 || (whole && bs * row % 128 == 0));
    }
    uint64_t vectors[KVL_MAX_PLANES] = {}, most = 0;
    for (uint32_t p = 0; p < P; ++p) {
        const uint64_t bytes = (uint64_t)plan->max_unit_rows * plan->layout.row_bytes[p];
        vectors[p] = (bytes + (lines || vpt == 2 ? 0 : vec ? 112 : 127) + 15) / 16;
        most = std::max(most, (bytes + (vec ? 0 : 127) + 4096 * vpt - 1) / (4096 * vpt));
    }
    // Lanes of a tile: 256, or fewer where that leaves clearly fewer without work.  Both directions, us, 256 / 128 / 64 lanes
    // (share of the lanes busy): 336-byte rows by 16, 31 MB, 27.9 / 24.1 / 24.3 (.67 .89 .89); 496 by 1, 9 MB, 30.9 / 20.9 /
    // 16.9 (.14 .28 .56); 48 by 100, 31 MB, 32.8 / 28.1 / 26.9 (.60 .80 .96); 2064 by 1, 45.4 / 48.4 / 42.6 (.53 .53 .71);
    // 333 by 100, 59 MB, 49.0 / 50.4 / 52.7 (.91 .96 .99); 132 by 32, 28 MB, 30.5 / 23.5 / 22.4 (.53 .71 .85); 132 and 64 by
    // 64, 28 MB, 23.4 / 24.5 / 22.2 (.63 .78 .89).  In several planes 64 lanes or 256 (four layers, 256 / 128 / 64: 32 and 656 by
    // 32, 73 MB, 197 / 203 / 198 (.77 .90 .98); 1152 and 128 by 16, 169 MB, 410 / 430 / 419 (.83 1 1); 144 and 352 by 64, 139
    // MB, 337 / 344 / 337 (.86 .97 1); 132 and 64 by 64, blocks on lines, 96 MB, 285 / 249 / 242 (.77 .88 .94)).
    uint32_t threads = 256;
    if (!far_host) {
        auto busy = [&](uint64_t t) {
            uint64_t work = 0, lanes = 0;
            for (uint32_t p = 0; p < P; ++p) {
                work += vectors[p];
                lanes += (vectors[p] + t - 1) / t * t;
            }
            return (double)work / (double)lanes;
        };
        if (P > 1) {
            if (busy(64) > busy(threads) + 0.17) threads = 64;
        } else {
            if (busy(128) > busy(threads) + 0.07) threads = 128;
            if (busy(64) > busy(threads) + 0.09) threads = 64;
        }
    }
    // (a cap that was asked for is meant for each plane, see kvl_tuning_t)
    const uint32_t cap = plan->tuning.max_groups ? (uint32_t)std::min<uint64_t>((uint64_t)plan->tuning.max_groups * P, UINT32_MAX)
                                                 : (far_host ? (vec ? kHostSideGroups : 2 * kHostSideGroups) : 0u);
    auto tiles_of = [&](uint64_t lanes) {
        uint64_t n = 0;
        for (uint32_t p = 0; p < P; ++p) n += (vectors[p] + lanes * vpt - 1) / (lanes * vpt);
        return n;
    };
    // Under a cap on the workgroups they are widened until more than kCappedLanes are at work, or a quarter of them where
    // that makes no fewer tiles (the other wavefronts then only fetch descriptors ahead).  Load + persist of four layers, us, 64
    // or 128 / 256 lanes: 132-byte rows by 64, 33 MB, 64 workgroups 2911 / 919, 1024 225 / 116, 4096 106.6 / 100.0 (128 lanes
    // 100.9); 336 by 16, 32 MB, 512 224 / 179, 4096 95.7 / 107; 496 by 1, 9 MB, 64 1509 / 1413, 1024 129 / 140, 4096 61 / 88.
    while (threads < 256 && cap && a.n_units * tiles_of(threads) > cap &&
           (uint64_t)cap * threads <= (tiles_of(2 * threads) < tiles_of(threads) ? kCappedLanes : kCappedLanes / 4))
        threads *= 2;
    uint64_t tpu = 0;
    for (uint32_t p = 0; p < KVL_MAX_PLANES; ++p) {
        const uint64_t tiles = (vectors[p] + (uint64_t)threads * vpt - 1) / ((uint64_t)threads * vpt);
        tpu += tiles;
        a.tile_end[p] = (uint32_t)std::min<uint64_t>(tpu, UINT32_MAX);
    }
    // (the limit is that of tiles of 256 lanes, whatever their lanes are)
    if (a.n_units * most > (uint64_t)INT32_MAX || tpu > (uint64_t)INT32_MAX) return KVL_ERANGE;
    // (an order of 512 KiB is level; 128 KiB are 1 % behind)
    const uint64_t run_bytes = far_host ? 0 : 256u << 10;
    bool quick = vec && !far_host && a.fb_elems <= UINT32_MAX;
    for (uint32_t p = 1; p < P; ++p) quick = quick && a.row_elems[p] == a.row_elems[0];
    const TileDivisor by_tiles((uint32_t)tpu);
    a.magic = by_tiles.magic;
    a.shift = by_tiles.shift;
    a.tokens_magic = UINT32_MAX / a.block_tokens;
    On on(plan, stream);
    // the tiles of all planes are numbered with 32 bits: descriptors that have more go in several launches
    const uint32_t n_all = a.n_units, per_launch = (uint32_t)(INT32_MAX / tpu);
    for (uint32_t first = 0; first < n_all; first += per_launch) {
        a.n_units = std::min(per_launch, n_all - first);
        const uint32_t n_tiles = a.n_units * (uint32_t)tpu;
        bool walk = false;
        dim3 grid(launch_groups(n_tiles, threads, cap, &walk)), block(threads);
        if (quick && !walk) {
            const uint32_t per_plane = (uint32_t)tpu / P, tokens = a.block_tokens;
            const TileDivisor d(per_plane);
            TileMore more{};
            for (uint32_t p = 1; p < P; ++p) {
                more.pool[p - 1] = a.pool[p];
                more.xfer[p - 1] = a.blocks + a.layer_plane_off[p] * 16;
            }
            grid = dim3(n_tiles / P, P);
#define KVL_FB_QUICK(TO_POOL) \
            KVL_LAUNCH((kvl_fullblock_quick_kernel<TO_POOL>), grid, block, on, a.units, a.pool[0], a.blocks + a.layer_plane_off[0] * 16, (uint32_t)a.fb_elems, \
                       a.row_elems[0], per_plane, d.magic, d.shift << 16 | threads, tokens, UINT32_MAX / tokens, tile_order(grid.x, 16ull * threads, run_bytes), more)
            if (to_pool) KVL_FB_QUICK(true);
            else KVL_FB_QUICK(false);
#undef KVL_FB_QUICK
            a.units += a.n_units;
            continue;
        }
        const uint32_t order = walk ? 0u : tile_order(n_tiles, 16ull * vpt * threads, run_bytes);
#define KVL_FB_LAUNCH(...) \
        KVL_LAUNCH((kvl_fullblock_kernel<__VA_ARGS__>), grid, block, on, a, (uint32_t)tpu, n_tiles, order)
        if (to_pool) {
            if (!vec && far_host) KVL_FB_LAUNCH(true, false, 1, true, 2, false);
            else if (!vec) KVL_FB_LAUNCH(true, false, 1, true, 2, true);
            else if (far_host) KVL_FB_LAUNCH(true, true, 2, false, 3, false);
            else KVL_FB_LAUNCH(true, true, 1, true, 2, true);
        } else {
            if (!vec && far_host) KVL_FB_LAUNCH(false, false, 1, true, 3, false);
            else if (!vec && level) KVL_FB_LAUNCH(false, false, 1, true, 3, false);
            else if (!vec) KVL_FB_LAUNCH(false, false, 1, true, 1, true);
            else if (far_host) KVL_FB_LAUNCH(false, true, 2, true, 0, false);
            else KVL_FB_LAUNCH(false, true, 1, true, 3, true);
        }
        a.units += a.n_units;
    }
#undef KVL_FB_LAUNCH
    return on.made();
}

// Bytes of one Layer Block (all planes of one block, one layer).
uint64_t layer_block_bytes(const kvl_plan_t *plan) {
    uint64_t lb = 0;
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p)
        lb += (uint64_t)plan->layout.block_tokens * plan->layout.row_bytes[p];
    return lb;
}

// What every Full-Block call asks of its plan and sizes.
int check_fullblock_args(const kvl_plan_t *plan, bool to_pool, uint64_t blocks_bytes, uint32_t layer) {
    if (!plan) return KVL_EINVAL;
    if ((plan->flags & KVL_HOST_ONLY) || !(plan->flags & KVL_NO_MERGE)) return KVL_EINVAL;
    if (!(plan->flags & (to_pool ? KVL_SCATTER : KVL_GATHER))) return KVL_EINVAL;
    if (layer >= plan->layout.n_layers) return KVL_EINVAL;
    const uint64_t fb = layer_block_bytes(plan) * plan->layout.n_layers;
    if (blocks_bytes < plan->blocks_touched * fb) return KVL_ESPACE;
    return KVL_OK;
}

int fullblock_layer(const kvl_plan_t *plan, bool to_pool, uintptr_t blocks, uint64_t blocks_bytes,
                    uint32_t layer, void *const *pool_planes, hipStream_t stream) {
    if (!pool_planes) return KVL_EINVAL;
    int rc = check_fullblock_args(plan, to_pool, blocks_bytes, layer);
    if (rc != KVL_OK) return rc;
    if (plan->units.empty()) return KVL_OK;
    if (!blocks) return KVL_EINVAL;
    const uint64_t lb = layer_block_bytes(plan), fb = lb * plan->layout.n_layers;
    rc = check_device(plan);
    if (rc == KVL_OK) rc = check_pool(plan, pool_planes, plan->layout.pool_blocks);
    if (rc == KVL_OK)
        rc = check_buffer(plan, reinterpret_cast<const void *>(blocks), plan->blocks_touched * fb, true);
    if (rc != KVL_OK) return rc;
    return fullblock_launch(plan, to_pool, blocks, fb, (uint64_t)layer * lb, 0, (uint32_t)plan->units.size(),
                            pool_planes, stream, is_host_memory(plan, reinterpret_cast<const void *>(blocks)));
}

}  // namespace kvl

extern "C" {

int kvl_fullblocks_to_pool_layer(const kvl_plan_t *plan, const void *full_blocks, uint64_t full_blocks_bytes,
                                 uint32_t layer, void *const *pool_planes, void *stream) {
    return kvl::fullblock_layer(plan, true, reinterpret_cast<uintptr_t>(full_blocks), full_blocks_bytes, layer,
                                pool_planes, (hipStream_t)stream);
}

int kvl_pool_to_fullblocks_layer(const kvl_plan_t *plan, const void *const *pool_planes, uint32_t layer,
                                 void *full_blocks, uint64_t full_blocks_bytes, void *stream) {
    return kvl::fullblock_layer(plan, false, reinterpret_cast<uintptr_t>(full_blocks), full_blocks_bytes, layer,
                                const_cast<void *const *>(pool_planes), (hipStream_t)stream);
}

int kvl_move_layer(const kvl_plan_t *plan, const void *const *src_pool_planes, void *const *dst_pool_planes,
                   void *stream) {
    if (!plan || !src_pool_planes || !dst_pool_planes) return KVL_EINVAL;
    if (!plan->paired || (plan->flags & KVL_HOST_ONLY)) return KVL_EINVAL;
    if (plan->units.empty()) return KVL_OK;
    int rc = kvl::check_pool(plan, src_pool_planes, plan->layout.pool_blocks);
    if (rc == KVL_OK) rc = kvl::check_pool(plan, dst_pool_planes, plan->dst_pool_blocks);
    if (rc != KVL_OK) return rc;
    // the gather kernel with the destination pool in the transfer buffer's place:
    // a paired descriptor's xfer_row is a row of the destination pool
    uintptr_t xp[KVL_MAX_PLANES];
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p) {
        if (!dst_pool_planes[p]) return KVL_EINVAL;
        xp[p] = reinterpret_cast<uintptr_t>(dst_pool_planes[p]);
    }
    return kvl::launch_units(plan, true, 0, (uint32_t)plan->units.size(), 0, plan->layout.n_planes,
                             const_cast<void *const *>(src_pool_planes), xp, (hipStream_t)stream);
}

int kvl_pack_layer(const kvl_plan_t *plan, const void *const *pool_planes, void *xfer,
                   uint64_t xfer_capacity, void *stream) {
    if (!plan || !pool_planes) return KVL_EINVAL;
    if (!(plan->flags & KVL_GATHER) || (plan->flags & KVL_HOST_ONLY) || plan->paired) return KVL_EINVAL;
    if (xfer_capacity < plan->payload_bytes) return KVL_ESPACE;
    if (plan->units.empty()) return KVL_OK;
    if (!xfer) return KVL_EINVAL;
    int rc = kvl::check_pool(plan, pool_planes, plan->layout.pool_blocks);
    if (rc == KVL_OK) rc = kvl::check_buffer(plan, xfer, plan->payload_bytes, true);
    if (rc != KVL_OK) return rc;
    uintptr_t xp[KVL_MAX_PLANES];
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p)
        xp[p] = reinterpret_cast<uintptr_t>(xfer) + plan->plane_base[p];
    return kvl::launch_units(plan, true, 0, (uint32_t)plan->units.size(), 0, plan->layout.n_planes,
                             const_cast<void *const *>(pool_planes), xp, (hipStream_t)stream,
                             kvl::is_host_memory(plan, xfer));
}

int kvl_unpack_layer(const kvl_plan_t *plan, const void *xfer, uint64_t xfer_bytes,
                     void *const *pool_planes, void *stream) {
    if (!plan || !pool_planes) return KVL_EINVAL;
    if (!(plan->flags & KVL_SCATTER) || (plan->flags & KVL_HOST_ONLY)) return KVL_EINVAL;
    if (xfer_bytes < plan->payload_bytes) return KVL_ESPACE;
    if (plan->units.empty()) return KVL_OK;
    if (!xfer) return KVL_EINVAL;
    int rc = kvl::check_pool(plan, pool_planes, plan->layout.pool_blocks);
    if (rc == KVL_OK) rc = kvl::check_buffer(plan, xfer, plan->payload_bytes, true);
    if (rc != KVL_OK) return rc;
    uintptr_t xp[KVL_MAX_PLANES];
    for (uint32_t p = 0; p < plan->layout.n_planes; ++p)
        xp[p] = reinterpret_cast<uintptr_t>(xfer) + plan->plane_base[p];
    return kvl::launch_units(plan, false, 0, (uint32_t)plan->units.size(), 0, plan->layout.n_planes,
                             pool_planes, xp, (hipStream_t)stream, kvl::is_host_memory(plan, xfer));
}

int kvl_copy_linear(const void *src, void *dst, uint64_t bytes, void *stream) {
    if (bytes == 0) return KVL_OK;
    if (!src || !dst) return KVL_EINVAL;
    if (bytes % 16 || reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(dst) % 16)
        return KVL_EINVAL;
    int rc = kvl_check_buffer(src, bytes, 1);
    if (rc == KVL_OK) rc = kvl_check_buffer(dst, bytes, 1);
    if (rc != KVL_OK) return rc;
    // a launch holds fewer than 2^32 lanes: larger copies go in several
    const uint64_t n = bytes / 16, per_launch = (kvl::kMaxLanesPerLaunch / 256) * 256;
    for (uint64_t first = 0; first < n; first += per_launch) {
        const uint64_t m = std::min<uint64_t>(per_launch, n - first);
        hipLaunchKernelGGL(kvl::kvl_linear_kernel, dim3((uint32_t)((m + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           static_cast<const kvl::v4u *>(src) + first, static_cast<kvl::v4u *>(dst) + first, m);
        KVL_HIP(hipGetLastError());
    }
    return KVL_OK;
}

int kvl_ceiling_kernel(const kvl_ceiling_t *c, const void *src, uint64_t src_bytes, void *dst, uint64_t dst_bytes,
                       uint64_t bytes, const uint32_t *block_table, void *stream) {
    using namespace kvl;
    if (!c || !src || !dst || bytes == 0) return KVL_EINVAL;
    if (c->mode > KVL_CEILING_WRITE || c->skew_bytes % 16 || c->skew_bytes >= 128 || c->block_bytes % 16) return KVL_EINVAL;
    if (bytes % 16 || reinterpret_cast<uintptr_t>(src) % 128 || reinterpret_cast<uintptr_t>(dst) % 128) return KVL_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    // The halves of a copy alone go in order in wide workgroups: workgroups of one wavefront are launched at some 4.8 a nanosecond,
    // which would bound them (4 GiB read or written so 4.8 TB/s, in wide ones 6.9 and 7.0; the copy has half as many for its traffic).
    const bool halves = c->mode != KVL_CEILING_COPY;
    if (c->block_bytes == 0) {
        // one linear stream; the skew shifts the source
        if (src_bytes < bytes + c->skew_bytes || dst_bytes < bytes) return KVL_ESPACE;
        int rc = kvl_check_buffer(src, bytes + c->skew_bytes, 0);
        if (rc == KVL_OK) rc = kvl_check_buffer(dst, bytes, 0);
        if (rc != KVL_OK) return rc;
        const uint64_t n = bytes / 16, per_launch = (kMaxLanesPerLaunch / 256) * 256;
        const v4u *from = reinterpret_cast<const v4u *>(static_cast<const char *>(src) + c->skew_bytes);
        // (as the tiles of a contiguous table's descriptors)
        const uint32_t piece = kDefaultUnitBytes / 128;
        const LayerShape shape{bytes, (bytes + 127) / 128, ((bytes + 127) / 128 + piece - 1) / piece, piece, false, false};
        const uint32_t threads = halves ? kDefaultBlockThreads : hop_threads(shape, 128);
        const uint64_t run_bytes = halves ? 0 : tile_run_bytes(shape, 128);
        for (uint64_t first = 0; first < n; first += per_launch) {
            const uint64_t m = std::min<uint64_t>(per_launch, n - first);
            const dim3 grid((uint32_t)((m + threads - 1) / threads)), block(threads);
            const uint32_t order = tile_order(grid.x, 16ull * threads, run_bytes);
            v4u *to = static_cast<v4u *>(dst) + first;
            if (c->mode == KVL_CEILING_COPY)
                hipLaunchKernelGGL((kvl_ceiling_linear_kernel<0, kLinearNtLoad, kLinearStorePolicy>), grid, block, 0, s, from + first, to, m, order);
            else if (c->mode == KVL_CEILING_READ)
                hipLaunchKernelGGL((kvl_ceiling_linear_kernel<1, kLinearNtLoad, kLinearStorePolicy>), grid, block, 0, s, from + first, to, m, order);
            else
                hipLaunchKernelGGL((kvl_ceiling_linear_kernel<2, kLinearNtLoad, kLinearStorePolicy>), grid, block, 0, s, from + first, to, m, order);
            KVL_HIP(hipGetLastError());
        }
        return KVL_OK;
    }
    if (bytes % c->block_bytes || c->hop_blocks_log2 > 31) return KVL_EINVAL;
    const uint64_t n_blocks = bytes / c->block_bytes, hop_blocks = 1ull << c->hop_blocks_log2;
    if (n_blocks > hop_blocks || n_blocks > UINT32_MAX) return KVL_EINVAL;
    const uint64_t hop_bytes = hop_blocks * c->block_bytes, dense_bytes = bytes + c->skew_bytes;
    const bool gather = c->hopping_side == 0;
    if ((gather ? src_bytes : dst_bytes) < hop_bytes || (gather ? dst_bytes : src_bytes) < dense_bytes) return KVL_ESPACE;
    int rc = kvl_check_buffer(src, gather ? hop_bytes : dense_bytes, 0);
    if (rc == KVL_OK) rc = kvl_check_buffer(dst, gather ? dense_bytes : hop_bytes, 0);
    if (rc == KVL_OK && block_table) rc = kvl_check_buffer(block_table, n_blocks * 4, 0);
    if (rc != KVL_OK) return rc;
    CeilingArgs a{};
    a.dense = reinterpret_cast<uintptr_t>(gather ? dst : src);
    a.hopping = reinterpret_cast<uintptr_t>(gather ? const_cast<void *>(src) : dst);
    a.table = block_table;
    a.n_blocks = (uint32_t)n_blocks;
    a.hop_mask = (uint32_t)(hop_blocks - 1);
    a.mul = 0x9e3779b1u;                    // odd
    a.block_vecs = c->block_bytes / 16;
    a.skew_vecs = c->skew_bytes / 16;
    // a copy's tiles, lanes and order as the default kernels have them for a layer of such blocks
    const bool lines = c->skew_bytes == 0 && c->block_bytes % 128 == 0;
    const uint32_t row = lines ? 128 : 16, lead = lines ? 0 : 7;
    const LayerShape shape{bytes, bytes / row, n_blocks, c->block_bytes / row, false, false};
    const uint32_t threads = halves ? kDefaultBlockThreads : hop_threads(shape, row);
    // (the limit is that of tiles of 256 lanes, whatever their lanes are)
    const uint64_t most = n_blocks * ((a.block_vecs + 7 + 255) / 256);
    if (most > (1ull << 24) || most * 256 > kMaxLanesPerLaunch) return KVL_ERANGE;
    a.tiles_per_block = (a.block_vecs + lead + threads - 1) / threads;
    const TileDivisor d(a.tiles_per_block);
    a.magic = d.magic;
    a.shift = d.shift;
    const dim3 grid((uint32_t)(n_blocks * a.tiles_per_block)), block(threads);
    a.order = halves ? 0 : tile_order(grid.x, 16ull * threads, tile_run_bytes(shape, row));
#define KVL_CEIL(G, N, S)                                                                                              \
    do {                                                                                                            \
        if (c->mode == KVL_CEILING_COPY) hipLaunchKernelGGL((kvl_ceiling_pattern_kernel<0, G, N, S>), grid, block, 0, s, a); \
        else if (c->mode == KVL_CEILING_READ) hipLaunchKernelGGL((kvl_ceiling_pattern_kernel<1, G, N, S>), grid, block, 0, s, a); \
        else hipLaunchKernelGGL((kvl_ceiling_pattern_kernel<2, G, N, S>), grid, block, 0, s, a);                     \
    } while (0)
    // the cache policies of the default gather and scatter of such a layer
    const uint32_t v = default_tile_code(gather, lines, bytes, false);
    if (gather && v == kDefaultPackCode) KVL_CEIL(true, true, 2);
    else if (gather) KVL_CEIL(true, true, 0);
    else if (v == kNtUnpackCode) KVL_CEIL(false, true, 1);
    else if (v == kDefaultUnpackCode) KVL_CEIL(false, true, 3);
    else KVL_CEIL(false, false, 3);
#undef KVL_CEIL
    KVL_HIP(hipGetLastError());
    return KVL_OK;
}

const char *kvl_variant_name(uint32_t v) {
    static thread_local char name[64];
    if (v == 0) return "default";
    if (v > kvl::kNumVariants) return nullptr;
    v -= 1;
    static const char *modes[4] = {"wg/unit", "wave/unit", "tile x1", "tile x2"};
    static const char *sp[4] = {"", " st:nt", " st:sc1", " st:sc1+nt"};
    if (v & 256u)
        std::snprintf(name, sizeof name, "pipe%s%s%s", (v & 4u) ? " ld:nt" : "", sp[(v >> 3) & 3u],
                      (v & 64u) ? " noalign" : "");
    else if (v & 128u)
        std::snprintf(name, sizeof name, "flat%s%s", (v & 4u) ? " ld:nt" : "", sp[(v >> 3) & 3u]);
    else
        std::snprintf(name, sizeof name, "%s%s%s%s%s", modes[v & 3u], (v & 4u) ? " ld:nt" : "",
                      sp[(v >> 3) & 3u], (v & 32u) ? " deep" : "", (v & 64u) ? " noalign" : "");
    return name;
}

}  // extern "C"
