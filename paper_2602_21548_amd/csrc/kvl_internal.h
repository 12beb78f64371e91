// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "kvl.h"

struct kvl_plan_s {
    kvl_layout_t layout{};
    uint32_t flags = 0;
    bool paired = false;                         // made by kvl_plan_pair: xfer_row holds destination pool rows
    uint64_t dst_pool_blocks = 0;                // paired plans: blocks of the destination pool
    uint32_t n_req = 0;
    uint64_t hit_tokens = 0;                     // T
    uint64_t payload_bytes = 0;                  // all planes
    uint64_t plane_base[KVL_MAX_PLANES] = {};    // byte offset of each plane in the transfer buffer
    uint32_t max_unit_rows = 0;
    uint64_t blocks_touched = 0;                 // Full Blocks a buffer of this plan's ranges holds
    bool vec16 = false;                          // every row size is a multiple of 16 bytes
    std::vector<kvl_unit_t> units;               // host copy of the descriptors
    bool threads_chosen = false;                 // the caller named block_threads (else the launcher may halve the default)
    std::vector<uint32_t> block_first_unit;      // KVL_NO_MERGE plans, made on demand: first descriptor of each block
    std::vector<uint32_t> block_row_lo, block_row_hi;   // with it: rows [lo, hi) of each block that the plan moves
    kvl_unit_t *d_units = nullptr;               // device copy (absent for KVL_HOST_ONLY)
    size_t d_units_capacity = 0;                 // bytes of the cached buffer d_units lives in
    uint32_t *d_row_map = nullptr;               // behind the descriptors in the same buffer, where they are small
                                                 // (see kvl_rows_kernel): the pool row of every transfer row
    mutable hipEvent_t map_event = nullptr;      // with it: recorded after the kernel that makes the map,
    mutable bool map_pending = false;            // and whether that kernel may still have to run
    int device = -1;
    // One event per stream on which kernels that read d_units were enqueued (the caller's streams and
    // the lanes), taken along by every such launch: once all of them have fired no kernel reads the
    // buffer any more and it may be handed to another plan.  They go with the launches because a stream
    // of the caller's may be gone by the time the plan is destroyed; the default stream may not (see
    // DefaultStreamEvent).
    mutable std::vector<std::pair<hipStream_t, hipEvent_t>> stream_events;
    mutable bool null_stream_use = false;        // launched on the default stream (which carries no events)
    mutable bool untracked_use = false;          // a launch could not be followed (too many streams, a stream
                                                 // under capture, a failed record): wait for the device instead
    kvl_tuning_t tuning{};                       // resolved (no zero fields)
    // h2d path: one lane (a stream of the library's own) and one "lane done" event per staging slot
    std::vector<hipStream_t> lanes;
    std::vector<uint32_t> lane_cu_mask;          // empty: lanes may use every compute unit
    std::vector<hipEvent_t> ev_lane_done;
    hipEvent_t ev_entry = nullptr, ev_entry2 = nullptr;
};

namespace kvl {

void set_hip_error(hipError_t e);

#define KVL_HIP(expr)                                   \
    do {                                                \
        hipError_t kvl_e_ = (expr);                     \
        if (kvl_e_ != hipSuccess) {                     \
            ::kvl::set_hip_error(kvl_e_);               \
            return KVL_EHIP;                            \
        }                                               \
    } while (0)

constexpr uint32_t kDefaultUnitBytes = 128u << 10;
constexpr uint32_t kDefaultBlockThreads = 256;
constexpr uint32_t kHostSideGroups = 64;    // workgroups of a kernel whose far side is host memory (see kvl_tile_walk_kernel)
// Rows that are no multiple of 16 bytes (launch_any says why): the largest descriptor, in vectors, dealt out flat in a hop,
// and in moves and across the host link;
constexpr uint32_t kAnyFlatWindows = 160, kAnyFlatLinesWindows = 256, kAnyFlatPastWindows = 288;
// of a capped launch, the lanes from which narrow workgroups pay (half of what the machine holds);
constexpr uint64_t kCappedLanes = 1u << 18;
// up to which payload the on-die cache holds the layer from the gather's stores to the scatter's loads, beside two other
// layers' in turn (256 MB hold three of 85 MB), and up to which it pays to read each line out of it once.
// (Dealt out flat, 26 by 16, 73 MB, passing by / kept 81 / 85.)
constexpr uint64_t kCachedFlatBytes = 64u << 20, kCachedLayerBytes = 76u << 20, kReadOnceBytes = 640u << 20;
// The same for blocks of whole lines in several planes (gather, scatter), and up to which one the scatter's tiles are halved.
constexpr uint64_t kReadOnceManyBytes = 572u << 20, kScatterOnceManyBytes = 400u << 20, kHalveBytes = 336u << 20;
// Odd rows in several planes: descriptors from which the gather starts late (launch_any).
constexpr uint32_t kLateTileBytes = 32u << 10;
// Above the first of these payloads and up to the second (the third of rows off the lines) the gather's stores stay in the L2 caches,
// 32 MB in all, for the scatter, whose tiles the same XCDs take, instead of being written through; but where the launch carries an
// event, which waits for the caches to be written back (eager hops on a stream of the caller's, 4.6 MB of 1152-byte rows by 16, us,
// through / so: 8.50 / 9.05; 9.8 MB by 64 10.68 / 11.11).  Without one, hops of three layers with buffers of their own in turn in a HIP
// graph, through / so: 1152 by 16, 1.0 MB 3.91 / 3.99, 2.5 MB 4.29 / 4.45, 2.9 MB 4.88 / 4.76, 3.4 MB 5.42 / 5.13, 4.2 MB 5.53 / 5.22; 1152 by
// 64, 4.6 MB 5.73 / 5.26; 656 by 64, 2.8 MB 4.81 / 4.70, 6.6 MB 7.23 / 6.53; 333 by 64, 2.4 MB 4.79 / 4.84, 4.9 MB 6.54 / 5.98, 10.6 MB
// 9.69 / 9.65; 1152 by 1, 2.0 MB 4.13 / 4.23, 5.9 MB 6.45 / 5.68; eager ones on the default stream are bound by the host up to 6 MB, then 1152
// by 64, 7.5 MB 7.03 / 6.46, 9.7 MB 8.28 / 8.01.  Above they lose (1152 by 64, 10.9 MB 9.2 / 9.4, 16 MB 12.3 / 13.0; 1026 by 64, 22 MB
// 16.5 / 17.4), but with one transfer buffer for all layers, whose lines are then written again where they lie (656 by 64, 10.6 MB
// 8.91 / 8.10; 333 by 64, 10.8 MB 9.38 / 8.61).  Odd rows that are dealt out flat lose everywhere.
constexpr uint64_t kSmallFromBytes = 2816u << 10, kSmallBytes = 10u << 20, kSmallOffLinesBytes = 12u << 20;
inline bool gather_stays(bool lines, uint64_t payload, bool event) {
    return !event && payload > kSmallFromBytes && payload <= (lines ? kSmallBytes : kSmallOffLinesBytes);
}
// Between these two payloads the scatter's stores of whole lines are nt ones, which the L2 caches take up, instead of sc1+nt, which
// wait for the memory.  Hops of three layers with buffers of their own (with one buffer), us, sc1+nt / nt: 1152-byte rows by 64, 11.9 MB 9.7 /
// 9.3 (9.0 / 9.15), 13.9 MB 11.1 / 10.5 (10.3 / 10.3), 17 MB 12.7 / 12.1 (12.2 / 11.9), 19.6 MB 14.0 / 13.75 (13.6 / 13.3), 23.2 MB 16.0 /
// 16.0 (15.7 / 15.65), 28.9 MB 18.9 / 19.0; 1152 by 1, by the row map, 17 MB 13.2 / 12.4.  Rows off the lines lose, and planes of unlike
// rows (1024 and 128 by 64, 13.9 MB 12.3 / 12.6).
constexpr uint64_t kNtScatterFromBytes = 12u << 20, kNtScatterBytes = 22u << 20;
inline bool scatter_nt(bool lines, uint64_t payload) { return lines && payload > kNtScatterFromBytes && payload <= kNtScatterBytes; }
// Likewise a move's stores between these two.  Moves of three pairs of pools, us, sc1+nt / nt: 656-byte rows by 64, 14.5 MB 5.7 / 5.8, 20.7 MB
// 7.7 / 7.7, 25.8 MB 9.9 / 9.4, 33 MB 12.25 / 11.5, 46.5 MB 16.4 / 15.9, 77.5 MB 25.8 / 25.4, 134 MB 43.0 / 43.0, 207 MB 64.8 / 65.5; 1152 by 64
// 25.8 MB 9.9 / 9.3, 33 MB 12.1 / 11.4, 77.5 MB 25.2 / 24.8, 207 MB 62.9 / 63.4.  On a stream of the caller's and in a HIP graph 1152 by 64, 31 MB
// 11.1 / 10.7 and 11.5 / 11.0, 400 by 16, 49 MB 18.1 / 18.05 and 43 MB 16.4 / 16.1, but 656 by 64, 25 MB 9.4 / 9.6 and 9.3 / 9.4.
constexpr uint64_t kNtMoveBytes = 23u << 20, kNtMoveEndBytes = 76u << 20;
inline bool move_nt(uint64_t payload) { return payload > kNtMoveBytes && payload <= kNtMoveEndBytes; }
// Tiles of one plane, or of planes alike: their lanes and their order by the layer's size (hop_threads, tile_run_bytes).
constexpr uint64_t kNarrowBytes = 28u << 20, kWaveTileBytes = 512u << 20, kLongRunBytes = 288u << 20;
constexpr uint64_t kOrderBytes = 224u << 20, kOrderBlockBytes = 48u << 10, kVeryLongRunBlockBytes = 14u << 10, kMoveRunBytes = 96u << 20, kRowsRunBytes = 512u << 10, kOddOrderBytes = 48u << 20;
constexpr uint64_t kFlatOrderBytes = 160u << 20, kOnDieBytes = 256u << 20;
// Up to this payload planes of unlike rows share a launch (kvl_planes_kernel): beyond it a launch of their own is less than a
// hundredth of their time, and each plane better off in the form that suits it (hops apart / at once, 2048- and 656-byte
// rows by 16, 285 MB 176 / 177, 631 MB 412 / 412; 1024 and 128 by 24, 873 MB, 557 / 565; moves 512 and 528 by 128, 289 MB
// 91.0 / 89.9, 591 MB 181 / 183).
constexpr uint64_t kPlanesAtOnceBytes = 384u << 20;
// Up to these, by tiles, whatever lanes suit each plane (see launch_planes):
constexpr uint64_t kPlanesAlikeBytes = 104u << 20, kPlanesUnlikeBytes = 60u << 20;
// Beyond this one a scatter of theirs by the row map fetches its entries as kvl_rows_kernel does (see kvl_planes_kernel),
// or beyond kPlainReadBackBytes where rows of 16 to 63 vectors are off the lines.
constexpr uint64_t kPlanesCachedBytes = 236u << 20;
constexpr uint32_t kNumVariants = 512;       // explicit variants are 1 .. kNumVariants
bool valid_block_threads(uint32_t t);

// A launch may not have 2^32 or more lanes along x.  How many workgroups of `threads` lanes a
// launch over `work` workgroups' worth of tiles gets: all of them if that fits (and no cap is
// asked for), else as many as fit, each walking over several tiles.  *walk says which.
constexpr uint64_t kMaxLanesPerLaunch = (1ull << 32) - 1;
inline uint32_t launch_groups(uint64_t work, uint32_t threads, uint32_t cap, bool *walk) {
    uint64_t most = kMaxLanesPerLaunch / threads;
    if (cap && cap < most) most = cap;
    *walk = work > most;
    return (uint32_t)(*walk ? most : work);
}

// Rows that are no multiple of a 128-byte line: up to this payload the scatter reads the transfer buffer with plain
// loads (the on-die cache still has it), beyond it with non-temporal ones (64-token blocks of 656-byte rows, hop:
// 100 MB 63 us against 73; 140 MB 107 against 104; 1 GB 771 against 748; 576-byte rows, 1 GB, 745 against 702).
// The line lies where it does for callers that use one transfer buffer again and again, as an engine does: 64-token blocks of
// 656-byte rows, hop, plain loads / nt loads by the row map, us, one layer in a loop 96 MB 57.6 / 58.3, 117 MB 69.1 / 70.1; one
// transfer buffer and six pools in turn 57.7 / 58.5, 69.4 / 70.2; but three or four layers in turn, each with its own transfer
// buffer, 62.5 / 58.2 and 65.2 / 58.3, 78.7 / 70.2 and 79.1 / 70.3.
constexpr uint64_t kPlainReadBackBytes = 112u << 20;

// Tiles of a launch by descriptors: the default workgroup, halved where that leaves clearly fewer lanes without
// work (32-token blocks of 656-byte rows are 5.1 tiles of 256 lanes: 5.1 TB/s; 10.3 tiles of 128 lanes: 5.8).
inline uint32_t tile_threads(uint64_t unit_vecs) {
    auto idle = [&](uint64_t t) { return 1.0 - (double)unit_vecs / (double)((unit_vecs + t - 1) / t * t); };
    return idle(kDefaultBlockThreads) - idle(kDefaultBlockThreads / 2) > 0.07 ? kDefaultBlockThreads / 2 : kDefaultBlockThreads;
}

// What the order of a layer's tiles and their lanes are chosen by.
struct LayerShape {
    uint64_t payload, tokens, units, max_unit_rows;     // (as in kvl_plan_s)
    bool paired, capped;                                // a move; a cap on the workgroups
};
inline LayerShape shape_of(const kvl_plan_s *plan) {
    return {plan->payload_bytes, plan->hit_tokens, plan->units.size(), plan->max_unit_rows, plan->paired, plan->tuning.max_groups != 0};
}

// Bytes of the run of tiles that one XCD takes before the next run's turn (tile_number); 0: tile by tile.  One plan for several
// layers and one transfer buffer, us, tile by tile / runs of 128 / 256 / 512 KiB:
//  - hops: 656-byte rows by 64, 186 MB 120 / 107 / 105 / 105, 443 MB 286 / 267 / 264 / 266, 613 MB 393 / 378 / 378 / 381; 1152 by
//    64, 281 MB 156.6 / 154.3 / 154.3 / 153.6, 414 MB 235.7 / 235.9 / 233.4 / 235.0, 655 MB 384 / 380 / 383 / 387.
//  - small blocks of whole lines beyond the on-die cache lose: hops, 512 by 64, 175 MB 100.6 / 98.9 / 99.3 / 99.2, 344 MB 199 / 201 /
//    202 / 201, 2.6 GB 1681 / 1752 / 1727 / 1727; 1024 by 8, 334 MB 195 / 198 / 196 / 199, 2.6 GB 1670 / 1749 / 1719 / 1724; but 1024 by
//    48, 587 MB 346 / 344 / 347 / 351.
//  - short blocks off the lines in large layers like them longest: hops with buffers of their own, runs of 128 / 512 / 1024 / 2048 KiB, 400 by
//    24, 620 MB 418 / 409 / 405 / 406, 2.6 GB 1775 / 1754 / 1746 / 1749; 176 by 64, 620 MB 419 / 411 / 408 / 407, 5.2 GB 3479 / 3466 / 3455 /
//    3456; 272 by 64 (17 KB), 2.6 GB 1766 / 1782 / 1779 / 1785; 656 by 64, 1.0 GB 642 / 648 / 651 / 652.
//  - moves of three pairs of pools: 2048 + 2048 by 64, 62 MB 20.5 / 20.5 / 20.1 / 20.25, 114 MB 36.0 / 35.4 / 35.5 / 35.5, 413 MB 126.1 / 122.1 / 122.4 /
//    122.0, 2.8 GB 849 / 810 / 810 / 810; 512 by 256, 723 MB 219.3 / 211.7 / 211.9 / 212.0; 656 by 64, 114 MB 37.4 / 37.0 / 37.0 / 37.2, 723 MB 228.0 /
//    225.1 / 223.5 / 224.0, 2.8 GB 894 / 879 / 867 / 866; 1152 by 64 level up to 723 MB (218.8 / 218.0 / 217.8 / 217.3), 2.8 GB 844 / 852 / 843 / 839.
inline uint64_t tile_run_bytes(const LayerShape &s, uint32_t row_bytes) {
    const bool lines = row_bytes % 128 == 0;
    const double descriptor_bytes = (double)s.tokens * row_bytes / (double)s.units;
    const bool small_blocks = descriptor_bytes < (double)kOrderBlockBytes;
    if (lines && small_blocks && s.payload > kOrderBytes) return 0;
    if (s.paired) return !lines || s.payload > kMoveRunBytes ? 256u << 10 : 0;
    if (s.payload > kWaveTileBytes && descriptor_bytes < (double)kVeryLongRunBlockBytes) return 1u << 20;
    return s.payload <= kLongRunBytes ? 512u << 10 : s.payload <= kWaveTileBytes ? 256u << 10 : 128u << 10;
}

// Lanes of a hop's tiles: 128 in small layers, one wavefront where large layers go in runs, else 256 unless that leaves more of
// them without work.  Hops, us, 256 / 128 / 64 lanes: 1152-byte rows by 64, 12.6 MB 10.1 / 10.0 / 10.3; 656 by 64, 12.9 MB 12.0 / 11.7 /
// 12.6, 151 MB 86.2 / - / 88.8, 1.2 GB 728.5 / - / 727.8, contiguous 4.3 GB 2528 / - / 2513; 576 by 32, 112 MB 66.5 / - / 65.8, 563 MB
// 373 / - / 362; 80 by 256, 186 MB 109.7 / - / 107.8; tile by tile 768 by 40 (7.5 tiles of 256), 665 MB 446 / 412 / 408; 1152 by 20 (5.6),
// 655 MB 419 / 435 / 410; 1152 by 16 (4.5), 259 MB 147.7 / 147.3 / 151.1, 655 MB 413 / 408 / 406.  Descriptors that are not alike have
// a launch of the largest one's tiles, and wide workgroups are the fewest of those that find nothing to do.
inline uint32_t hop_threads(const LayerShape &s, uint32_t row_bytes) {
    const uint64_t largest = s.max_unit_rows * (row_bytes / 16);
    const bool alike = 2 * s.max_unit_rows * s.units <= 3 * s.tokens;
    const uint64_t vecs = largest + (row_bytes % 128 ? 7 : 0);         // with those before the first on its line
    if (!alike || s.capped || s.units * (vecs / 64 + 1) > INT32_MAX) return tile_threads(largest);
    if (s.payload <= kNarrowBytes) return 128;
    const bool in_runs = tile_run_bytes(s, row_bytes) != 0, large = s.payload > kWaveTileBytes;
    if (large && in_runs) return 64;
    const uint32_t narrow = in_runs || large ? 64 : 128;
    auto idle = [&](uint64_t t) { return 1.0 - (double)vecs / (double)((vecs + t - 1) / t * t); };
    return idle(kDefaultBlockThreads) - idle(narrow) > (in_runs ? 0.07 : large ? 0.03 : 0.05) ? narrow : kDefaultBlockThreads;
}

// Lanes of a move's workgroups: one wavefront where the descriptors are alike and begin on lines, else as tile_threads
// says.  A launch has the tiles of the largest descriptor for every one, and narrow workgroups make four times as many of
// those that find nothing to do.  300 MB, us with 64 / 128 / 256 lanes: 1152-byte rows by 64, all alike, 92.1 / 94.9 /
// 93.5; by 20 tokens at random (largest 1.4 times the average) 99.1 / 98.3 / 101.2; runs of 16-token blocks (1.9 times)
// 121.6 / 104.6 / 100.1; 256-byte rows by 4 in runs (2.6 times) 178.8 / 165.2 / 117.0; 656-byte rows by 16 and 64, alike,
// 99.5 / 105.8 / 99.8 and 97.7 / 95.3 / 95.1.
inline uint32_t move_threads(const kvl_plan_s *plan, uint32_t row_bytes) {
    const uint64_t largest = (uint64_t)plan->max_unit_rows * (row_bytes / 16);
    const bool alike = 2ull * plan->max_unit_rows * plan->units.size() <= 3 * plan->hit_tokens;
    return row_bytes % 128 == 0 && alike ? 64 : tile_threads(largest);
}

// Whether a launch over planes of unlike rows, one of this size among them, is laid out over the transfer rows (launch_planes) instead
// of over the descriptors' tiles, which have the size of the largest descriptor's.  (One plane, or planes alike, go as rows_ahead
// says.)  Measured on hops of one plane by tiles in order, 16 requests of
// uneven length, random tables, three layers each with its own plan and buffers in turn; us a hop, tiles / rows:
//  - tiles that would leave lanes idle, and descriptors of less than a workgroup: by rows both ways.  1 GB, 1152-byte rows
//    by 1 (72 vectors) 747 / 579, by 4 (1.1 tiles) 630 / 580, by 8 (2.25 tiles) 577 / 575, by 10 569 / 574; 2048 by 1 779 /
//    667, by 2 (one full tile) 660 / 666; 910 MB, 64 by 64 904 / 644, 128 by 50 629 / 588, 80 by 256 649 / 610.  The
//    scatter into rows that are no multiple of a line writes them in halves this way (a tile begins on a line) and wants a
//    worse filled tile before it gains: scatter alone, 656 by 32 (85 % busy) +2 %, 272 by 16 (53 %) -2 %.  Rows that do not
//    straddle lines lose in longer descriptors, where only the last tile is badly filled: 910 MB, 64 by 256 584 / 612, 256
//    by 100 586 / 605, 128 by 100 569 / 582 (1152 by 8, 576 vectors, 651 / 633; 64 by 128, 512, 618 / 624).
//  - the scatter of layers about the size of the on-die cache.  Rows that are no multiple of a line: 150 MB 656 by 64
//    101.7 / 92.5, 80 by 256 109.4 / 97.9, 303 MB 656 by 64 207 / 184, 272 by 256 199 / 182, 405 MB 265 / 253 and 269 /
//    260.  Rows of whole lines from 512 bytes: 303 MB 512 by 64 193 / 182, 2048 by 64 188 / 176 (with one plan for the
//    three layers 173.6 / 174.6), 425 MB 2048 by 64 257 / 245, 546 MB 325 / 316; shorter ones 303 MB 128 by 64 197 / 200,
//    425 MB 128 by 256 264 / 277, 256 by 256 259 / 272, 384 by 64 264 / 262, 546 MB 338 / 342.
inline bool takes_row_map(const kvl_plan_s *plan, uint32_t row_bytes, bool pack) {
    if (plan->paired || !plan->vec16 || plan->units.empty() || plan->max_unit_rows > 4096) return false;
    const bool lines = row_bytes % 128 == 0, straddle = !lines && 128 % row_bytes != 0;
    const uint64_t row = row_bytes / 16, largest = plan->max_unit_rows * row;
    const uint64_t t = tile_threads(largest), tiles = (largest + (lines ? 0 : 7) + t - 1) / t;
    const double average = (double)plan->hit_tokens * (double)row / (double)plan->units.size();
    const double busy = average / (double)(tiles * t);
    if (average < 200 || busy < (!straddle && largest >= 768 ? 0.66 : pack || lines ? 0.91 : 0.80)) return true;
    if (pack || row_bytes < 48) return false;
    const uint64_t mb = plan->payload_bytes >> 20;
    return lines ? row_bytes >= 512 && mb >= 256 && mb < 576 : plan->payload_bytes > kPlainReadBackBytes && mb < 432;
}

// The same for a launch of one plane, or of planes alike, whose tiles go to the XCDs in runs: by rows both ways where descriptors are
// small or tiles badly filled, and the scatter of layers a little larger than the on-die cache.
//  - hops with one plan and one transfer buffer for several layers, us, by rows, in runs as well / by tiles in runs: 272 by 16, 98 MB
//    60.4 / 59.9, 335 MB 207 / 225; 336 by 16, 351 MB 217 / 229; 1040 by 8, 362 MB 224 / 234; 656 by 16, 181 MB 106.8 / 104.8, 1.1 GB 779 /
//    766; 400 by 24, 189 MB 111.1 / 109.4; lines: 1152 by 4, 324 MB, in order, 191 / 194, 873 MB 567 / 570; 1024 by 8, 1.0 GB 661 / 640.
//  - the same with the scatter by rows, its gather by tiles: 656 by 64, 368 MB 219.2 / 215.0; 272 by 100, 335 MB 202.3 / 196.8; 1152 by 64,
//    324 MB 181.9 / 179.8.  Each layer with a plan and a transfer buffer of its own: 656 by 64, 368 MB 222 / 230; 272 by 100, 335 MB 204 /
//    216; 1040 by 64, 362 MB 215 / 220; 1152 by 64, 324 MB 188 / 192; but 656 by 64, 181 MB 103.6 / 102.5, 613 MB 394 / 377; 2048 + 2048 by
//    64, 521 MB 295.4 / 294.5.
inline bool rows_ahead(const kvl_plan_s *plan, uint32_t row_bytes, bool pack) {
    if (plan->paired || !plan->vec16 || plan->units.empty() || plan->max_unit_rows > 4096) return false;
    const bool lines = row_bytes % 128 == 0;
    const uint64_t row = row_bytes / 16, largest = plan->max_unit_rows * row + (lines ? 0 : 7);
    const uint64_t t = hop_threads(shape_of(plan), row_bytes), tiles = (largest + t - 1) / t;
    const double average = (double)plan->hit_tokens * (double)row / (double)plan->units.size();
    if (average < (lines ? 320 : 576) || average < 0.66 * (double)(tiles * t)) return true;
    const uint64_t mb = plan->payload_bytes >> 20;
    return !pack && row_bytes >= (lines ? 512 : 48) && mb >= 244 && mb < (lines ? 480 : 432);
}

// Cut [0, n_units) of one plane into chunks of at most chunk_bytes.
int make_chunks(const kvl_plan_t *plan, uint64_t chunk_bytes, std::vector<kvl_chunk_t> &out);

// Enqueue the copy of descriptors [unit_begin, unit_end) of planes
// [plane_begin, plane_end).  xfer_plane[p] is the address at which transfer row
// 0 of plane p would lie (it may point before a staging slot; only rows of the
// given descriptors are touched).
// far_host: the transfer side lies in host memory (the kernel crosses the host link).
int launch_units(const kvl_plan_t *plan, bool pack, uint32_t unit_begin, uint32_t unit_end,
                 uint32_t plane_begin, uint32_t plane_end,
                 void *const *pool_planes, const uintptr_t *xfer_plane, hipStream_t stream,
                 bool far_host = false);
// true if HIP knows ptr as pinned host memory (false when the plan skips pointer checks)
bool is_host_memory(const kvl_plan_t *plan, const void *ptr);

int upload_units(kvl_plan_t *plan);
// whether a launch on `stream` may read plan->d_row_map; orders the stream after the map's making if that is needed
bool row_map_ready(const kvl_plan_t *plan, hipStream_t stream);
// The event that a launch reading the plan's descriptors is to take with it on `stream` (null: none).  Where *passes is
// set, launched() is told afterwards whether the launch was made.
struct DefaultStreamEvent;
hipEvent_t launch_event(const kvl_plan_t *plan, hipStream_t stream, DefaultStreamEvent **passes);
void launched(DefaultStreamEvent *passes, bool ok);
void drop_stream_events(const kvl_plan_t *plan);
// lanes come from, and go back to, a small pool shared by all plans
hipStream_t take_pooled_lane(int device);
void return_lane(hipStream_t lane, int device);
// kvl_check_buffer unless the plan opted out
int check_buffer(const kvl_plan_t *plan, const void *ptr, uint64_t bytes, bool allow_host);
int check_pool(const kvl_plan_t *plan, const void *const *planes, uint64_t pool_blocks);
int ensure_lanes(kvl_plan_t *plan, size_t lanes);
int lanes_follow(kvl_plan_t *plan, size_t lanes, hipStream_t copy_s, hipStream_t kern_s);

int check_device(const kvl_plan_t *plan);
uint64_t layer_block_bytes(const kvl_plan_t *plan);
int check_fullblock_args(const kvl_plan_t *plan, bool to_pool, uint64_t blocks_bytes, uint32_t layer);
int fullblock_launch(const kvl_plan_t *plan, bool to_pool, uintptr_t base, uint64_t block_pitch,
                     uint64_t layer_off, uint32_t unit_begin, uint32_t unit_end,
                     void *const *pool_planes, hipStream_t stream, bool far_host = false);
// Enqueue the move of one layer between a buffer of Full Blocks and a paged pool.
int fullblock_layer(const kvl_plan_t *plan, bool to_pool, uintptr_t blocks, uint64_t blocks_bytes,
                    uint32_t layer, void *const *pool_planes, hipStream_t stream);


// Host-buffer paths (kvl_h2d.hip), shared with the layer-wise streaming loop.
int enqueue_h2d_layer(kvl_plan_t *plan, const std::vector<kvl_chunk_t> &chunks,
                      const void *host_xfer, void *dev_staging, uint64_t chunk_bytes, size_t lanes,
                      void *const *pool_planes, hipStream_t kern_s, hipEvent_t wait_before_scatter);
int check_h2d_args(const kvl_plan_t *plan, const void *host, const void *staging,
                   uint64_t staging_bytes, uint64_t chunk_bytes, size_t *slots);
int enqueue_zero_copy_layer(const kvl_plan_t *plan, const void *host_xfer, void *const *pool_planes,
                            hipStream_t kern_s, hipEvent_t wait_before_scatter);
int enqueue_d2h_pack_layer(kvl_plan_t *plan, const std::vector<kvl_chunk_t> &chunks,
                           const void *const *pool_planes, void *dev_staging, uint64_t chunk_bytes,
                           size_t lanes, void *host_xfer, hipEvent_t wait_first, hipStream_t collector);
int check_d2h_args(const kvl_plan_t *plan, const void *staging, uint64_t staging_bytes, uint64_t chunk_bytes,
                   const void *host, uint64_t host_capacity, size_t *slots);
int check_fullblock_staging(const kvl_plan_t *plan, const void *staging, uint64_t staging_bytes,
                            uint64_t chunk_bytes, size_t *slots);
int enqueue_h2d_fullblocks_layer(kvl_plan_t *plan, const void *full_blocks, uint32_t layer,
                                 void *dev_staging, uint64_t chunk_bytes, size_t lanes,
                                 void *const *pool_planes, hipStream_t kern_s, hipEvent_t wait_before_scatter);

}  // namespace kvl
