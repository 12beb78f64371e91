// What the library enqueues, and where, watched through a stand-in for the HIP runtime (fake_hip.h): launch shapes at
// sizes that no test machine holds, waits, events and captures.  Built and run by tests/test_host_launches.py, one
// check (named on the command line) to a process.
#include <cstdio>
#include <numeric>

#include "fake_hip.h"
#include "kvl_plan.hip"
#include "kvl_kernels.hip"

using fake::launches;
using namespace kvl;

#define REQUIRE(c) do { if (!(c)) { std::printf("%s failed at line %d\n", #c, __LINE__); return 1; } } while (0)

static bool is(const fake::Launch &l, const char *kernel) { return l.kernel.find(kernel) != std::string::npos; }
static uint64_t groups(const fake::Launch &l) { return (uint64_t)l.grid.x * l.grid.y * l.grid.z; }

// A plan made without kvl_plan, for sizes that only the launcher sees: `n` descriptors of one row each but the last, of `last`.
static kvl_plan_s made(uint64_t n, uint32_t last, uint32_t row, uint32_t planes = 1) {
    kvl_plan_s p;
    p.layout.n_layers = 1;
    p.layout.block_tokens = 1;
    p.layout.n_planes = planes;
    for (uint32_t q = 0; q < planes; ++q) p.layout.row_bytes[q] = row;
    p.layout.pool_blocks = p.dst_pool_blocks = n + last;
    p.flags = KVL_GATHER | KVL_SCATTER | KVL_NO_POINTER_CHECKS;
    p.hit_tokens = n - 1 + last;
    p.payload_bytes = p.hit_tokens * row * planes;
    p.blocks_touched = p.hit_tokens;
    p.max_unit_rows = last;
    p.vec16 = row % 16 == 0;
    p.units.resize(n);
    p.units.back() = kvl_unit_t{0, (uint32_t)(n - 1), last, 0};
    static kvl_unit_t somewhere;
    p.d_units = &somewhere;
    p.device = 0;
    p.tuning = kvl_tuning_t{kvl::kDefaultUnitBytes, kvl::kDefaultBlockThreads, 0, 0};
    return p;
}
static void *const kPlanes[KVL_MAX_PLANES] = {(void *)(1ull << 40), (void *)(1ull << 41), (void *)(1ull << 42), (void *)(1ull << 43)};

// kvl_plan over `blocks` whole blocks in reverse order (no two merge)
static kvl_plan_t *plan_of_blocks(uint32_t blocks, uint32_t bs, uint32_t row, uint32_t flags) {
    std::vector<int32_t> table(blocks);
    for (uint32_t i = 0; i < blocks; ++i) table[i] = (int32_t)(blocks - 1 - i);
    kvl_layout_t lay{};
    lay.n_layers = lay.n_planes = 1;
    lay.block_tokens = bs;
    lay.row_bytes[0] = row;
    lay.pool_blocks = blocks;
    kvl_request_t req{};
    req.hit_tokens = blocks * bs;
    req.n_blocks = blocks;
    req.block_table = table.data();
    kvl_plan_t *p = nullptr;
    return kvl_plan(&lay, &req, 1, flags | KVL_NO_POINTER_CHECKS, &p) == KVL_OK ? p : nullptr;
}
static kvl_plan_t *plan_of_single_tokens(uint32_t tokens, uint32_t row, uint32_t flags) { return plan_of_blocks(tokens, 1, row, flags); }

// Moves: a launch has the largest descriptor's tiles for every descriptor, so narrow workgroups are for descriptors that
// are alike.  Single rows with one long run among them keep the gather's shape, and its limit on tiles.
static int check_move_shapes() {
    for (uint64_t n : {1000000ull, 20000000ull}) {
        kvl_plan_s p = made(n, 113, 1152);
        p.paired = true;
        uintptr_t to[KVL_MAX_PLANES] = {1ull << 44};
        launches.clear();
        REQUIRE(kvl::launch_units(&p, true, 0, (uint32_t)n, 0, 1, kPlanes, to, nullptr) == KVL_OK);
        REQUIRE(launches.size() == 1 && launches[0].block.x == 256);
        // 113 rows of 72 vectors are 32 tiles; beyond 2^32 lanes the workgroups walk
        REQUIRE(groups(launches[0]) == std::min<uint64_t>(n * 32, kvl::kMaxLanesPerLaunch / 256));
        p.d_units = nullptr;
    }
    kvl_plan_s p = made(1000, 1, 1152);
    p.paired = true;
    for (kvl_unit_t &u : p.units) u.n_rows = 64;
    p.max_unit_rows = 64;
    p.hit_tokens = 64 * 1000;
    uintptr_t to[KVL_MAX_PLANES] = {1ull << 44};
    launches.clear();
    REQUIRE(kvl::launch_units(&p, true, 0, 1000, 0, 1, kPlanes, to, nullptr) == KVL_OK);
    REQUIRE(launches.size() == 1 && launches[0].block.x == 64 && launches[0].grid.x == 1000 * 72);
    p.layout.row_bytes[0] = 656;            // off the lines: as tile_threads says
    launches.clear();
    REQUIRE(kvl::launch_units(&p, true, 0, 1000, 0, 1, kPlanes, to, nullptr) == KVL_OK);
    REQUIRE(launches.size() == 1 && launches[0].block.x == kvl::tile_threads(64 * 41));
    p.d_units = nullptr;
    return 0;
}

// Full Blocks: the limit on tiles is that of the widest plane, though the tiles of all planes are numbered through.
static int check_full_block_planes() {
    kvl_plan_s p = made(20000000, 1, 2048, 4);
    p.layout.block_tokens = p.max_unit_rows = 64;           // ragged: blocks of one row, some of 64 (32 tiles a plane)
    launches.clear();
    REQUIRE(kvl::fullblock_launch(&p, true, 1ull << 44, 4 * 64 * 2048, 0, 0, 20000000, kPlanes, nullptr) == KVL_OK);
    REQUIRE(launches.size() == 2);
    for (const fake::Launch &l : launches) REQUIRE(is(l, "kvl_fullblock_kernel") && groups(l) * l.block.x <= kvl::kMaxLanesPerLaunch);
    launches.clear();
    REQUIRE(kvl::fullblock_launch(&p, true, 1ull << 44, 4 * 64 * 2048, 0, 5, 1005, kPlanes, nullptr) == KVL_OK);
    REQUIRE(launches.size() == 1 && groups(launches[0]) == 1000 * 128);
    for (uint32_t cap : {10u, UINT32_MAX}) {                // at most so many workgroups for each plane
        launches.clear();
        p.tuning.max_groups = cap;
        REQUIRE(kvl::fullblock_launch(&p, true, 1ull << 44, 4 * 64 * 2048, 0, 5, 1005, kPlanes, nullptr) == KVL_OK);
        REQUIRE(launches.size() == 1 && groups(launches[0]) == (cap == 10 ? 40 : 1000 * 128));
    }
    p.tuning.max_groups = 0;
    p.max_unit_rows = 64 * 64;
    REQUIRE(kvl::fullblock_launch(&p, true, 1ull << 44, 4 * 64 * 2048, 0, 0, 20000000, kPlanes, nullptr) == KVL_ERANGE);
    p.d_units = nullptr;
    return 0;
}

// A plan of `n` descriptors of `rows` rows each, as whole blocks have them.
static kvl_plan_s alike(uint64_t n, uint32_t rows, uint32_t row, uint32_t planes = 1) {
    kvl_plan_s p = made(n, rows, row, planes);
    p.layout.block_tokens = rows;
    for (uint64_t k = 0; k < n; ++k) p.units[k] = kvl_unit_t{(uint32_t)(k * rows), (uint32_t)(k * rows), rows, (uint32_t)k};
    p.hit_tokens = n * rows;
    p.payload_bytes = p.hit_tokens * row * planes;
    p.blocks_touched = n;
    return p;
}

// A plan of `n` descriptors of `rows` rows in planes of unlike rows; with a row map, made, if `map`.
static uint32_t g_map;
static kvl_plan_s unlike(uint64_t n, uint32_t rows, std::vector<uint32_t> row_bytes, bool map) {
    kvl_plan_s p = alike(n, rows, row_bytes[0], (uint32_t)row_bytes.size());
    p.payload_bytes = 0;
    for (size_t q = 0; q < row_bytes.size(); ++q) {
        p.layout.row_bytes[q] = row_bytes[q];
        p.payload_bytes += p.hit_tokens * row_bytes[q];
    }
    if (map) p.d_row_map = &g_map;
    return p;
}

// Odd rows: narrow workgroups are for launches that fill the machine.  Where a cap keeps them below that, they are wide.
static int check_capped_odd_rows() {
    const struct { uint32_t cap, pack, unpack; } shapes[] = {{0, 64, 128}, {64, 256, 256}, {1023, 256, 256}, {2047, 256, 256}, {2048, 128, 128}, {4095, 128, 128},
                                                             {4096, 64, 128}, {UINT32_MAX, 64, 128}};
    for (const auto &q : shapes)
        for (bool gather : {true, false}) {
            kvl_plan_s p = alike(30000, 64, 132);           // 254 MB, 529 vectors each
            p.tuning.max_groups = q.cap;
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44};
            launches.clear();
            REQUIRE(launch_units(&p, gather, 0, 30000, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
            const bool walks = q.cap && q.cap != UINT32_MAX;
            REQUIRE(launches.size() == 1 && is(launches[0], walks ? "kvl_any_walk_kernel" : "kvl_any_tile_kernel"));
            REQUIRE(launches[0].block.x == (gather ? q.pack : q.unpack) && (!walks || groups(launches[0]) == q.cap));
            launches.clear();                               // fewer tiles than the cap allows: as without one
            if (q.cap != 64) {
                REQUIRE(launch_units(&p, gather, 0, 100, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
                REQUIRE(launches[0].block.x == (gather ? 64 : 128) && is(launches[0], "kvl_any_tile_kernel"));
            }
            p.d_units = nullptr;
        }
    // too few for 256 lanes each: flat, as without lines to lay tiles on
    for (uint32_t cap : {1023u, 1024u}) {
        kvl_plan_s p = alike(5000, 4, 1026);                // 258 windows
        p.tuning.max_groups = cap;
        uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44};
        launches.clear();
        REQUIRE(launch_units(&p, true, 0, 5000, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
        for (const fake::Launch &l : launches) REQUIRE(is(l, cap < 1024 ? "kvl_any_flat_kernel" : "kvl_any_walk_kernel") && groups(l) <= cap);
        p.d_units = nullptr;
    }
    return 0;
}

// Odd rows in larger layers: policies, lines (last template argument: the source's) and lanes by the payload and the planes.
static int check_large_odd_layers() {
    const struct { uint32_t row, rows, planes, mib; const char *gather, *scatter; uint32_t gather_lanes, scatter_lanes; } shapes[] = {
        {132, 64, 1, 70, "tile_kernel<true, true, 2, true>", "tile_kernel<false, false, 3, false>", 64, 128},
        {132, 64, 1, 330, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 128},
        {132, 64, 1, 340, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 256},
        {132, 64, 1, 635, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 256},
        {132, 64, 1, 645, "tile_kernel<true, true, 1, true>", "tile_kernel<false, true, 1, false>", 256, 256},
        {132, 64, 2, 395, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 256},
        {132, 64, 2, 405, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, false>", 64, 256},
        {132, 64, 2, 565, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, false>", 64, 256},
        {132, 64, 2, 580, "tile_kernel<true, true, 1, true>", "tile_kernel<false, true, 1, false>", 256, 256},
        {333, 64, 2, 635, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 256},     // (not of whole lines)
        {1026, 64, 2, 500, "tile_kernel<true, true, 2, true>", "tile_kernel<false, true, 1, true>", 64, 256},    // 64 KiB and more
        {516, 64, 2, 600, "walk_kernel<true, true, 1, true>", "walk_kernel<false, true, 1, false>", 256, 256},
        {516, 64, 1, 700, "tile_kernel<true, true, 1, true>", "tile_kernel<false, true, 1, false>", 256, 256},
        {200, 16, 1, 70, "any_flat_kernel<true, true, 1>", "any_flat_kernel<false, true, 1>", 1024, 1024},           // 201, of whole lines
        {300, 8, 1, 60, "any_flat_kernel<true, true, 2>", "any_flat_kernel<false, false, 3>", 1024, 1024},          // 151 windows
        {300, 8, 1, 70, "any_flat_kernel<true, true, 1>", "any_flat_kernel<false, true, 1>", 1024, 1024},
        {120, 32, 1, 60, "any_tile_kernel<true, true, 2, true>", "any_tile_kernel<false, false, 3, false>", 64, 256},  // 241, of whole lines
        {120, 32, 1, 70, "any_flat_kernel<true, true, 1>", "any_flat_kernel<false, true, 1>", 1024, 1024},
        {124, 32, 1, 70, "any_flat_kernel<true, true, 1>", "any_flat_kernel<false, true, 1>", 1024, 1024},           // 249
        {70, 64, 1, 70, "any_tile_kernel<true, true, 2, true>", "any_tile_kernel<false, false, 3, false>", 64, 128}};  // 281
    for (const auto &q : shapes)
        for (bool gather : {true, false}) {
            const uint64_t n = ((uint64_t)q.mib << 20) / (q.rows * q.row * q.planes);
            kvl_plan_s p = alike(n, q.rows, q.row, q.planes);
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
            launches.clear();
            REQUIRE(launch_units(&p, gather, 0, (uint32_t)n, 0, q.planes, kPlanes, xfer, nullptr) == KVL_OK);
            const uint32_t lanes = gather ? q.gather_lanes : q.scatter_lanes;
            const bool tiled = !is(launches[0], "flat");
            if (launches.size() != 1 || !is(launches[0], gather ? q.gather : q.scatter) || launches[0].block.x != lanes ||
                (tiled && launches[0].grid.x != n * ((q.rows * q.row + 127 + 16 * lanes - 1) / (16 * lanes)))) {
                std::printf("%u by %u, %u planes, %u MiB: %s, %u workgroups of %u lanes\n", q.row, q.rows, q.planes, q.mib,
                            launches[0].kernel.c_str(), launches[0].grid.x, launches[0].block.x);
                return 1;
            }
            p.d_units = nullptr;
        }
    return 0;
}

// Full Blocks likewise: 64-lane workgroups for 132-byte rows by 64 without a cap, under one as wide as it takes.
static int check_capped_full_blocks() {
    const struct { uint32_t cap, block; } shapes[] = {{0, 64}, {64, 256}, {1024, 256}, {2048, 256}, {2049, 128}, {4096, 128}, {4097, 64}};
    for (const auto &q : shapes)
        for (bool to_pool : {true, false}) {
            kvl_plan_s p = alike(4000, 64, 132);
            p.tuning.max_groups = q.cap;
            launches.clear();
            REQUIRE(fullblock_launch(&p, to_pool, 1ull << 44, 64 * 132, 0, 0, 4000, kPlanes, nullptr) == KVL_OK);
            REQUIRE(launches.size() == 1 && launches[0].block.x == q.block && (!q.cap || groups(launches[0]) == q.cap));
            launches.clear();                               // fewer tiles than the cap allows
            REQUIRE(fullblock_launch(&p, to_pool, 1ull << 44, 64 * 132, 0, 0, 7, kPlanes, nullptr) == KVL_OK);
            REQUIRE(launches[0].block.x == 64 && groups(launches[0]) <= 64);
            p.d_units = nullptr;
        }
    return 0;
}

// Full Blocks: lanes of a tile by what idles over the planes, 128 in a single plane alone.
static int check_full_block_lanes() {
    const struct { uint32_t rows, a, b, lanes; } shapes[] = {{64, 1152, 0, 256}, {16, 336, 0, 128}, {100, 48, 0, 64}, {1, 2064, 0, 64}, {16, 1152, 128, 256},
                                                              {64, 144, 352, 256}, {32, 32, 656, 64}, {64, 132, 64, 64}, {16, 656, 128, 64}, {64, 1024, 128, 256}};
    for (const auto &q : shapes)
        for (bool to_pool : {true, false}) {
            kvl_plan_s p = q.b ? unlike(2000, q.rows, {q.a, q.b}, false) : alike(2000, q.rows, q.a);
            launches.clear();
            REQUIRE(fullblock_launch(&p, to_pool, 1ull << 44, (uint64_t)q.rows * (q.a + q.b), 0, 0, 2000, kPlanes, nullptr) == KVL_OK);
            if (launches.size() != 1 || launches[0].block.x != q.lanes) {
                std::printf("%u + %u by %u: %u lanes\n", q.a, q.b, q.rows, launches[0].block.x);
                return 1;
            }
            p.d_units = nullptr;
        }
    // odd rows out of the pool: on lines of the source, or written through where every block lies on lines of both sides
    const struct { uint32_t row, rows, off; bool lines; } odd[] = {{1026, 64, 0, true}, {200, 16, 0, true}, {1026, 64, 16, false}, {1026, 64, 1, false}, {333, 64, 0, false}};
    for (const auto &q : odd) {
        kvl_plan_s p = alike(2000, q.rows, q.row);
        launches.clear();
        REQUIRE(fullblock_launch(&p, false, (1ull << 44) + q.off, q.rows * q.row, 0, 0, 2000, kPlanes, nullptr) == KVL_OK);
        REQUIRE(is(launches[0], q.lines ? "<false, false, 1, true, 3, false>" : "<false, false, 1, true, 1, true>"));
        p.d_units = nullptr;
    }
    return 0;
}

// kvl_plan enqueues the making of the row map and waits for nothing that runs on the device, whoever answers for the
// plan's lifetime; the array of a plan dropped before its map was made comes back when the map's kernel has run.
static int check_caller_syncs() {
    for (uint32_t flags : {KVL_GATHER | KVL_CALLER_SYNCS, KVL_GATHER}) {
        kvl_release_cached_memory();
        launches.clear();
        fake::mallocs = fake::waited = 0;
        kvl_plan_t *p = plan_of_single_tokens(5000, 1152, flags);
        REQUIRE(p && p->d_row_map && launches.size() == 1 && is(launches[0], "kvl_row_map_kernel"));
        REQUIRE(fake::waited == 0 && fake::mallocs == 1);
        const void *first = p->d_units;
        kvl_plan_destroy(p);
        p = plan_of_single_tokens(5000, 1152, flags);
        REQUIRE(p && p->d_units != first && fake::mallocs == 2 && fake::waited == 0);
        for (const fake::Launch &l : launches) fake::finish(l.stream);
        kvl_plan_t *q = plan_of_single_tokens(5000, 1152, flags);
        REQUIRE(q && q->d_units == first && fake::mallocs == 2 && fake::waited == 0);
        kvl_plan_destroy(p);
        kvl_plan_destroy(q);
    }
    return 0;
}

static int pack(kvl_plan_t *p, hipStream_t s) {
    return kvl_pack_layer(p, kPlanes, (void *)(1ull << 44), p->payload_bytes, s);
}

// A captured launch uses the row map if it has been made by then, also where no launch came before it; one that is
// captured earlier goes without.  Neither does anything that a capture forbids, and no more does an eager launch beside one.
static int check_row_map_under_capture() {
    fake::Stream a, b;
    kvl_plan_t *p = plan_of_single_tokens(5000, 1152, KVL_GATHER);
    REQUIRE(p && p->d_row_map);
    fake::Stream *map_stream = launches.back().stream;
    fake::begin_capture(a);
    REQUIRE(pack(p, fake::handle(a)) == KVL_OK && is(launches.back(), "kvl_flat_kernel"));
    REQUIRE(pack(p, fake::handle(b)) == KVL_OK && is(launches.back(), "kvl_rows_kernel"));      // eager, beside it
    REQUIRE(fake::waits.size() == 1 && fake::waits[0].first == &b);
    fake::finish(map_stream);
    REQUIRE(pack(p, fake::handle(a)) == KVL_OK && is(launches.back(), "kvl_rows_kernel"));
    fake::end_capture(a);
    REQUIRE(!fake::capture_broken && fake::waits.size() == 1);
    kvl_plan_destroy(p);
    return 0;
}

// Every stream that launches before the map has been made waits for it; none does afterwards.
static int check_row_map_on_two_streams() {
    fake::Stream a, b;
    kvl_plan_t *p = plan_of_single_tokens(5000, 1152, KVL_GATHER);
    fake::Stream *map_stream = launches.back().stream;
    for (fake::Stream *s : {&a, &b, &fake::null_stream, &b}) {
        fake::waits.clear();
        REQUIRE(pack(p, s == &fake::null_stream ? nullptr : fake::handle(*s)) == KVL_OK);
        REQUIRE(is(launches.back(), "kvl_rows_kernel") && fake::waits.size() == 1 && fake::waits[0].first == s);
    }
    fake::finish(map_stream);
    fake::waits.clear();
    REQUIRE(pack(p, fake::handle(a)) == KVL_OK && pack(p, fake::handle(b)) == KVL_OK && fake::waits.empty());
    kvl_plan_destroy(p);
    return 0;
}

// Plans used on the default stream: nothing is put there but the caller's launches, and an array goes back when a launch
// made there after its plan's end has finished -- the first one, which alone carries an event for it.
static int check_default_stream() {
    auto plan = [] {
        kvl_plan_t *p = plan_of_single_tokens(5000, 1152, KVL_GATHER);
        fake::finish(launches.back().stream);          // (its map has been made)
        return p;
    };
    kvl_release_cached_memory();
    kvl_plan_t *a = plan(), *b = plan();
    fake::records.clear();
    fake::waited = fake::mallocs = 0;
    launches.clear();
    REQUIRE(pack(a, nullptr) == KVL_OK && pack(b, nullptr) == KVL_OK);
    REQUIRE(!launches[0].event && !launches[1].event);
    const void *mem_a = a->d_units;
    kvl_plan_destroy(a);
    const uint64_t queued = fake::null_stream.queued;
    kvl_plan_t *c = plan();                             // looks at what was retired
    REQUIRE(fake::null_stream.queued == queued && fake::mallocs == 1 && c->d_units != mem_a);
    fake::finish(&fake::null_stream);
    kvl_plan_t *d = plan();                             // a's launch has finished, but nothing there says so
    REQUIRE(fake::null_stream.queued == queued && fake::mallocs == 2);
    launches.clear();
    REQUIRE(pack(b, nullptr) == KVL_OK && pack(b, nullptr) == KVL_OK && pack(c, nullptr) == KVL_OK);
    REQUIRE(launches[0].event && !launches[1].event && !launches[2].event);
    kvl_plan_t *e = plan();
    REQUIRE(fake::mallocs == 3);                        // b's launch has not finished
    fake::null_stream.done = fake::null_stream.queued - 2;
    kvl_plan_t *f = plan();
    REQUIRE(fake::mallocs == 3 && f->d_units == mem_a);
    // a launch that is being made while a plan is destroyed does not speak for that plan's launches
    kvl_plan_destroy(c);
    DefaultStreamEvent *passes = nullptr;
    hipEvent_t ev = launch_event(b, nullptr, &passes);
    REQUIRE(ev && passes);
    (void)fake::launch(nullptr, dim3(1), dim3(64), nullptr, nullptr, ev);
    REQUIRE(pack(d, nullptr) == KVL_OK);
    kvl_plan_destroy(d);
    launched(passes, true);
    REQUIRE(g_retired.size() == 2 && g_waiting == 1 && !g_retired.back().passed);
    // nor one that failed
    ev = launch_event(b, nullptr, &passes);
    REQUIRE(ev && passes);
    launched(passes, false);
    REQUIRE(g_waiting == 1);
    REQUIRE(fake::waited == 0);
    for (const auto &r : fake::records) REQUIRE(r.first != &fake::null_stream);
    kvl_plan_destroy(b);
    kvl_plan_destroy(e);
    kvl_plan_destroy(f);
    kvl_release_cached_memory();
    REQUIRE(g_retired.empty() && g_waiting == 0 && fake::device_memory.empty());
    return 0;
}

// The arrays of a batch's two plans are kept for the next batch, whatever their row maps add to them.
static int check_cached_arrays() {
    for (uint32_t tokens : {5000u, 7000000u}) {
        kvl_release_cached_memory();
        fake::mallocs = fake::frees = 0;
        for (int batch = 0; batch < 2; ++batch) {
            kvl_plan_t *p[2];
            for (kvl_plan_t *&q : p) {
                q = plan_of_single_tokens(tokens, 1152, KVL_GATHER);
                REQUIRE(q && q->d_row_map);
                fake::finish(launches.back().stream);
            }
            for (kvl_plan_t *q : p) kvl_plan_destroy(q);
        }
        REQUIRE(fake::mallocs == 2 && fake::frees == 0);
    }
    // an engine that queues forty batches ahead, after plans of other sizes: nothing is freed, and nothing new allocated
    // for the next forty
    kvl_release_cached_memory();
    for (uint32_t tokens : {100u, 20000u, 40000u, 80000u, 160000u}) kvl_plan_destroy(plan_of_blocks(tokens, 64, 1152, KVL_GATHER));
    fake::frees = 0;
    for (int again = 0; again < 2; ++again) {
        fake::mallocs = 0;
        for (int batch = 0; batch < 40; ++batch) {
            kvl_plan_t *p = plan_of_blocks(10000, 64, 1152, KVL_GATHER);
            REQUIRE(p && !p->d_row_map && pack(p, nullptr) == KVL_OK);
            kvl_plan_destroy(p);
        }
        REQUIRE(fake::frees == 0 && fake::mallocs == (again ? 1 : 40));        // (the last one waits for a launch after it)
        fake::finish(&fake::null_stream);
    }
    kvl_release_cached_memory();
    fake::mallocs = fake::frees = 0;
    for (int batch = 0; batch < 2; ++batch) {               // 200 M rows in two million descriptors: no map of 800 MB beside 32
        kvl_plan_t *p = plan_of_blocks(2000000, 100, 16, KVL_GATHER);
        REQUIRE(p && !p->d_row_map);
        kvl_plan_destroy(p);
    }
    REQUIRE(fake::mallocs == 1 && fake::frees == 0);
    kvl_release_cached_memory();
    return 0;
}

// The bytes of the run of tiles that an XCD takes in the launch being made, from its `order` argument (0: in order).
static uint64_t g_run_bytes;
template <int ORDER> static void watch_order(const fake::Launch &l, void **args) {
    const uint32_t order = *(const uint32_t *)args[ORDER];
    g_run_bytes = order & 15u ? 16ull * l.block.x << (order & 15u) : 0;
}

// The reference stream of a shape has the cache policies, the tiles and the order of the tiled kernels on that shape, on both sides
// of every line.
static int check_ceiling_policies() {
    static uint32_t tile_orders[2];
    for (uint32_t row : {656u, 1152u, 384u})
        for (uint64_t payload : {2ull << 20, 8ull << 20, 16ull << 20, 100ull << 20, 200ull << 20, 400ull << 20, 5ull << 30})
            for (bool gather : {true, false}) {
                const uint32_t block = 64 * row, n = (uint32_t)(payload / block);
                kvl_plan_s p = made(n, 64, row);
                for (kvl_unit_t &u : p.units) u.n_rows = 64;
                p.hit_tokens = 64ull * n;
                p.payload_bytes = p.hit_tokens * row;
                uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44};
                launches.clear();
                fake::watch = [](const fake::Launch &l, void **args) {
                    const bool pattern = is(l, "kvl_ceiling_pattern_kernel");
                    tile_orders[pattern] = pattern ? ((const CeilingArgs *)args[0])->order : *(const uint32_t *)args[8];
                };
                REQUIRE(launch_units(&p, gather, 0, n, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
                const kvl_ceiling_t c{KVL_CEILING_COPY, block, gather ? 0u : 1u, row % 128 ? 16u : 0u, 18};
                REQUIRE(kvl_ceiling_kernel(&c, kPlanes[0], 1ull << 40, kPlanes[1], 1ull << 40, p.payload_bytes, nullptr, nullptr) == KVL_OK);
                fake::watch = nullptr;
                REQUIRE(launches[0].grid.x == launches[1].grid.x && launches[0].block.x == launches[1].block.x && tile_orders[0] == tile_orders[1]);
                // ..._tile_kernel<vectors per lane, nt loads, store policy>, kvl_ceiling_pattern_kernel<mode, gather, nt loads, store policy>
                const std::string &tile = launches[0].kernel, &ceiling = launches[1].kernel;
                const std::string policy = tile.substr(tile.find(", ") + 2, tile.find('>') - tile.find(", ") - 2);
                REQUIRE(ceiling.find(std::string("<0, ") + (gather ? "true, " : "false, ") + policy + ">") != std::string::npos);
                p.d_units = nullptr;
            }
    // a linear copy too; the halves of a copy alone go in order, in wide workgroups
    const kvl_ceiling_t modes[] = {{KVL_CEILING_COPY, 0, 0, 0, 0}, {KVL_CEILING_READ, 0, 0, 0, 0}, {KVL_CEILING_WRITE, 0, 0, 0, 0}, {KVL_CEILING_READ, 64 * 1152, 0, 0, 18}};
    for (const kvl_ceiling_t &c : modes) {
        launches.clear();
        const uint64_t bytes = c.block_bytes ? 50000ull * c.block_bytes : 4ull << 30;
        fake::watch = c.block_bytes ? (decltype(fake::watch))[](const fake::Launch &, void **args) { g_run_bytes = ((const CeilingArgs *)args[0])->order; } : watch_order<3>;
        REQUIRE(kvl_ceiling_kernel(&c, kPlanes[0], 1ull << 40, kPlanes[1], 1ull << 40, bytes, nullptr, nullptr) == KVL_OK);
        fake::watch = nullptr;
        const bool copy = c.mode == KVL_CEILING_COPY;
        REQUIRE(launches.size() == 1 && launches[0].block.x == (copy ? 64 : 256) && g_run_bytes == (copy ? 128 * 1024 : 0));
        REQUIRE(c.block_bytes || groups(launches[0]) * launches[0].block.x == bytes / 16);
    }
    return 0;
}

// Small layers: what the gather writes stays in the L2 caches where no event has to wait for it to be written back, from 2.75 MiB on.
// By tiles, by the row map (of single rows) and of odd rows.
static int check_small_gathers() {
    const struct { uint32_t row, rows; uint64_t least, most; } shapes[] = {{1152, 64, 2816u << 10, 10u << 20}, {656, 64, 2816u << 10, 12u << 20},
                                                                           {1152, 1, 2816u << 10, 10u << 20}, {656, 4, 2816u << 10, 12u << 20},
                                                                           {333, 64, 2816u << 10, 12u << 20}};
    for (const auto &q : shapes)
        for (uint64_t payload : {q.least - 80000, q.least + 80000, q.most - 80000, q.most + 80000}) {
            const uint32_t n = (uint32_t)(payload / (q.rows * q.row));
            const bool stays = payload > q.least && payload < q.most;
            fake::Stream own, captured;
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44};
            for (int where = 0; where < 4; ++where) {       // the default stream; the caller's, with an event and without; a capture
                kvl_plan_s p = alike(n, q.rows, q.row);
                p.d_row_map = &g_map;
                if (where == 2) p.flags |= KVL_CALLER_SYNCS;
                if (where == 3) fake::begin_capture(captured);
                launches.clear();
                REQUIRE(launch_units(&p, true, 0, n, 0, 1, kPlanes, xfer, where == 0 ? nullptr : fake::handle(where == 3 ? captured : own)) == KVL_OK);
                if (where == 3) fake::end_capture(captured);
                REQUIRE(launches.size() == 1 && launches[0].event == (where == 1));
                REQUIRE(is(launches[0], q.row == 333 ? "kvl_any_tile_kernel" : q.rows < 64 ? "kvl_rows_kernel" : "kvl_pack_quick_tile_kernel"));
                REQUIRE(is(launches[0], q.row == 333 || q.rows < 64 ? "<true, true, " : "<1, true, "));
                if (!is(launches[0], stays && where != 1 ? "true, 0" : "true, 2")) {
                    std::printf("%u by %u, %llu bytes, %d: %s\n", q.row, q.rows, (unsigned long long)payload, where, launches[0].kernel.c_str());
                    return 1;
                }
                p.d_units = nullptr;
            }
        }
    return 0;
}

// Odd rows: the order of the tiles by the layer's size alone, whatever its blocks and planes are; flat ones from 160 MiB.
static int check_odd_rows_order() {
    const struct { uint32_t row, rows, planes, mib, run_kib; } shapes[] = {
        {132, 64, 1, 40, 0}, {132, 64, 1, 50, 512}, {132, 64, 1, 250, 512}, {132, 64, 1, 260, 128}, {132, 64, 1, 300, 128}, {132, 64, 1, 390, 128},
        {132, 64, 1, 410, 128}, {132, 64, 1, 500, 128}, {132, 64, 1, 520, 512}, {72, 128, 1, 300, 128}, {260, 64, 1, 340, 128}, {132, 64, 2, 300, 128},
        {333, 64, 1, 11, 512}, {333, 64, 1, 13, 0}, {333, 64, 1, 300, 128}, {516, 64, 1, 300, 128}, {200, 16, 1, 150, 0}, {200, 16, 1, 170, 256},
        {200, 16, 1, 600, 256}};
    for (const auto &q : shapes)
        for (bool gather : {true, false}) {
            const uint64_t n = ((uint64_t)q.mib << 20) / (q.rows * q.row * q.planes);
            kvl_plan_s p = alike(n, q.rows, q.row, q.planes);
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
            launches.clear();
            fake::watch = q.row == 200 ? watch_order<9> : watch_order<8>;
            REQUIRE(launch_units(&p, gather, 0, (uint32_t)n, 0, q.planes, kPlanes, xfer, nullptr) == KVL_OK);
            fake::watch = nullptr;
            REQUIRE(launches.size() == 1 && is(launches[0], q.row == 200 ? "kvl_any_flat_kernel" : "kvl_any_tile_kernel"));
            if (g_run_bytes != q.run_kib * 1024) {
                std::printf("%u by %u, %u planes, %u MiB: runs of %llu KiB\n", q.row, q.rows, q.planes, q.mib, (unsigned long long)g_run_bytes >> 10);
                return 1;
            }
            p.d_units = nullptr;
        }
    return 0;
}

// An explicit variant is its form alone: tiles of the default width in order, also where the default takes them in runs.
static int check_variants_order() {
    const uint32_t n = 40000;
    for (uint32_t variant : {0u, 23u, 31u, 24u, 23u + 64u})
        for (bool gather : {true, false}) {
            kvl_plan_s p = alike(n, 64, 1152);              // 2.9 GB
            p.tuning.variant = variant;
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44};
            launches.clear();
            fake::watch = watch_order<8>;
            REQUIRE(launch_units(&p, gather, 0, n, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
            fake::watch = nullptr;
            REQUIRE(launches.size() == 1 && is(launches[0], "quick_tile_kernel") && launches[0].block.x == (variant ? 256 : 64));
            REQUIRE(g_run_bytes == (variant ? 0 : 128 * 1024));
            p.d_units = nullptr;
        }
    return 0;
}

// A tile's descriptor by multiplication is the quotient, for every workgroup number that a launch can have (around multiples of
// the divisor, at both ends).
static int check_tile_divisor() {
    std::vector<uint32_t> divisors = {2147483647u, 2147483646u, 1073741825u, 1073741824u, 1431655765u, 715827883u};
    for (uint32_t d = 1; d < 5000; ++d) divisors.push_back(d);
    for (uint32_t k = 12; k < 31; ++k)
        for (int e = -1; e <= 1; ++e) divisors.push_back((1u << k) + e);
    for (uint32_t d : divisors) {
        const TileDivisor t(d);
        const uint32_t last = 2147483647u / d;
        for (uint32_t q : {0u, 1u, 2u, 3u, last / 3, last / 2, last - (last > 0), last})
            for (int e = -1; e <= 1; ++e) {
                const int64_t b = (int64_t)q * d + e;
                if (b < 0 || b > 2147483647) continue;
                const uint32_t got = t.magic ? (uint32_t)(((uint64_t)b * t.magic) >> 32) >> t.shift : (uint32_t)b;
                REQUIRE(got == (uint32_t)b / d);
            }
    }
    return 0;
}

// Workgroups take every tile once, whatever their number, and of the whole rounds an XCD's workgroups (every eighth) take runs of
// neighbouring tiles in their order, every XCD as many.
static int check_tile_order() {
    std::vector<uint32_t> counts = {1, 7, 8, 15, 16, 17, 100003};
    for (uint32_t shift : {1u, 5u, 7u, 9u})
        for (uint32_t rounds : {1u, 2u, 8u, 9u})
            for (int e = -1; e <= 1; ++e) counts.push_back((rounds * 8u << shift) + e);
    for (uint32_t tiles : counts)
        for (uint64_t run : {0ull, 2048ull, 128ull << 10, 256ull << 10, 512ull << 10})
            for (uint32_t lanes : {64u, 128u, 256u, 1024u}) {
                const uint32_t order = tile_order(tiles, 16ull * lanes, run), whole = order & ~15u, length = 1u << (order & 15u);
                REQUIRE(whole <= tiles && (run || !order) && (!run || whole % (8 * length) == 0) && (!run || tiles - whole < 8 * length));
                REQUIRE(!run || 16ull * lanes * length == std::max<uint64_t>(run, 32ull * lanes));
                std::vector<uint32_t> by(tiles, UINT32_MAX);
                for (uint32_t b = 0; b < tiles; ++b) {
                    const uint32_t t = tile_number(b, order);
                    REQUIRE(t < tiles && by[t] == UINT32_MAX && (b < whole || t == b));
                    by[t] = b;
                }
                for (uint32_t t = 0; t < whole; ++t) REQUIRE(t % length == 0 || by[t] == by[t - 1] + 8);
                for (uint32_t t = 0; t + 8 * length <= whole; t += length)
                    for (uint32_t k = 1; k < 8; ++k) REQUIRE(t % (8 * length) != 0 || by[t] % 8 != by[t + k * length] % 8);
            }
    REQUIRE(tile_order(INT32_MAX, 1024, 128u << 10) / 8 % 128 == 0);
    // a pool row's place in its block by multiplication is the remainder, for any 32 bits
    for (uint32_t d : {1u, 2u, 3u, 7u, 16u, 24u, 64u, 100u, 4096u, 65535u, 1000003u, 2147483647u, 2147483648u, 4294967295u})
        for (uint32_t n : {0u, 1u, d - 1, d, d + 1, 2147483647u, 4294967295u / d * d - 1, 4294967295u / d * d, 4294967294u, 4294967295u})
            REQUIRE(remainder_by(n, d, UINT32_MAX / d) == n % d);
    return 0;
}

// Planes of unlike rows by the row map: beyond what the on-die cache holds the scatter looks its rows up through the scalar cache.
static int check_planes_by_rows() {
    const struct { uint32_t wide, narrow, rows, mib, mode; } shapes[] = {
        {512, 16, 256, 230, 1}, {512, 16, 256, 240, 2}, {512, 128, 8, 230, 1}, {512, 128, 8, 380, 2}, {656, 128, 1, 110, 1}, {656, 128, 1, 114, 2},
        {304, 80, 4, 200, 2}, {1152, 128, 1, 230, 1}, {1152, 128, 1, 240, 2}};
    for (const auto &q : shapes)
        for (bool gather : {true, false}) {
            const uint64_t n = ((uint64_t)q.mib << 20) / (q.rows * (q.wide + q.narrow));
            kvl_plan_s p = unlike(n, q.rows, {q.wide, q.narrow}, true);
            uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
            launches.clear();
            REQUIRE(launch_units(&p, gather, 0, (uint32_t)n, 0, 2, kPlanes, xfer, nullptr) == KVL_OK);
            const std::string mode = gather ? "<true, 2, 1>" : q.mode == 2 ? "<false, 3, 2>" : "<false, 3, 1>";
            if (launches.size() != 1 || !is(launches[0], ("kvl_planes_kernel" + mode).c_str())) {
                std::printf("%u + %u by %u, %u MiB: %s\n", q.wide, q.narrow, q.rows, q.mib, launches[0].kernel.c_str());
                return 1;
            }
            p.d_units = nullptr;
        }
    return 0;
}

// Planes of unlike rows by tiles: together, with which lanes, or apart.  `average` rows of a descriptor whose largest has `rows`.
static int check_planes_lanes() {
    const struct { bool move; uint32_t wide, narrow, rows; double average; uint32_t mib, together, lanes; } shapes[] = {
        {false, 1024, 128, 64, 64, 380, 1, 256}, {false, 1024, 128, 64, 64, 386, 0, 0}, {false, 256, 128, 100, 100, 100, 1, 256},
        {false, 256, 128, 100, 100, 200, 0, 0}, {false, 656, 336, 64, 64, 100, 1, 256}, {false, 656, 336, 64, 64, 300, 0, 0},
        {false, 1152, 640, 16, 16, 100, 1, 128}, {true, 1024, 128, 64, 64, 380, 1, 64}, {true, 512, 256, 8, 4.2, 45, 1, 128},
        {true, 512, 256, 8, 4.2, 64, 0, 0}, {true, 512, 1024, 4, 2.6, 300, 0, 0}, {true, 656, 336, 40, 25, 200, 1, 128},
        {true, 656, 336, 64, 64, 100, 1, 256}, {true, 656, 336, 64, 64, 350, 0, 0}, {true, 272, 144, 48, 48, 100, 1, 128}, {true, 160, 320, 16, 16, 100, 1, 128}, {true, 160, 320, 16, 16, 110, 0, 0}, {false, 1152, 640, 16, 16, 240, 1, 128},
        {true, 656, 128, 16, 10, 20, 1, 128}, {true, 256, 128, 16, 10.1, 40, 1, 128}, {true, 256, 128, 16, 10.1, 80, 0, 0}};
    for (const auto &q : shapes) {
        const uint64_t n = (uint64_t)(((uint64_t)q.mib << 20) / (q.average * (q.wide + q.narrow)));
        kvl_plan_s p = unlike(n, q.rows, {q.wide, q.narrow}, false);
        p.paired = q.move;
        p.hit_tokens = (uint64_t)(n * q.average);
        p.payload_bytes = p.hit_tokens * (q.wide + q.narrow);
        uintptr_t to[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
        for (bool gather : {true, false}) {
            if (!gather && (q.move || takes_row_map(&p, q.wide, false) || takes_row_map(&p, q.narrow, false))) continue;
            launches.clear();
            REQUIRE(launch_units(&p, gather, 0, (uint32_t)n, 0, 2, kPlanes, to, nullptr) == KVL_OK);
            const bool together = launches.size() == 1 && is(launches[0], "kvl_planes_kernel");
            if (together != (q.together != 0) || (together && launches[0].block.x != q.lanes) || (!together && launches.size() != 2)) {
                std::printf("%s of %u + %u by %u (%.1f), %u MiB: %zu launches, %u lanes\n", q.move ? "move" : gather ? "gather" : "scatter", q.wide,
                            q.narrow, q.rows, q.average, q.mib, launches.size(), launches[0].block.x);
                return 1;
            }
        }
        p.d_units = nullptr;
    }
    return 0;
}

// What the shared launch tells its workgroups covers every vector of its planes and descriptors once and no others, for ranges
// of both that begin anywhere.  (The workgroup's part follows kvl_planes_kernel.)
static uint64_t g_vectors[KVL_MAX_PLANES];
static uint32_t g_first_row;
static int check_planes_layout() {
    fake::watch = [](const fake::Launch &l, void **args) {
        if (!is(l, "kvl_planes_kernel")) return;
        const CopyArgs &a = *(const CopyArgs *)args[0];
        const PlanesArgs &pl = *(const PlanesArgs *)args[1];
        const bool rows = l.kernel.find(", 0>") == std::string::npos;
        g_first_row = pl.row_begin;
        for (uint32_t b = 0; b < l.grid.x; ++b) {
            uint32_t p = a.plane_begin;
            for (uint32_t q = 0; q + 1 < KVL_MAX_PLANES; ++q) p += b >= pl.group_end[q] ? 1u : 0u;
            const uint32_t group = b - (p > a.plane_begin ? pl.group_end[p - 1] : 0u), row = a.row_elems[p];
            const uintptr_t at = a.xfer[p] + (uint64_t)pl.row_begin * row * 16;
            const uint64_t span = rows ? (uint64_t)pl.n_rows * row : 64 * row;      // (64 rows to a descriptor)
            const uint64_t lead = rows ? (at >> 4) & 7 : pl.align_dst[p] ? 7 : 0;
            if (!rows && group / pl.per_unit[p] >= a.n_units) g_vectors[p] = ~0ull;
            const uint64_t tile = rows ? group : group % pl.per_unit[p];
            for (uint64_t k = tile * l.block.x; k < (tile + 1) * l.block.x; ++k) g_vectors[p] += k >= lead && k - lead < span ? 1 : 0;
        }
    };
    for (bool map : {false, true})
        for (uint32_t begin : {0u, 1u, 2u})
            for (uint32_t first : {0u, 7u, 99u}) {
                kvl_plan_s p = unlike(100, map ? 5 : 64, {1152, 1040, 1024, 2048}, map);
                uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, (1ull << 45) + 48, (1ull << 46) + 16, 1ull << 47};
                for (uint64_t &v : g_vectors) v = 0;
                launches.clear();
                REQUIRE(launch_units(&p, true, first, 100, begin, 4, kPlanes, xfer, nullptr) == KVL_OK);
                REQUIRE(launches.size() == 1 && is(launches[0], map ? "kvl_planes_kernel<true, 2, 1>" : "kvl_planes_kernel<true, 2, 0>"));
                REQUIRE(g_first_row == first * p.max_unit_rows);
                for (uint32_t q = 0; q < 4; ++q)
                    REQUIRE(g_vectors[q] == (q < begin ? 0 : (uint64_t)(100 - first) * p.max_unit_rows * (p.layout.row_bytes[q] / 16)));
                p.d_units = nullptr;
            }
    fake::watch = nullptr;
    // a map that is still being made is not waited for in a capture: the planes go apart, by their descriptors
    fake::Stream capturing, map_stream;
    map_stream.queued = 1;
    fake::Event made_by{&map_stream, 1};
    kvl_plan_s p = unlike(100, 5, {1152, 1040}, true);
    p.map_pending = true;
    p.map_event = reinterpret_cast<hipEvent_t>(&made_by);
    uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
    fake::begin_capture(capturing);
    launches.clear();
    REQUIRE(launch_units(&p, true, 0, 100, 0, 2, kPlanes, xfer, fake::handle(capturing)) == KVL_OK);
    REQUIRE(launches.size() == 2 && is(launches[0], "kvl_pack_quick_tile_kernel") && is(launches[1], "kvl_pack_quick_tile_kernel"));
    fake::finish(&map_stream);
    launches.clear();
    REQUIRE(launch_units(&p, true, 0, 100, 0, 2, kPlanes, xfer, fake::handle(capturing)) == KVL_OK);
    REQUIRE(launches.size() == 1 && is(launches[0], "kvl_planes_kernel<true, 2, 1>") && !fake::capture_broken && fake::waits.empty());
    fake::end_capture(capturing);
    p.d_units = nullptr;
    return 0;
}

// Row-map launches beyond 2^32 lanes: in parts that follow one another and leave out no row.
static uint64_t g_rows_covered;
static bool g_rows_right;
static int check_row_map_split() {
    const uint32_t n = 23000000, row = 3040, vectors = row / 16;        // 4.4e9 vectors
    kvl_plan_s p = made(n, 1, row);
    static uint32_t map;
    p.d_row_map = &map;
    REQUIRE(rows_ahead(&p, row, true));
    uintptr_t xfer[KVL_MAX_PLANES] = {(1ull << 44) + 112};              // the widest line-up
    launches.clear();
    g_rows_right = true;
    fake::watch = [](const fake::Launch &l, void **args) {
        const uint32_t begin = *(uint32_t *)args[2], vecs = *(uint32_t *)args[3];
        g_rows_right = g_rows_right && begin == g_rows_covered && vecs % (3040 / 16) == 0 && vecs + 7ull <= (uint64_t)l.grid.x * l.block.x &&
                       (uint64_t)l.grid.x * l.block.x <= kMaxLanesPerLaunch;
        g_rows_covered += vecs / (3040 / 16);
    };
    for (uint32_t first : {0u, 5u}) {
        p.units[first].xfer_row = first;
        g_rows_covered = first;
        launches.clear();
        REQUIRE(launch_units(&p, true, first, n, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
        REQUIRE(launches.size() == 2 && is(launches[0], "kvl_rows_kernel") && is(launches[1], "kvl_rows_kernel"));
        REQUIRE(g_rows_right && g_rows_covered == n);
    }
    REQUIRE((uint64_t)n * vectors > (1ull << 32));
    fake::watch = nullptr;
    p.d_units = nullptr;
    return 0;
}

// Planes of unlike rows: shapes on either side of the lines between the row map and the tiles (takes_row_map; one plane, or planes
// alike, go by check_tile_rules).
static int check_row_map_rule() {
    const struct { uint32_t row, bs, mb; bool gather, scatter; } shapes[] = {
        {1152, 1, 900, true, true}, {1152, 4, 900, true, true}, {2048, 1, 900, true, true}, {2048, 2, 900, false, false},
        {64, 64, 900, true, true}, {64, 128, 900, true, true}, {1152, 8, 900, true, true}, {64, 256, 900, false, false},
        {80, 256, 900, true, false}, {128, 50, 900, true, true}, {128, 100, 900, false, false}, {256, 100, 900, false, false},
        {192, 64, 900, true, true}, {272, 16, 900, true, true}, {144, 256, 900, true, false}, {1152, 64, 900, false, false},
        // scatters of layers about the size of the on-die cache
        {656, 64, 100, false, false}, {656, 64, 140, false, true}, {656, 100, 400, false, true}, {656, 64, 440, false, false},
        {272, 256, 300, false, true}, {1152, 64, 250, false, false}, {1152, 64, 300, false, true}, {512, 64, 300, false, true},
        {2048, 64, 560, false, true}, {2048, 64, 600, false, false}, {128, 64, 300, false, false}, {256, 256, 420, false, false},
        {384, 64, 540, false, false}};
    for (const auto &q : shapes) {
        const uint64_t n = ((uint64_t)q.mb << 20) / (q.bs * q.row);
        kvl_plan_s p = made(n, q.bs, q.row);
        p.layout.block_tokens = q.bs;
        p.hit_tokens = n * q.bs;
        p.payload_bytes = p.hit_tokens * q.row;
        if (takes_row_map(&p, q.row, true) != q.gather || takes_row_map(&p, q.row, false) != q.scatter) {
            std::printf("%u-byte rows by %u, %u MB: gather %d scatter %d\n", q.row, q.bs, q.mb, takes_row_map(&p, q.row, true), takes_row_map(&p, q.row, false));
            return 1;
        }
        p.d_units = nullptr;
    }
    return 0;
}

// Launches of one plane by the sizes: kernel (T tiles, R row map) and store policy, lanes, KiB of an XCD's run (0: in order), of the
// gather and of the scatter, on both sides of every limit; and of moves.
static int check_tile_rules() {
    struct Form { char kernel; int policy; uint32_t lanes, run_kib; };
    const struct { uint32_t row, rows, mib; Form gather, scatter; } hops[] = {
        // stores and lanes of small layers; plain loads of the scatter up to 112 MiB ('P')
        {1152, 64, 11, {'T', 2, 128, 512}, {'T', 3, 128, 512}}, {1152, 64, 13, {'T', 2, 128, 512}, {'T', 1, 128, 512}},
        {1152, 64, 21, {'T', 2, 128, 512}, {'T', 1, 128, 512}}, {1152, 64, 23, {'T', 2, 128, 512}, {'T', 3, 128, 512}},
        {1152, 1, 11, {'R', 2, 256, 512}, {'R', 3, 256, 512}}, {1152, 1, 13, {'R', 2, 256, 512}, {'R', 1, 256, 512}},
        {1152, 64, 27, {'T', 2, 128, 512}, {'T', 3, 128, 512}}, {1152, 64, 29, {'T', 2, 256, 512}, {'T', 3, 256, 512}},
        {656, 64, 13, {'T', 2, 128, 512}, {'P', 3, 128, 512}}, {656, 64, 111, {'T', 2, 256, 512}, {'P', 3, 256, 512}},
        {656, 64, 113, {'T', 2, 256, 512}, {'T', 3, 256, 512}},
        // tiles of 256 lanes badly filled: one wavefront in runs, 128 lanes in order
        {1152, 16, 29, {'T', 2, 64, 512}, {'T', 3, 64, 512}}, {1152, 16, 223, {'T', 2, 64, 512}, {'T', 3, 64, 512}},
        {1152, 16, 225, {'T', 2, 128, 0}, {'T', 3, 128, 0}}, {768, 40, 225, {'T', 2, 128, 0}, {'T', 3, 128, 0}},
        // small blocks of whole lines in order from 224 MiB (48 KiB are none); rows by the map likewise beyond the on-die cache
        {640, 64, 223, {'T', 2, 256, 512}, {'T', 3, 256, 512}}, {640, 64, 225, {'T', 2, 256, 0}, {'T', 3, 256, 0}},
        {768, 64, 225, {'T', 2, 256, 512}, {'T', 3, 256, 512}}, {1152, 1, 223, {'R', 2, 256, 512}, {'R', 3, 256, 512}},
        {1152, 1, 225, {'R', 2, 256, 0}, {'R', 3, 256, 0}}, {656, 4, 600, {'R', 2, 256, 512}, {'R', 1, 256, 512}},
        // the scatter by the row map in layers a little larger than the on-die cache
        {1152, 64, 243, {'T', 2, 256, 512}, {'T', 3, 256, 512}}, {1152, 64, 245, {'T', 2, 256, 512}, {'R', 3, 256, 512}},
        {1152, 64, 258, {'T', 2, 256, 512}, {'R', 3, 256, 0}}, {1152, 64, 479, {'T', 2, 256, 256}, {'R', 3, 256, 0}},
        {1152, 64, 481, {'T', 2, 256, 256}, {'T', 3, 256, 256}}, {656, 64, 243, {'T', 2, 256, 512}, {'T', 3, 256, 512}},
        {656, 64, 245, {'T', 2, 256, 512}, {'R', 1, 256, 512}}, {656, 64, 431, {'T', 2, 256, 256}, {'R', 1, 256, 512}},
        {656, 64, 433, {'T', 2, 256, 256}, {'T', 3, 256, 256}}, {384, 64, 300, {'T', 2, 256, 0}, {'T', 3, 256, 0}},
        {512, 64, 300, {'T', 2, 256, 0}, {'R', 3, 256, 0}}, {32, 500, 300, {'T', 2, 256, 256}, {'T', 3, 256, 256}},
        {48, 500, 300, {'T', 2, 256, 256}, {'R', 1, 256, 512}},
        // longer layers, shorter runs; short blocks off the lines longest
        {1152, 64, 287, {'T', 2, 256, 512}, {'R', 3, 256, 0}}, {1152, 64, 289, {'T', 2, 256, 256}, {'R', 3, 256, 0}},
        {1152, 64, 511, {'T', 2, 256, 256}, {'T', 3, 256, 256}}, {1152, 64, 513, {'T', 2, 64, 128}, {'T', 3, 64, 128}},
        {656, 64, 511, {'T', 2, 256, 256}, {'T', 3, 256, 256}}, {656, 64, 513, {'T', 2, 64, 128}, {'T', 3, 64, 128}},
        {656, 16, 511, {'T', 2, 64, 256}, {'T', 3, 64, 256}}, {656, 16, 513, {'T', 2, 64, 1024}, {'T', 3, 64, 1024}},
        {80, 256, 513, {'T', 2, 64, 128}, {'T', 3, 64, 128}}, {48, 256, 513, {'T', 2, 64, 1024}, {'T', 3, 64, 1024}},
        {768, 40, 513, {'T', 2, 64, 0}, {'T', 3, 64, 0}}, {512, 64, 2000, {'T', 2, 256, 0}, {'T', 3, 256, 0}},
        // descriptors of a few hundred vectors
        {1152, 4, 60, {'R', 2, 256, 512}, {'R', 3, 256, 512}}, {1152, 5, 60, {'T', 2, 64, 512}, {'T', 3, 64, 512}},
        {656, 14, 60, {'R', 2, 256, 512}, {'R', 1, 256, 512}}, {656, 15, 60, {'T', 2, 64, 512}, {'P', 3, 64, 512}},
        {272, 16, 60, {'R', 2, 256, 512}, {'R', 1, 256, 512}}};
    fake::watch = [](const fake::Launch &l, void **args) { is(l, "kvl_rows_kernel") ? watch_order<7>(l, args) : watch_order<8>(l, args); };
    uintptr_t xfer[KVL_MAX_PLANES] = {1ull << 44, 1ull << 45};
    for (const auto &q : hops)
        for (bool gather : {true, false})
            for (uint32_t planes : {1u, 2u}) {              // planes alike go as one does
                const Form &f = gather ? q.gather : q.scatter;
                const uint32_t n = (uint32_t)(((uint64_t)q.mib << 20) / (q.rows * q.row * planes));
                kvl_plan_s p = alike(n, q.rows, q.row, planes);
                p.d_row_map = &g_map;
                launches.clear();
                REQUIRE(launch_units(&p, gather, 0, n, 0, planes, kPlanes, xfer, nullptr) == KVL_OK);
                const std::string policy = std::to_string(f.policy), tile = gather ? "kvl_pack_quick_tile_kernel<1, " : "kvl_unpack_quick_tile_kernel<1, ";
                const std::string kernel = f.kernel == 'R' ? std::string("kvl_rows_kernel<") + (gather ? "true" : "false") + ", true, " + policy + ", "
                                                           : tile + (f.kernel == 'P' ? "false, " : "true, ") + policy + ">";
                if (launches.size() != 1 || !is(launches[0], kernel.c_str()) || launches[0].block.x != f.lanes || launches[0].grid.y != planes ||
                    g_run_bytes != f.run_kib * 1024) {
                    std::printf("%u by %u, %u MiB, %u planes, %s: %s, %u lanes, runs of %llu KiB\n", q.row, q.rows, q.mib, planes, gather ? "gather" : "scatter",
                                launches[0].kernel.c_str(), launches[0].block.x, (unsigned long long)g_run_bytes >> 10);
                    return 1;
                }
                p.d_units = nullptr;
            }
    const struct { uint32_t row, rows, mib, policy, lanes, run_kib; } moves[] = {
        {1152, 64, 22, 3, 64, 0}, {1152, 64, 24, 1, 64, 0}, {1152, 64, 75, 1, 64, 0}, {1152, 64, 77, 3, 64, 0}, {1152, 64, 95, 3, 64, 0},
        {1152, 64, 97, 3, 64, 256}, {1152, 64, 1023, 3, 64, 256}, {1152, 64, 1025, 3, 64, 256}, {656, 64, 22, 3, 256, 256}, {656, 64, 24, 1, 256, 256},
        {656, 64, 75, 1, 256, 256}, {656, 64, 77, 3, 256, 256}, {656, 64, 1025, 3, 256, 256}, {640, 64, 223, 3, 64, 256}, {640, 64, 225, 3, 64, 0},
        {640, 64, 1025, 3, 64, 0}, {656, 32, 300, 3, 128, 256}};
    for (const auto &q : moves) {
        const uint32_t n = (uint32_t)(((uint64_t)q.mib << 20) / (q.rows * q.row));
        kvl_plan_s p = alike(n, q.rows, q.row);
        p.paired = true;
        launches.clear();
        REQUIRE(launch_units(&p, true, 0, n, 0, 1, kPlanes, xfer, nullptr) == KVL_OK);
        const std::string kernel = "kvl_pack_quick_tile_kernel<1, true, " + std::to_string(q.policy) + ">";
        if (launches.size() != 1 || !is(launches[0], kernel.c_str()) || launches[0].block.x != q.lanes || g_run_bytes != q.run_kib * 1024) {
            std::printf("move %u by %u, %u MiB: %s, %u lanes, runs of %llu KiB\n", q.row, q.rows, q.mib, launches[0].kernel.c_str(), launches[0].block.x,
                        (unsigned long long)g_run_bytes >> 10);
            return 1;
        }
        p.d_units = nullptr;
    }
    // descriptors that are not alike: wide workgroups; a cap: a walk
    kvl_plan_s p = alike(20000, 64, 1152);
    p.max_unit_rows = 128;
    launches.clear();
    REQUIRE(launch_units(&p, true, 0, 20000, 0, 1, kPlanes, xfer, nullptr) == KVL_OK && is(launches[0], "quick_tile") && launches[0].block.x == 256);
    p.tuning.max_groups = 1000;
    fake::watch = nullptr;
    launches.clear();
    REQUIRE(launch_units(&p, true, 0, 20000, 0, 1, kPlanes, xfer, nullptr) == KVL_OK && is(launches[0], "kvl_tile_walk_kernel") && groups(launches[0]) == 1000);
    p.d_units = nullptr;
    return 0;
}

// Flat launches, of whole vectors and of odd rows: fewer than 2^31 lanes each (a descriptor is found by a multiplication that is
// exact up to there), the launches' descriptors following one another with none left out.
static const kvl_unit_t *g_next;
static bool g_flat_right;
static int check_flat_split() {
    fake::watch = [](const fake::Launch &l, void **args) {
        const kvl_unit_t *units = *(const kvl_unit_t **)args[0];
        const uint64_t n = *(uint32_t *)args[4], m = *(uint32_t *)args[5], lanes = (uint64_t)l.grid.x * l.block.x;
        g_flat_right = g_flat_right && units == g_next && n * m <= lanes && lanes < (1ull << 31) && *(uint32_t *)args[8] == l.block.x;
        g_next += n;
    };
    const struct { uint32_t n, row; bool move; const char *kernel; uint32_t launches; } shapes[] = {
        {17000000, 2048, false, "kvl_flat_kernel<", 2}, {17000000, 2048, true, "kvl_flat_kernel<", 2}, {14000000, 2535, false, "kvl_any_flat_kernel<", 2},
        {14000000, 2535, true, "kvl_any_flat_kernel<", 2}, {16000000, 2048, false, "kvl_flat_kernel<", 1}, {13000000, 2535, false, "kvl_any_flat_kernel<", 1},
        {100000, 16, true, "kvl_flat_kernel_short<", 1}, {100000, 33, false, "kvl_any_flat_kernel_short<", 1}};
    for (const auto &q : shapes) {
        kvl_plan_s p = made(q.n, 1, q.row);
        p.paired = q.move;
        uintptr_t to[KVL_MAX_PLANES] = {1ull << 44};
        for (uint32_t first : {0u, 5u}) {
            g_flat_right = true;
            g_next = p.d_units + first;
            launches.clear();
            REQUIRE(launch_units(&p, true, first, q.n, 0, 1, kPlanes, to, nullptr) == KVL_OK);
            REQUIRE(g_flat_right && g_next == p.d_units + q.n && launches.size() == q.launches);
            for (const fake::Launch &l : launches) REQUIRE(is(l, q.kernel));
        }
        p.d_units = nullptr;
    }
    fake::watch = nullptr;
    return 0;
}

// Full Blocks of planes alike: a plane's tiles to a row of the grid, every plane with its own pool and its own part of the blocks.
struct QuickArgs {
    uintptr_t pool[KVL_MAX_PLANES], blocks[KVL_MAX_PLANES];
    uint32_t fb_vecs, row, tiles, threads, tokens;
};
static QuickArgs g_quick;
static int check_full_blocks_alike() {
    const uint64_t base = 1ull << 44, offset = 3 * 4096;
    const struct { uint32_t row, rows, planes, off, lanes, tiles; } shapes[] = {{1152, 64, 1, 0, 256, 18}, {1152, 64, 1, 16, 256, 19}, {2048, 64, 2, 0, 256, 32},
                                                                                {336, 16, 1, 0, 128, 3}, {336, 100, 4, 0, 256, 9}, {80, 256, 3, 48, 256, 6}};
    for (const auto &q : shapes)
        for (bool to_pool : {true, false}) {
            kvl_plan_s p = alike(3000, q.rows, q.row, q.planes);
            const uint64_t pitch = 61ull * q.planes * q.rows * q.row;
            fake::watch = [](const fake::Launch &, void **args) {
                const TileMore &more = *(const TileMore *)args[11];
                g_quick.pool[0] = *(uintptr_t *)args[1];
                g_quick.blocks[0] = *(uintptr_t *)args[2];
                for (uint32_t k = 1; k < KVL_MAX_PLANES; ++k) {
                    g_quick.pool[k] = more.pool[k - 1];
                    g_quick.blocks[k] = more.xfer[k - 1];
                }
                g_quick.fb_vecs = *(uint32_t *)args[3];
                g_quick.row = *(uint32_t *)args[4];
                g_quick.tiles = *(uint32_t *)args[5];
                g_quick.threads = *(uint32_t *)args[7] & 0xffff;
                g_quick.tokens = *(uint32_t *)args[8];
                watch_order<10>(launches.back(), args);
            };
            launches.clear();
            REQUIRE(fullblock_launch(&p, to_pool, base + q.off, pitch, offset, 0, 3000, kPlanes, nullptr) == KVL_OK);
            fake::watch = nullptr;
            if (launches.size() != 1 || !is(launches[0], to_pool ? "kvl_fullblock_quick_kernel<true>" : "kvl_fullblock_quick_kernel<false>") ||
                launches[0].block.x != q.lanes || g_quick.threads != q.lanes || g_quick.tiles != q.tiles) {
                std::printf("%u by %u, %u planes: %s, %u lanes, %u tiles\n", q.row, q.rows, q.planes, launches[0].kernel.c_str(), launches[0].block.x, g_quick.tiles);
                return 1;
            }
            REQUIRE(launches[0].grid.x == 3000 * q.tiles && launches[0].grid.y == q.planes && g_run_bytes == 256 * 1024);
            REQUIRE(g_quick.fb_vecs == pitch / 16 && g_quick.row == q.row / 16 && g_quick.tokens == q.rows);
            for (uint32_t k = 0; k < q.planes; ++k)
                REQUIRE(g_quick.pool[k] == (uintptr_t)kPlanes[k] && g_quick.blocks[k] == base + q.off + offset + (uint64_t)k * q.rows * q.row);
            // in the general kernel: bytes off the vectors, the host link, a walk, a pitch beyond 32 bits
            for (int other = 0; other < 4; ++other) {
                launches.clear();
                p.tuning.max_groups = other == 2 ? 7 : 0;
                REQUIRE(fullblock_launch(&p, to_pool, base + (other == 0), other == 3 ? 1ull << 36 : pitch, offset, 0, 3000, kPlanes, nullptr, other == 1) == KVL_OK);
                REQUIRE(launches.size() == 1 && is(launches[0], "kvl_fullblock_kernel<"));
            }
            p.d_units = nullptr;
        }
    return 0;
}

int main(int argc, char **argv) {
    const std::map<std::string, int (*)()> checks = {
        {"move_shapes", check_move_shapes},
        {"full_block_planes", check_full_block_planes},
        {"capped_odd_rows", check_capped_odd_rows},
        {"capped_full_blocks", check_capped_full_blocks},
        {"large_odd_layers", check_large_odd_layers},
        {"full_block_lanes", check_full_block_lanes},
        {"caller_syncs", check_caller_syncs},
        {"row_map_under_capture", check_row_map_under_capture},
        {"row_map_on_two_streams", check_row_map_on_two_streams},
        {"default_stream", check_default_stream},
        {"cached_arrays", check_cached_arrays},
        {"ceiling_policies", check_ceiling_policies},
        {"planes_by_rows", check_planes_by_rows},
        {"planes_lanes", check_planes_lanes},
        {"planes_layout", check_planes_layout},
        {"row_map_split", check_row_map_split},
        {"tile_divisor", check_tile_divisor},
        {"row_map_rule", check_row_map_rule},
        {"tile_order", check_tile_order},
        {"small_gathers", check_small_gathers},
        {"odd_rows_order", check_odd_rows_order},
        {"variants_order", check_variants_order},
        {"tile_rules", check_tile_rules},
        {"flat_split", check_flat_split},
        {"full_blocks_alike", check_full_blocks_alike},
    };
    if (argc != 2 || !checks.count(argv[1])) {
        for (const auto &c : checks) std::printf("%s\n", c.first.c_str());
        return argc == 1 ? 0 : 2;
    }
    const int rc = checks.at(argv[1])();
    if (rc == 0) std::printf("ok\n");
    return rc;
}
