// Device code of the copy kernels (gfx950).  Included by kvl_kernels.hip only.
//
// The work is pure data movement (no arithmetic on the payload).  A copy
// descriptor names a span of token rows that is contiguous in the paged pool and
// in the transfer buffer, so each descriptor is a straight 16-byte-vector copy;
// what the block table fragments is only where each span starts.  The kernels
// therefore read a descriptor (wave-uniform, through the scalar cache), form two
// 64-bit addresses and either move one 16-byte vector per lane (the tiled form,
// the default) or loop over the span with several loads in flight per lane.
// Consecutive lanes touch consecutive 16-byte vectors, so every wavefront load
// or store covers 1 KiB of contiguous memory.
//
// kvl_tuning_t::variant is 0 for the default below, else 1 + code with
// code = mode | ntl << 2 | sp << 3 | deep << 5 | noalign << 6:
//   mode 0  one workgroup per descriptor, each lane loops over the span
//   mode 1  one wavefront per descriptor, each lane loops over the span
//   mode 2  tiled: a descriptor is cut into tiles of blockDim vectors and every
//           lane moves exactly one 16-byte vector
//   mode 3  tiled, two vectors per lane
//   ntl     non-temporal loads
//   sp      store cache policy: 0 plain, 1 nt, 2 sc1, 3 sc1 nt
//   deep    modes 0-1: 8 instead of 4 vectors in flight per lane
//   noalign modes 2-3: do not line tiles up with the destination's 128-byte lines
//           (they are lined up by default whenever the rows are not multiples of 128 bytes)
//   pipe    (code bit 8, with ntl, sp and noalign only) the tiled form on a fixed grid of resident
//           workgroups, each walking over its tiles with loads, stores and descriptor fetches
//           software-pipelined (see kvl_tile_pipe_kernel)
//   flat    (code bit 7, with ntl and sp only) no tiles: lane g of the launch takes vector
//           g mod m of descriptor g div m, m = vectors of the largest descriptor; for
//           descriptors far smaller than a workgroup (token-granular pools)
// All of them take their tiles in order (tile_number).
// The default is the tiled form, or the row-map form (kvl_rows_kernel, for plans that have a
// map) where rows_ahead says so (for planes of unlike rows takes_row_map); without a map,
// descriptors of less than half a workgroup go flat: on single-token blocks of 1152 bytes the tiled form in workgroups
// of 256 lanes leaves 72 % of them idle.
// Measured on MI355X (5.2 GB of 72 KiB blocks in random order), the tiled form
// with one vector per lane is the fastest: it leaves no
// dependency between a lane's memory operations and lets the hardware fill the
// memory system with resident wavefronts.  Its lanes (64 in large layers) and the order of its tiles are
// chosen by hop_threads, move_threads and tile_run_bytes.  Cache policies, measured with gather
// and scatter alternating as they do in use: the gather (random reads,
// sequential writes) runs best with non-temporal loads and sc1 stores; the
// scatter (sequential reads, random writes) with sc1+nt stores and non-temporal
// loads, plain ones where rows that are not multiples of 128 bytes make neighbouring
// wavefronts share source lines and the layer is small enough for the on-die cache
// still to hold them (kPlainReadBackBytes).  Together the policies are worth 5-15 % over plain
// loads and stores.  Layers of a few MB store otherwise: see gather_stays, scatter_nt and move_nt.  With rows that
// are not multiples of 128 bytes the tiles are
// also lined up with the destination's cache lines (worth 5-9 % on 656-byte rows).
#pragma once

#include "kvl_internal.h"

namespace kvl {

// default variant codes (see the list above) and the plain copy's policies
constexpr uint32_t kDefaultPackCode = 2u | 4u | (2u << 3);   // tile x1, nt loads, sc1 stores
constexpr uint32_t kSmallPackCode = 2u | 4u;                 // tile x1, nt loads, plain stores
constexpr uint32_t kDefaultUnpackCode = 2u | 4u | (3u << 3);    // tile x1, nt loads, sc1+nt stores
constexpr uint32_t kNtUnpackCode = 2u | 4u | (1u << 3);         // tile x1, nt loads, nt stores (see kNtScatterBytes)
constexpr uint32_t kDefaultUnpackCodeOddRows = 2u | (3u << 3);  // tile x1, plain loads, sc1+nt stores
// A move reads one pool and writes another, both in hops, and nobody reads the result at once: it writes past the caches,
// in workgroups as move_threads says.  64-token blocks, us, as the gather does it / this way: 1152-byte rows, 600 MB,
// 218 / 199 (206 with 256 lanes), 2 GB 667 / 616; 656-byte rows, 600 MB, 213 / 196, 3 GB 1142 / 1074.  Single-token
// blocks, flat: 1152 bytes, 600 MB, 267 -> 227 with 1024 lanes and nt stores, 656 bytes, 300 MB, 145 -> 109.
constexpr uint32_t kMoveCode = 2u | 4u | (3u << 3);             // tile x1, nt loads, sc1+nt stores
constexpr uint32_t kNtMoveCode = 2u | 4u | (1u << 3);           // tile x1, nt loads, nt stores (see kNtMoveBytes)
constexpr uint32_t kFlatMoveCode = 128u | 4u | (1u << 3);       // flat, nt loads, nt stores
constexpr uint32_t kFlatPackCode = 128u | 4u | (2u << 3);       // flat, nt loads, sc1 stores
constexpr uint32_t kFlatUnpackCode = 128u | 4u | (1u << 3);     // flat, nt loads, nt stores
// The tiled form's code for a plain gather or scatter; `lines`: every row begins on a 128-byte line; `event`: the launch carries one.
inline uint32_t default_tile_code(bool pack, bool lines, uint64_t payload, bool event) {
    if (pack) return gather_stays(lines, payload, event) ? kSmallPackCode : kDefaultPackCode;
    if (scatter_nt(lines, payload)) return kNtUnpackCode;
    return lines || payload > kPlainReadBackBytes ? kDefaultUnpackCode : kDefaultUnpackCodeOddRows;
}
constexpr bool kLinearNtLoad = true;
constexpr int kLinearStorePolicy = 2;

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
// Every buffer is device (or device-mapped) memory: say so, so that the
// compiler emits global_load / global_store rather than flat accesses.
typedef const v4u __attribute__((address_space(1))) *gsrc_t;
typedef v4u __attribute__((address_space(1))) *gdst_t;

struct CopyArgs {
    const kvl_unit_t *units;       // device descriptors
    uint32_t unit_begin;           // first descriptor of this launch
    uint32_t n_units;              // descriptors in this launch
    uint32_t plane_begin;          // blockIdx.y + plane_begin is the plane
    uint32_t row_elems[KVL_MAX_PLANES];  // row size in 16-byte vectors (vector kernels) or bytes
    uintptr_t pool[KVL_MAX_PLANES];      // plane base of the paged pool
    uintptr_t xfer[KVL_MAX_PLANES];      // address of transfer row 0 of the plane
};


template <bool NT>
__device__ __forceinline__ v4u load16(gsrc_t p) {
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}

// Store with a cache policy.  The compiler only offers the non-temporal hint;
// the system-scope write-through forms (sc1) are written out as instructions.
// A store needs no wait: nothing here reads what it wrote.  The s_nop after a written-out
// store covers the one hazard the compiler cannot see through the asm: a vector-ALU write to the
// store's data registers in the next two issue slots (it handles that itself for stores it
// emits; in a loop the next instruction may well be such a write).
template <int SP>
__device__ __forceinline__ void store16(gdst_t p, v4u v) {
    if (SP == 0) *p = v;
    else if (SP == 1) __builtin_nontemporal_store(v, p);
    else if (SP == 2) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
    else asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

// `lanes` threads copy n 16-byte vectors; this thread is `lane`.  U loads are
// issued before the first store so that U KiB per wavefront are in flight.
template <int U, bool NTL, int SP>
__device__ __forceinline__ void copy_span(gsrc_t __restrict__ src, gdst_t __restrict__ dst,
                                          uint32_t n, uint32_t lane, uint32_t lanes) {
    // n is below 2^32: a descriptor never spans more than 1 GiB
    const uint32_t step = lanes * U;
    const uint32_t last = lanes * (U - 1);
    uint32_t i = lane;
    // no division: a lane takes a full step while its last vector is in range
    for (; (uint64_t)i + last < n; i += step) {
        v4u v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = load16<NTL>(src + i + k * lanes);
#pragma unroll
        for (int k = 0; k < U; ++k) store16<SP>(dst + i + k * lanes, v[k]);
    }
    // ragged tail: this lane has at most U-1 vectors left
    v4u v[U];
#pragma unroll
    for (int k = 0; k < U - 1; ++k) {
        const uint64_t j = (uint64_t)i + (uint64_t)k * lanes;
        if (j < n) v[k] = load16<NTL>(src + j);
    }
#pragma unroll
    for (int k = 0; k < U - 1; ++k) {
        const uint64_t j = (uint64_t)i + (uint64_t)k * lanes;
        if (j < n) store16<SP>(dst + j, v[k]);
    }
}

template <bool PACK, bool WAVE, int U, bool NTL, int SP>
__device__ __forceinline__ void units_body(const CopyArgs &a) {
    uint32_t u_idx, lane, lanes;
    if (WAVE) {
        const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        u_idx = blockIdx.x * (blockDim.x >> 6) + wave;
        lane = threadIdx.x & 63u;
        lanes = 64;
    } else {
        u_idx = blockIdx.x;
        lane = threadIdx.x;
        lanes = blockDim.x;
    }
    if (u_idx >= a.n_units) return;
    const kvl_unit_t u = a.units[a.unit_begin + u_idx];
    const uint32_t p = a.plane_begin + blockIdx.y;
    const uint64_t row = a.row_elems[p];
    const uintptr_t pool = a.pool[p] + (uint64_t)u.pool_row * row * 16u;
    const uintptr_t xfer = a.xfer[p] + (uint64_t)u.xfer_row * row * 16u;
    const uint32_t n = u.n_rows * (uint32_t)row;
    if (PACK) copy_span<U, NTL, SP>((gsrc_t)pool, (gdst_t)xfer, n, lane, lanes);
    else copy_span<U, NTL, SP>((gsrc_t)xfer, (gdst_t)pool, n, lane, lanes);
}

// gather: paged pool -> transfer buffer
template <bool WAVE, int U, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_pack_kernel(const CopyArgs a) {
    units_body<true, WAVE, U, NTL, SP>(a);
}

// scatter: transfer buffer -> paged pool
template <bool WAVE, int U, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_unpack_kernel(const CopyArgs a) {
    units_body<false, WAVE, U, NTL, SP>(a);
}

// One descriptor in one scalar load (field by field the compiler fetches them one after the other, each as late as it can).
typedef const v4u __attribute__((address_space(4), aligned(4))) *cunit_vec_t;
__device__ __forceinline__ kvl_unit_t fetch_unit(const kvl_unit_t *units, uint32_t i) {
    const v4u d = *((cunit_vec_t)(uintptr_t)units + i);
    return kvl_unit_t{d.x, d.y, d.z, d.w};
}

// The tile that workgroup b takes.  Workgroups go round the eight XCDs, each with an L2 of its own, so taken in order the tiles of
// a block are dealt to all of them: a line that two tiles share is read by two XCDs, and every XCD works on every page.  Here an
// XCD takes runs of 2^shift tiles one after the other (how long: tile_run_bytes, launch_any), the runs going round the XCDs, from one round to
// the next by one place on; the tiles behind the last whole round keep their order.  `order` is the number of tiles in whole
// rounds, a multiple of 16, with the shift in its low bits; 0 leaves the order as it is.  Hops, us, in order / in runs: 1152-byte
// rows by 64, 149 MB 84.9 / 82.8, contiguous 2.7 GB 1580 / 1522; 656 by 64, 186 MB 110.6 / 104.7, 11 GB 6913 / 6710, contiguous
// 4.3 GB 2849 / 2513; 2048 + 2048 by 64, 10 GB 6080 / 5943.  Runs of 16 to 64 KB are slower than any order (73,728-byte blocks,
// 4 GB: 2 tiles 2726, 4 2661, 16 2461, 32 2425, 64 2408, 256 2459; in order 2435).
__host__ __device__ __forceinline__ uint32_t tile_number(uint32_t b, uint32_t order) {
    if (b >= (order & ~15u)) return b;
    const uint32_t shift = order & 15u, i = b >> 3, round = i >> shift;
    return (((round << 3) | ((b + round) & 7u)) << shift) | (i & ((1u << shift) - 1u));
}

// A tile of a descriptor: `threads` lanes move VPT vectors each.
template <bool PACK, int VPT, bool NTL, int SP>
__device__ __forceinline__ void tile_span(const kvl_unit_t u, uintptr_t pool_base, uintptr_t xfer_base, uint32_t row, uint32_t tile,
                                          uint32_t threads, uint32_t align_dst) {
    const uint32_t n = u.n_rows * row;
    const uintptr_t pool = pool_base + (uint64_t)u.pool_row * row * 16u;
    const uintptr_t xfer = xfer_base + (uint64_t)u.xfer_row * row * 16u;
    gsrc_t src = (gsrc_t)(PACK ? pool : xfer);
    gdst_t dst = (gdst_t)(PACK ? xfer : pool);
    // With rows that are not multiples of 128 bytes a span starts anywhere in a
    // cache line.  Tiles are then laid from the 128-byte boundary below the
    // span's first destination byte, so that every wavefront's store covers
    // whole lines (its load may straddle them, which costs far less): the first
    // `lead` lanes of the first tile idle.
    const uint32_t lead = align_dst ? ((uint32_t)((PACK ? xfer : pool) >> 4) & 7u) : 0u;
    const uint32_t first = tile * (threads * VPT);
    if (first >= n + lead) return;      // this tile lies beyond the descriptor's end
    v4u v[VPT];
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const uint32_t pos = first + k * threads + threadIdx.x;
        if (pos >= lead && pos - lead < n) v[k] = load16<NTL>(src + (pos - lead));
    }
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
        const uint32_t pos = first + k * threads + threadIdx.x;
        if (pos >= lead && pos - lead < n) store16<SP>(dst + (pos - lead), v[k]);
    }
}

// Tiled form: the grid is (descriptors x tiles_per_unit, planes); a workgroup
// takes tile `t` of its descriptor and each lane moves VPT vectors.  With one
// vector per lane there is no loop and no dependency between a lane's memory
// operations: the hardware keeps the memory system busy by the sheer number of
// resident wavefronts rather than by unrolling.
//
// A wavefront lives for one load and one store, so what it waits for before them counts: the descriptor is found without
// a division (`magic` and the shift in `how`, see TileDivisor), fetched in one load, and the arguments are scalars, which the
// hardware puts into registers before the wavefront starts (-amdgpu-kernarg-preload-count).  Hops, 1152-byte rows by 64, us,
// four scalar loads one after the other / so: 11 MB 9.9 / 9.3, 22 MB 16.3 / 15.7, 80 MB 47.8 / 46.9.
struct TileMore {                       // planes after the first of a launch
    uintptr_t pool[KVL_MAX_PLANES - 1], xfer[KVL_MAX_PLANES - 1];
};
#define KVL_TILE_PARAMS                                                                                            \
    const kvl_unit_t *units, uintptr_t pool, uintptr_t xfer, uint32_t row, uint32_t tiles_per_unit, uint32_t magic, \
        uint32_t how, uint32_t threads, uint32_t order

template <bool PACK, int VPT, bool NTL, int SP>
__device__ __forceinline__ void tile_group(KVL_TILE_PARAMS) {
    const uint32_t b = tile_number(blockIdx.x, order);
    const uint32_t u_idx = magic ? (uint32_t)(((uint64_t)b * magic) >> 32) >> (how >> 1) : b;
    tile_span<PACK, VPT, NTL, SP>(fetch_unit(units, u_idx), pool, xfer, row, b - u_idx * tiles_per_unit, threads, how & 1u);
}

template <int VPT, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_pack_quick_tile_kernel(KVL_TILE_PARAMS, const TileMore more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    tile_group<true, VPT, NTL, SP>(units, pool, xfer, row, tiles_per_unit, magic, how, threads, order);
}

template <int VPT, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_unpack_quick_tile_kernel(KVL_TILE_PARAMS, const TileMore more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    tile_group<false, VPT, NTL, SP>(units, pool, xfer, row, tiles_per_unit, magic, how, threads, order);
}

// Thin form of the tiled kernels: a fixed, small number of workgroups, each walking over
// the tiles gridDim.x apart.  For buffers on the far side of the host link: a few hundred
// wavefronts keep the link full (its rate times its latency is about 100 KB in flight),
// so there is no reason to fill every compute unit with wavefronts that wait for it, and
// kernels of other streams keep the machine.  The trip count is fixed at launch.
template <bool PACK, int VPT, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_tile_walk_kernel(const CopyArgs a, uint32_t tiles_per_unit,
                                                             uint32_t align_dst, uint32_t n_tiles) {
    const uint32_t p = a.plane_begin + blockIdx.y;
    for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        // (with the descriptor in one load a streamed load of eight layers takes 15.01 ms, so 14.87)
        const uint32_t u_idx = t / tiles_per_unit;
        tile_span<PACK, VPT, NTL, SP>(a.units[a.unit_begin + u_idx], a.pool[p], a.xfer[p], a.row_elems[p], t - u_idx * tiles_per_unit,
                                      blockDim.x, align_dst);
    }
}

// Pipelined form of the tiled kernels: a fixed grid that fills the machine once (every
// workgroup resident), each workgroup walking over the tiles gridDim.x apart with its work
// software-pipelined three deep -- while the vectors of tile i are on their way, the loads of
// tile i+1 have been issued and the descriptor of tile i+2 is being fetched.  One-shot
// workgroups (the tiled form above) start with a dependent chain, descriptor fetch then data
// load, during which their wavefronts hold a slot but have nothing in flight; on workloads of
// many small descriptors the memory system then runs below saturation (its request queues
// hardly ever push back) although every wavefront slot is taken.  Here a wavefront always has
// one or two loads outstanding and the descriptor latency is hidden behind them.  The tiles a
// workgroup visits and their order over the machine are those of the tiled form, so the
// access stream the memory sees is the same.  The trip count is fixed at launch.
struct PipeStage {
    kvl_unit_t u;       // descriptor of the stage's tile
    uint32_t tile;      // index of the tile inside its descriptor
    bool valid;         // false: the workgroup has run out of tiles
};
// The descriptors are not written while a kernel runs: read through the constant address
// space they stay scalar loads inside the loop (a plain global pointer may alias the stores
// there, and the compiler then reads it with vector loads it has to wait for at once).
typedef const kvl_unit_t __attribute__((address_space(4))) *cunits_t;

// Inside the loop nothing is conditional: a lane whose position falls outside its descriptor
// (the idle lead of an aligned first tile, the ragged end of the last) moves the descriptor's
// nearest vector instead, a duplicate of what the lane that owns that vector moves, and the
// loop covers only the trips in which every workgroup has a tile.  With a branch around a
// load or a store the compiler can no longer tell how many memory operations are in flight
// and drains them all before every store; without one it waits for exactly the load it needs.
// The last few tiles of each workgroup are done one by one after the loop.
template <bool PACK, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_tile_pipe_kernel(const CopyArgs a, uint32_t tiles_per_unit,
                                                             uint32_t align_dst, uint32_t n_tiles) {
    const uint32_t p = a.plane_begin + blockIdx.y;
    const uint32_t row = a.row_elems[p];
    const uintptr_t pool_base = a.pool[p], xfer_base = a.xfer[p];
    cunits_t units = (cunits_t)(uintptr_t)(a.units + a.unit_begin);
    const uint32_t last_unit = a.n_units - 1;               // the launcher passes at least one descriptor
    const uint32_t G = gridDim.x;                           // <= n_tiles
    // the tile `k` strides ahead of this workgroup's first is tile (k*G + blockIdx.x): kept as
    // (descriptor, tile inside it) and advanced without a division
    const uint32_t step_u = G / tiles_per_unit, step_t = G - step_u * tiles_per_unit;
    uint32_t f_u = blockIdx.x / tiles_per_unit, f_t = blockIdx.x - f_u * tiles_per_unit;   // the fetch stage's tile
    auto fetch = [&](PipeStage &s) {
        s.tile = f_t;
        s.valid = f_u <= last_unit;
        cunits_t q = units + (f_u <= last_unit ? f_u : last_unit);     // always a load, never past the end
        s.u.pool_row = q->pool_row;
        s.u.xfer_row = q->xfer_row;
        s.u.n_rows = q->n_rows;
        f_u += step_u;
        f_t += step_t;
        if (f_t >= tiles_per_unit) {
            f_t -= tiles_per_unit;
            ++f_u;
        }
    };
    // this lane's vector of a stage's tile (descriptors are never empty)
    auto place = [&](const PipeStage &s, gsrc_t &src, gdst_t &dst) {
        const uint32_t n = s.u.n_rows * row;
        const uintptr_t pool = pool_base + (uint64_t)s.u.pool_row * row * 16u;
        const uintptr_t xfer = xfer_base + (uint64_t)s.u.xfer_row * row * 16u;
        const uint32_t lead = align_dst ? ((uint32_t)((PACK ? xfer : pool) >> 4) & 7u) : 0u;
        const uint32_t pos = s.tile * blockDim.x + threadIdx.x;
        uint32_t j = pos >= lead ? pos - lead : 0u;
        j = j < n ? j : n - 1;
        src = (gsrc_t)(PACK ? pool : xfer) + j;
        dst = (gdst_t)(PACK ? xfer : pool) + j;
    };
    // trips in which every workgroup has a tile; the loop takes them two at a time and stops
    // two short, so that its three stages never run past them
    const uint32_t full = n_tiles / G;
    const uint32_t looped = full >= 2 ? (full - 2) & ~1u : 0u;
    // Two sets of registers, A for the even tiles and B for the odd ones, so that nothing is
    // moved from one to the other (a move of loaded data would have to wait for it).
    PipeStage s_a, s_b;
    gsrc_t src_a, src_b;
    gdst_t dst_a, dst_b;
    v4u v_a, v_b;
    fetch(s_a);                                   // tile 0 of this workgroup (there always is one)
    fetch(s_b);                                   // tile 1
    place(s_a, src_a, dst_a);
    v_a = load16<NTL>(src_a);
    fetch(s_a);                                   // tile 2
    for (uint32_t i = 0; i < looped; i += 2) {
        // (a scalar load can only be waited for together with every other one in flight, so a
        // descriptor is fetched after the step's use of the one fetched before it)
        place(s_b, src_b, dst_b);
        v_b = load16<NTL>(src_b);                 // tile i + 1 on its way
        fetch(s_b);                               // descriptor of tile i + 3, first needed two steps on
        store16<SP>(dst_a, v_a);                  // tile i: waits for its own load only
        place(s_a, src_a, dst_a);
        v_a = load16<NTL>(src_a);                 // tile i + 2
        fetch(s_a);                               // tile i + 4
        store16<SP>(dst_b, v_b);                  // tile i + 1
    }
    // in flight: tile `looped` in v_a; s_b holds tile looped + 1, s_a tile looped + 2
    store16<SP>(dst_a, v_a);
    // the remaining tiles of this workgroup (at most three: looped + 1, + 2, + 3), one at a
    // time; they may not exist, and their idle lanes are switched off rather than duplicated
    PipeStage s_c;
    fetch(s_c);                                   // tile looped + 3
    auto copy_tile = [&](const PipeStage &s) {
        const uint32_t n = s.valid ? s.u.n_rows * row : 0u;
        const uintptr_t pool = pool_base + (uint64_t)s.u.pool_row * row * 16u;
        const uintptr_t xfer = xfer_base + (uint64_t)s.u.xfer_row * row * 16u;
        const uint32_t lead = align_dst ? ((uint32_t)((PACK ? xfer : pool) >> 4) & 7u) : 0u;
        const uint32_t pos = s.tile * blockDim.x + threadIdx.x;
        if (pos >= lead && pos - lead < n) {
            gsrc_t sp = (gsrc_t)(PACK ? pool : xfer) + (pos - lead);
            gdst_t dp = (gdst_t)(PACK ? xfer : pool) + (pos - lead);
            store16<SP>(dp, load16<NTL>(sp));
        }
    };
    copy_tile(s_b);
    copy_tile(s_a);
    copy_tile(s_c);
}

// Flat form for descriptors much smaller than a workgroup: the lanes of the launch are
// dealt to the descriptors m at a time (m = max_unit_rows * row, the vectors of the
// largest descriptor), so lane g moves vector g mod m of descriptor g div m; a shorter
// descriptor leaves its last lanes idle.  The launcher keeps n_units * m below 2^31.
// What a wavefront waits for before its data bounds it, and the instructions for that: the arguments are in registers, the
// division is a multiplication of the wavefront's first lane, and the descriptors that its lanes lie in, at most K, come through
// the scalar cache (m below 16: each lane loads its own).  Against a division and a load of the descriptor per lane, us: hops,
// 130-byte rows by 16, 31 MB 28.9 / 27.7, 207 MB 170 / 162; 82 by 24, 207 MB 193 / 175; 33 by 16, 31 MB 36.7 / 34.5; 20 by 64, 207 MB 183 /
// 165; moves, 1152 by 1, 31 MB 12.7 / 11.6, 310 MB 109.4 / 104.8; 150 by 24, 620 MB 221 / 211.
template <int K>
__device__ __forceinline__ void flat_pick(const kvl_unit_t *units, uint32_t last, uint32_t u_idx, uint32_t m, uint32_t at, kvl_unit_t *u,
                                          uint32_t *off, uint32_t *nth) {
    kvl_unit_t d[K];
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] = fetch_unit(units, min(u_idx + (uint32_t)k, last));
    uint32_t skip = 0;
    *u = d[0];
#pragma unroll
    for (int k = 1; k < K; ++k) {
        const bool past = at >= (uint32_t)k * m;
        u->pool_row = past ? d[k].pool_row : u->pool_row;
        u->xfer_row = past ? d[k].xfer_row : u->xfer_row;
        u->n_rows = past ? d[k].n_rows : u->n_rows;
        skip = past ? (uint32_t)k * m : skip;
        *nth = past ? u_idx + (uint32_t)k : *nth;
    }
    *off = at - skip;
}

// This lane's descriptor and its place in it; false: beyond the last descriptor.  (Descriptors of less than 63 lanes, SHORT, in kernels of
// their own: the branches cost the others 1 %.)
constexpr uint32_t kFlatShort = 63;
template <bool SHORT>
__device__ __forceinline__ bool flat_unit(const kvl_unit_t *units, uint32_t n_units, uint32_t m, uint32_t magic, uint32_t shift,
                                          uint32_t group, uint32_t threads, kvl_unit_t *u, uint32_t *off) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t first = group * threads + __builtin_amdgcn_readfirstlane(threadIdx.x - lane);
    if (SHORT && m < 16) {
        const uint32_t g = first + lane, u_idx = magic ? __umulhi(g, magic) >> shift : g;
        if (u_idx >= n_units) return false;
        *u = units[u_idx];
        *off = g - u_idx * m;
        return true;
    }
    const uint32_t u_idx = __umulhi(first, magic) >> shift;
    if (u_idx >= n_units) return false;
    const uint32_t at = first - u_idx * m + lane;       // below m + 63
    uint32_t nth = u_idx;
    if (!SHORT) flat_pick<2>(units, n_units - 1u, u_idx, m, at, u, off, &nth);
    else if (m >= 32) flat_pick<3>(units, n_units - 1u, u_idx, m, at, u, off, &nth);
    else flat_pick<5>(units, n_units - 1u, u_idx, m, at, u, off, &nth);
    return nth < n_units;
}
#define KVL_FLAT_PARAMS                                                                                            \
    const kvl_unit_t *units, uintptr_t pool, uintptr_t xfer, uint32_t row, uint32_t n_units, uint32_t m, uint32_t magic, \
        uint32_t shift, uint32_t threads
#define KVL_FLAT_ARGS units, pool, xfer, row, n_units, m, magic, shift, threads

template <bool PACK, bool NTL, int SP, bool SHORT>
__device__ __forceinline__ void flat_body(KVL_FLAT_PARAMS, const TileMore &more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    kvl_unit_t u;
    uint32_t off;
    if (!flat_unit<SHORT>(units, n_units, m, magic, shift, blockIdx.x, threads, &u, &off)) return;
    if (off >= u.n_rows * row) return;
    gsrc_t src = (gsrc_t)((PACK ? pool : xfer) + (uint64_t)(PACK ? u.pool_row : u.xfer_row) * row * 16u);
    gdst_t dst = (gdst_t)((PACK ? xfer : pool) + (uint64_t)(PACK ? u.xfer_row : u.pool_row) * row * 16u);
    store16<SP>(dst + off, load16<NTL>(src + off));
}

template <bool PACK, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_flat_kernel(KVL_FLAT_PARAMS, const TileMore more) {
    flat_body<PACK, NTL, SP, false>(KVL_FLAT_ARGS, more);
}

template <bool PACK, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_flat_kernel_short(KVL_FLAT_PARAMS, const TileMore more) {
    flat_body<PACK, NTL, SP, true>(KVL_FLAT_ARGS, more);
}

// Row-map form for descriptors of a few rows: the transfer side is dense, so the launch is laid out over it
// (lane g moves vector g of the range, lined up with the transfer buffer's 128-byte lines) and each row's
// place in the pool comes from a table with one entry per row, made from the descriptors when they are
// uploaded.  However ragged the descriptors are, no lane idles.  A wavefront's 64 vectors lie in at most K
// rows: their entries are fetched through the scalar cache and each lane picks its own (K == 0, for rows below
// 256 bytes: a vector load per lane).  A million single-row blocks of 1152 bytes, 1.17 GB a layer, gather + scatter:
// 1122 us (tiled, because one chance pair of neighbours made the largest descriptor two rows, + flat) -> 763 us (6.1 TB/s).
typedef const uint32_t __attribute__((address_space(4))) *cmap_t;

template <bool PACK, bool NTL, int SP, int K>
__device__ __forceinline__ void rows_body(const uint32_t *row_map, uintptr_t pool_base, uintptr_t xfer_base, uint32_t row,
                                          uint32_t row_begin, uint32_t n_vecs, uint32_t group, uint32_t threads) {
    const uintptr_t xfer = xfer_base + (uint64_t)row_begin * row * 16u;
    const uint32_t lead = (uint32_t)(xfer >> 4) & 7u;
    const uint32_t pos = group * threads + threadIdx.x;
    const uint32_t g = pos - lead;
    if (pos < lead || g >= n_vecs) return;
    cmap_t map = (cmap_t)(uintptr_t)(row_map + row_begin);
    uint32_t pool_row, off;             // the lane's row in the pool and its vector inside that row
    if (K == 0) {
        const uint32_t r = g / row;
        off = g - r * row;
        pool_row = map[r];
    } else {
        const uint32_t first = __builtin_amdgcn_readfirstlane(g);       // of the wavefront's lanes with work
        const uint32_t r = first / row;
        uint32_t entry[K > 0 ? K : 1];
#pragma unroll
        for (int k = 0; k < K; ++k) entry[k] = map[r + k];              // (the table is padded by 8 entries)
        off = g - r * row;
        pool_row = entry[0];
        uint32_t skip = 0;
#pragma unroll
        for (int k = 1; k < K; ++k) {
            const bool past = off >= (uint32_t)k * row;
            pool_row = past ? entry[k] : pool_row;
            skip = past ? (uint32_t)k * row : skip;
        }
        off -= skip;
    }
    const uintptr_t pool = pool_base + ((uint64_t)pool_row * row + off) * 16u;
    gsrc_t src = (gsrc_t)(PACK ? pool : xfer + (uint64_t)g * 16u);
    gdst_t dst = (gdst_t)(PACK ? xfer + (uint64_t)g * 16u : pool);
    store16<SP>(dst, load16<NTL>(src));
}

template <bool PACK, bool NTL, int SP, int K>
__global__ void __launch_bounds__(1024) kvl_rows_kernel(const uint32_t *row_map, uintptr_t pool, uint32_t row_begin, uint32_t n_vecs,
                                                        uintptr_t xfer, uint32_t row, uint32_t threads, uint32_t order,
                                                        const TileMore more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    rows_body<PACK, NTL, SP, K>(row_map, pool, xfer, row, row_begin, n_vecs, tile_number(blockIdx.x, order), threads);
}

// Planes of unlike rows in one launch, the workgroups of one plane after those of the other, each plane with its own number:
// a launch of its own costs a narrow plane more than its bytes do, on the host and between the kernels.  By tiles or by the
// row map, with the cache policies of the kernels above.  Planes of 1024 and 128 bytes by 64, us, apart / at once: hop 3 MB
// 23.3 / 17.6, 105 MB 66.3 / 62.5, 330 MB 200 / 194; move 3 MB 11.5 / 9.0; 512, 16 and 128 bytes, hop 28 MB 30.1 / 21.2.
struct PlanesArgs {
    uint32_t group_end[KVL_MAX_PLANES];        // workgroups up to and with this plane
    uint32_t per_unit[KVL_MAX_PLANES];         // tiles of a descriptor
    uint32_t align_dst[KVL_MAX_PLANES];        // the destination's spans may begin off a line
    uint32_t plain[KVL_MAX_PLANES];            // scatter by tiles: plain loads
    uint32_t row_begin, n_rows;                // transfer rows of the launch's descriptors
};

// SP: the stores (a scatter's by the row map off lines are nt).  ROWS: 0 by tiles; else by the row
// map, the entries of rows of 16 to 63 vectors by a vector load per lane (1), or through the scalar cache as kvl_rows_kernel has
// them (2).  The latter is better in a scatter of a layer beyond the on-die cache (512- and 16-byte rows by 256, scatter, us, 1 /
// 2: 289 MB 99.7 / 92.1, 367 MB 121.9 / 113.8; 512 and 128 by 8, 402 MB, 134.8 / 128.4; 200 MB 59.0 / 59.3), or of one that is
// read by nt loads, off the lines (304 and 80 by 4, 218 MB, 71.8 / 69.0; 656 and 128 by 64, 186 MB, 62.4 / 60.4); not in a gather
// (349 MB 103.7 / 104.6, 219 MB of 512 and 128 66.7 / 68.8).
template <bool PACK, int SP, int ROWS>
__global__ void __launch_bounds__(1024) kvl_planes_kernel(const CopyArgs a, const PlanesArgs pl, const uint32_t *row_map) {
    uint32_t p = a.plane_begin;
#pragma unroll
    for (uint32_t q = 0; q + 1 < KVL_MAX_PLANES; ++q) p += blockIdx.x >= pl.group_end[q] ? 1u : 0u;
    const uint32_t group = blockIdx.x - (p > a.plane_begin ? pl.group_end[p - 1] : 0u);
    const uint32_t row = a.row_elems[p];
    const uint32_t n_vecs = pl.n_rows * row;
    constexpr int kMid = ROWS == 2 ? 3 : 0, kShort = ROWS == 2 ? 5 : 0;        // rows of 32 to 63 and of 16 to 31 vectors
#define KVL_PLANE_ROWS(POLICY, K) \
    rows_body<PACK, true, POLICY, K>(row_map, a.pool[p], a.xfer[p], row, pl.row_begin, n_vecs, group, blockDim.x)
    if (!ROWS) {
        const uint32_t u_idx = group / pl.per_unit[p], tile = group - u_idx * pl.per_unit[p];
        const kvl_unit_t u = fetch_unit(a.units, a.unit_begin + u_idx);
        if (!PACK && pl.plain[p]) tile_span<PACK, 1, false, SP>(u, a.pool[p], a.xfer[p], row, tile, blockDim.x, pl.align_dst[p]);
        else tile_span<PACK, 1, true, SP>(u, a.pool[p], a.xfer[p], row, tile, blockDim.x, pl.align_dst[p]);
    } else if (PACK || row % 8 == 0) {
        if (row >= 64) KVL_PLANE_ROWS(SP, 2);
        else if (ROWS == 2 && row >= 32) KVL_PLANE_ROWS(SP, kMid);
        else if (ROWS == 2 && row >= 16) KVL_PLANE_ROWS(SP, kShort);
        else KVL_PLANE_ROWS(SP, 0);
    } else {
        if (row >= 64) KVL_PLANE_ROWS(1, 2);
        else if (ROWS == 2 && row >= 32) KVL_PLANE_ROWS(1, kMid);
        else if (ROWS == 2 && row >= 16) KVL_PLANE_ROWS(1, kShort);
        else KVL_PLANE_ROWS(1, 0);
    }
#undef KVL_PLANE_ROWS
}

// Rows or addresses that are not multiples of 16 bytes.  The vector unit takes 16-byte accesses at any
// byte address (the ABI's unaligned access mode), so only the ends of a span need care: vectors are
// laid out from the 16-byte boundary at or below the span's first destination byte, and the two that
// stick out over an end are pushed inside the span, where they move some bytes a second time (the same
// bytes to the same place).  Nothing is conditional but the lanes without work.  Bound by memory like the
// forms above: a 280 MB layer of 132-byte rows in 64-token blocks, gather + scatter, 618 us byte by byte
// (1.8 TB/s), 205 us now (5.5 TB/s).
typedef v4u __attribute__((aligned(1))) v4u_any;
typedef const v4u_any __attribute__((address_space(1))) *gsrc_any_t;
typedef v4u_any __attribute__((address_space(1))) *gdst_any_t;
typedef uint8_t __attribute__((address_space(1))) *gbytes_t;

template <bool NT>
__device__ __forceinline__ v4u load16_any(uintptr_t p) {
    if (NT) return __builtin_nontemporal_load((gsrc_any_t)p);
    return *(gsrc_any_t)p;
}

template <int SP>
__device__ __forceinline__ void store16_any(uintptr_t p, v4u v) {
    if (SP == 0) *(gdst_any_t)p = v;
    else if (SP == 1) __builtin_nontemporal_store(v, (gdst_any_t)p);
    else store16<SP>((gdst_t)p, v);          // written out as an instruction: no alignment is assumed
}

// Vector `k` of a span of n bytes, vectors counted from `lead` bytes below its first byte.
template <bool NTL, int SP>
__device__ __forceinline__ void copy_any(uintptr_t src, uintptr_t dst, uint32_t n, uint32_t lead, uint32_t k) {
    int64_t at = (int64_t)((uint64_t)k * 16u) - (int64_t)lead;
    if (at <= -16 || at >= (int64_t)n) return;
    if (n >= 16) {
        const int64_t last = (int64_t)n - 16;
        at = at < 0 ? 0 : at > last ? last : at;
        store16_any<SP>(dst + at, load16_any<NTL>(src + at));
    } else {
        // spans shorter than a vector: byte by byte, each lane its own 16-byte window
        const uint32_t end = (uint32_t)(at + 16 < (int64_t)n ? at + 16 : (int64_t)n);
        for (uint32_t i = at < 0 ? 0u : (uint32_t)at; i < end; ++i) ((gbytes_t)dst)[i] = ((gbytes_t)src)[i];
    }
}

// Tiled: a tile is blockDim vectors; one workgroup per tile, or (the walk) gridDim.x of them walking over n_tiles.
// Tiles begin on 128-byte lines of the destination, or (SRC) of the source: then every line of the source is read by one
// wavefront alone, but for those that two descriptors share.  A line that the on-die cache holds is taken out of it by a
// non-temporal load, so that a line shared by two wavefronts is fetched from memory by the second.  Lines of the destination
// are shared by two wavefronts instead.  A scatter's stores to them meet in the L2, which they must not be written through for
// (hops of 304 MB, 1026-byte rows by 64, us: gather and scatter on lines of the destination 209, of the source with nt stores
// out of the scatter 195, with sc1+nt ones 219); a gather's are written through (sc1) all the same, because they leave the
// layer in the on-die cache for the scatter (hops, sc1 / nt stores out of the gather: 132 by 64, 197 MB, 136 / 156; 1026 by 64,
// 305 MB, 190 / 221).
template <bool PACK, bool NTL, int SP, bool SRC>
__device__ __forceinline__ void any_span(const kvl_unit_t u, uintptr_t pool_base, uintptr_t xfer_base, uint32_t row, uint32_t k) {
    const uintptr_t pool = pool_base + (uint64_t)u.pool_row * row;
    const uintptr_t xfer = xfer_base + (uint64_t)u.xfer_row * row;
    const uintptr_t src = PACK ? pool : xfer, dst = PACK ? xfer : pool;
    copy_any<NTL, SP>(src, dst, u.n_rows * row, (uint32_t)(SRC ? src : dst) & 127u, k);
}

template <bool PACK, bool NTL, int SP, bool SRC>
__global__ void __launch_bounds__(1024) kvl_any_tile_kernel(KVL_TILE_PARAMS, const TileMore more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    const uint32_t b = tile_number(blockIdx.x, order);
    const uint32_t u_idx = magic ? (uint32_t)(((uint64_t)b * magic) >> 32) >> (how >> 1) : b;
    any_span<PACK, NTL, SP, SRC>(fetch_unit(units, u_idx), pool, xfer, row, (b - u_idx * tiles_per_unit) * threads + threadIdx.x);
}

// (With as many workgroups as tiles: a form that starts late, its arguments fetched one after the other.)
template <bool PACK, bool NTL, int SP, bool SRC>
__global__ void __launch_bounds__(1024) kvl_any_walk_kernel(const CopyArgs a, uint32_t tiles_per_unit, uint32_t n_tiles, uint32_t order) {
    const uint32_t p = a.plane_begin + blockIdx.y;
    const uint32_t row = a.row_elems[p];
    const uintptr_t pool = a.pool[p], xfer = a.xfer[p];
    for (uint32_t t = tile_number(blockIdx.x, order); t < n_tiles; t += gridDim.x) {
        const uint32_t u_idx = t / tiles_per_unit;
        any_span<PACK, NTL, SP, SRC>(fetch_unit(a.units, a.unit_begin + u_idx), pool, xfer, row,
                                     (t - u_idx * tiles_per_unit) * blockDim.x + threadIdx.x);
    }
}

// Flat, as kvl_flat_kernel: m lanes per descriptor (m = the most 16-byte windows that the largest one touches).
template <bool PACK, bool NTL, int SP, bool SHORT>
__device__ __forceinline__ void any_flat_body(KVL_FLAT_PARAMS, uint32_t order, const TileMore &more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        xfer = more.xfer[blockIdx.y - 1];
    }
    kvl_unit_t u;
    uint32_t off;
    if (!flat_unit<SHORT>(units, n_units, m, magic, shift, tile_number(blockIdx.x, order), threads, &u, &off)) return;
    const uintptr_t in_pool = pool + (uint64_t)u.pool_row * row;
    const uintptr_t in_xfer = xfer + (uint64_t)u.xfer_row * row;
    const uintptr_t dst = PACK ? in_xfer : in_pool;
    copy_any<NTL, SP>(PACK ? in_pool : in_xfer, dst, u.n_rows * row, (uint32_t)dst & 15u, off);
}

template <bool PACK, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_any_flat_kernel(KVL_FLAT_PARAMS, uint32_t order, const TileMore more) {
    any_flat_body<PACK, NTL, SP, false>(KVL_FLAT_ARGS, order, more);
}

template <bool PACK, bool NTL, int SP>
__global__ void __launch_bounds__(1024) kvl_any_flat_kernel_short(KVL_FLAT_PARAMS, uint32_t order, const TileMore more) {
    any_flat_body<PACK, NTL, SP, true>(KVL_FLAT_ARGS, order, more);
}

// Storage layout <-> paged pool for one layer.  Same tiling as above; the far
// side is a buffer of Full Blocks ([layer, tokens, bytes] per block), so a
// descriptor (which never spans blocks here) lands at
//   block_index * FB + (layer, plane) offset + row-in-block * row.
// The buffer may be pinned host memory: then these accesses cross the host link.
struct FullBlockArgs {
    const kvl_unit_t *units;
    uint32_t n_units;
    uint32_t block_tokens;
    uint32_t row_elems[KVL_MAX_PLANES];       // 16-byte vectors (VEC) or bytes per row
    uintptr_t pool[KVL_MAX_PLANES];
    uintptr_t blocks;                          // base of the Full-Block buffer
    uint64_t fb_elems;                         // elements per Full Block
    uint64_t layer_plane_off[KVL_MAX_PLANES];  // element offset of (layer, plane) inside a Full Block
    uint32_t tile_end[KVL_MAX_PLANES];         // tiles of a descriptor up to and with this plane
    uint32_t magic, shift, tokens_magic;       // division by a descriptor's tiles (TileDivisor) and by block_tokens (remainder_by)
};

// n mod d, with magic = floor((2^32 - 1) / d): the quotient by multiplication is right or one too small, for any 32 bits.
__host__ __device__ __forceinline__ uint32_t remainder_by(uint32_t n, uint32_t d, uint32_t magic) {
    const uint32_t r = n - (uint32_t)(((uint64_t)n * magic) >> 32) * d;
    return r >= d ? r - d : r;
}

// A tile is VPT * blockDim vectors of a descriptor's plane; lane t takes vectors t, t + blockDim, ...  of it, all loads
// before the first store.  VEC: whole 16-byte vectors; else any byte addresses, one vector per lane (copy_any).
// Bound by memory: the policies are those of the copy kernels with the same direction through the on-die cache (into
// the pool nt loads and sc1 stores, which leave the layer there for whoever reads it next; out of it nt loads and
// sc1+nt stores).  Both directions in turn, 64-token blocks of 61 layers, us a layer, against plain loads with sc1+nt
// stores one way and nt loads with plain stores the other: 1152-byte rows, 101 MB a layer, 89 -> 63; 221 MB 185 -> 142;
// 1.8 GB 1388 -> 1305; 656-byte rows, 58 MB, 59 -> 46.  SRC (one vector per lane): tiles begin on 128-byte lines of the
// source, which a non-temporal load then takes out of the cache once (kvl_any_tile_kernel): blocks that begin off a line,
// both directions, 336-byte rows by 100, 43 MB, 35.6 -> 31.2; at byte addresses, where they began on lines of the
// destination, with nt stores out of the pool (763 by 64, 52 MB, 40.2 -> 35.7), but for blocks that begin and end on lines of
// both sides, where sc1+nt stores are ahead (four layers, nt / sc1+nt: 1026 by 64, 144 MB, 348 / 342; 661 by 256, 169 MB, 409 /
// 398; 200 by 16, 98 MB, 285 / 276).  Across the host link the old ones stay for whole vectors (the link is the bound); at byte
// addresses the new ones are ahead there too (out of the pool, new / old: 741-byte rows by 64, 40 MB, 706 / 727; 57 by 16, 20 MB,
// 382 / 426; 132 by 1, 8 MB, 255 / 425; into it level).
// The descriptor comes in one load and by multiplications; both directions of four layers of 16, us, with divisions and a load of each field /
// so: 1024- and 128-byte rows by 64, 13.7 MB 48.2 / 46.1, 51 MB 131 / 129; by 1, 26 MB 96.3 / 93.0; 132 by 64, 13.7 MB 49.5 / 47.1.
template <bool TO_POOL, bool VEC, int VPT, bool NTL, int SP, bool SRC>
__device__ __forceinline__ void fullblock_tile(const FullBlockArgs &a, uint32_t tiles_per_unit, uint32_t tile_index) {
    const uint32_t u_idx = a.magic ? (uint32_t)(((uint64_t)tile_index * a.magic) >> 32) >> a.shift : tile_index;
    uint32_t tile = tile_index - u_idx * tiles_per_unit;
    const kvl_unit_t u = fetch_unit(a.units, u_idx);
    // a descriptor's tiles are those of its planes one after the other, each plane its own number of them
    uint32_t p = 0;
#pragma unroll
    for (uint32_t q = 0; q + 1 < KVL_MAX_PLANES; ++q) p += tile >= a.tile_end[q] ? 1u : 0u;
    tile -= p ? a.tile_end[p - 1] : 0u;
    const uint32_t row = a.row_elems[p], pool_row = u.pool_row;
    const uint32_t n = u.n_rows * row;
    const uint32_t first = tile * (blockDim.x * VPT) + threadIdx.x;
    const uint32_t within = remainder_by(pool_row, a.block_tokens, a.tokens_magic);
    const uint64_t in_pool = (uint64_t)pool_row * row;
    const uint64_t in_blocks = (uint64_t)u.block_index * a.fb_elems + a.layer_plane_off[p] + (uint64_t)within * row;
    if (VEC) {
        gsrc_t src = TO_POOL ? (gsrc_t)a.blocks + in_blocks : (gsrc_t)a.pool[p] + in_pool;
        gdst_t dst = TO_POOL ? (gdst_t)a.pool[p] + in_pool : (gdst_t)a.blocks + in_blocks;
        if (SRC) {
            const uint32_t lead = (uint32_t)((uintptr_t)src >> 4) & 7u;
            if (first >= lead && first - lead < n) store16<SP>(dst + (first - lead), load16<NTL>(src + (first - lead)));
            return;
        }
        if (first >= n) return;
        v4u v[VPT];
#pragma unroll
        for (int k = 0; k < VPT; ++k) {
            const uint32_t i = first + k * blockDim.x;
            if (i < n) v[k] = load16<NTL>(src + i);
        }
#pragma unroll
        for (int k = 0; k < VPT; ++k) {
            const uint32_t i = first + k * blockDim.x;
            if (i < n) store16<SP>(dst + i, v[k]);
        }
    } else {
        const uintptr_t pool = a.pool[p] + in_pool, blocks = a.blocks + in_blocks;
        const uintptr_t src = TO_POOL ? blocks : pool, dst = TO_POOL ? pool : blocks;
        copy_any<NTL, SP>(src, dst, n, (uint32_t)(SRC ? src : dst) & 127u, first);
    }
}

// gridDim.x workgroups walk over the n_tiles tiles (one tile each when there are as many).
template <bool TO_POOL, bool VEC, int VPT, bool NTL, int SP, bool SRC>
__global__ void __launch_bounds__(256) kvl_fullblock_kernel(const FullBlockArgs a, uint32_t tiles_per_unit,
                                                            uint32_t n_tiles, uint32_t order) {
    for (uint32_t t = tile_number(blockIdx.x, order); t < n_tiles; t += gridDim.x)
        fullblock_tile<TO_POOL, VEC, VPT, NTL, SP, SRC>(a, tiles_per_unit, t);
}

// Planes alike, of whole vectors in device memory: the first one's arguments in registers (`blocks`: its part of the first Full Block),
// the descriptor in one load, no division, tiles in runs, as in the quick tiles above.  Both directions of four layers of 16, us, before /
// so: 1152-byte rows by 64, 10 MB a layer 42.3 / 36.9, 25 MB 74.0 / 67.6, 88 MB 218 / 207; 1152 by 16, 10 MB 43.2 / 36.2; 496 by 1, 27 MB
// 138 / 125; 4096 by 64 (Layer Blocks 4 MiB apart), 24 MB 81.6 / 64.6, 211 MB 583 / 464.
// In small layers, where the host's part of a call is most of it, ahead too: the eight calls of four layers of 1152 by 64 on the default stream,
// 0.3 MB 32.1 / 26.7, 2.2 MB 32.9 / 26.0, 5.3 MB 37.7 / 30.0; in a HIP graph 0.3 MB 15.4 / 14.3, 2.2 MB 24.8 / 18.6, 4.6 MB 28.9 / 21.5.
template <bool TO_POOL>
__global__ void __launch_bounds__(256) kvl_fullblock_quick_kernel(const kvl_unit_t *units, uintptr_t pool, uintptr_t blocks, uint32_t fb_vecs,
                                                                  uint32_t row, uint32_t tiles_per_unit, uint32_t magic, uint32_t shift_threads,
                                                                  uint32_t block_tokens, uint32_t tokens_magic, uint32_t order,
                                                                  const TileMore more) {
    if (blockIdx.y) {
        pool = more.pool[blockIdx.y - 1];
        blocks = more.xfer[blockIdx.y - 1];
    }
    const uint32_t b = tile_number(blockIdx.x, order);
    const uint32_t u_idx = magic ? (uint32_t)(((uint64_t)b * magic) >> 32) >> (shift_threads >> 16) : b;
    const kvl_unit_t u = fetch_unit(units, u_idx);
    const uint32_t n = u.n_rows * row, first = (b - u_idx * tiles_per_unit) * (shift_threads & 0xffffu) + threadIdx.x;
    const gdst_t in_pool = (gdst_t)pool + (uint64_t)u.pool_row * row;
    const gdst_t in_blocks = (gdst_t)blocks + ((uint64_t)u.block_index * fb_vecs + (uint64_t)remainder_by(u.pool_row, block_tokens, tokens_magic) * row);
    const gsrc_t src = (gsrc_t)(TO_POOL ? in_blocks : in_pool);
    const gdst_t dst = TO_POOL ? in_pool : in_blocks;
    const uint32_t lead = (uint32_t)((uintptr_t)src >> 4) & 7u;
    if (first >= lead && first - lead < n) store16<TO_POOL ? 2 : 3>(dst + (first - lead), load16<true>(src + (first - lead)));
}

// Reference streams for measuring what the memory can do (kvl_ceiling_kernel): the tiled form
// with its addresses computed instead of read from descriptors.  Block u of the dense side
// lives in block (u * mul) mod 2^k of the hopping side (mul odd: a bijection), or in block
// table[u] if a table is given (one scalar load, as the descriptor fetch of the real kernels).
struct CeilingArgs {
    uintptr_t dense, hopping;       // base addresses
    const uint32_t *table;          // optional
    uint32_t magic, shift, order;   // the block of a tile by multiplication (TileDivisor); the order of the tiles (tile_number)
    uint32_t n_blocks, hop_mask, mul;
    uint32_t block_vecs, tiles_per_block, skew_vecs;
};

// MODE 0: copy, 1: read only, 2: write only.  GATHER: the source hops, else the destination.
template <int MODE, bool GATHER, bool NTL, int SP>
__global__ void __launch_bounds__(256) kvl_ceiling_pattern_kernel(const CeilingArgs a) {
    const uint32_t w = tile_number(blockIdx.x, a.order);
    const uint32_t u = a.magic ? (uint32_t)(((uint64_t)w * a.magic) >> 32) >> a.shift : w;
    const uint32_t tile = w - u * a.tiles_per_block;
    const uint32_t hb = a.table ? a.table[u] : ((u * a.mul) & a.hop_mask);
    const uintptr_t hop = a.hopping + (uint64_t)hb * a.block_vecs * 16u;
    const uintptr_t den = a.dense + ((uint64_t)u * a.block_vecs + a.skew_vecs) * 16u;
    gsrc_t src = (gsrc_t)(GATHER ? hop : den);
    gdst_t dst = (gdst_t)(GATHER ? den : hop);
    const uint32_t lead = (uint32_t)((GATHER ? den : hop) >> 4) & 7u;     // tiles start on a destination line
    const uint32_t pos = tile * blockDim.x + threadIdx.x;
    if (pos < lead || pos - lead >= a.block_vecs) return;
    if (MODE == 0) {
        store16<SP>(dst + (pos - lead), load16<NTL>(src + (pos - lead)));
    } else if (MODE == 1) {
        const v4u v = load16<NTL>(src + (pos - lead));
        if (v.x == 0x9e3779b9u && v.y == 0x7f4a7c15u && v.z == 0xf39cc060u && v.w == 0x5cedc834u)
            store16<SP>(dst + (pos - lead), v);     // keeps the load alive; the pattern does not occur in the buffers
    } else {
        const v4u v = {pos, u, tile, hb};
        store16<SP>(dst + (pos - lead), v);
    }
}

template <int MODE, bool NTL, int SP>
__global__ void __launch_bounds__(256) kvl_ceiling_linear_kernel(const v4u *src, v4u *dst, uint64_t n, uint32_t order) {
    const uint64_t i = (uint64_t)tile_number(blockIdx.x, order) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (MODE == 0) {
        store16<SP>((gdst_t)dst + i, load16<NTL>((gsrc_t)src + i));
    } else if (MODE == 1) {
        const v4u v = load16<NTL>((gsrc_t)src + i);
        if (v.x == 0x9e3779b9u && v.y == 0x7f4a7c15u && v.z == 0xf39cc060u && v.w == 0x5cedc834u)
            store16<SP>((gdst_t)dst + i, v);
    } else {
        const v4u v = {(uint32_t)i, 1u, 2u, 3u};
        store16<SP>((gdst_t)dst + i, v);
    }
}

// Straight copy, one vector per lane: the tiled kernel without descriptors.
__global__ void __launch_bounds__(256) kvl_linear_kernel(const v4u *src, v4u *dst, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) store16<kLinearStorePolicy>((gdst_t)dst + i, load16<kLinearNtLoad>((gsrc_t)src + i));
}

}  // namespace kvl
