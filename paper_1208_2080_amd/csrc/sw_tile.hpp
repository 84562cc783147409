// Tile-level helpers shared by the sweep kernels of both models (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sw_device.hpp"

namespace swmi {

// Waves of a tile workgroup where tiles are many: every wave owns 16 rows of a 64-
// or 128-row tile (8 of a 32-row tile), one column per lane.  64-row tiles have up
// to sixteen waves, of four rows, where tiles are few (start_bond_label, start_flip).
template <int TY>
constexpr uint32_t waves_of() { return TY == 128 ? 8u : 4u; }
template <int TY>
constexpr uint32_t threads_of() { return 64u * waves_of<TY>(); }

// Value of the neighbouring lane of the pair (lane ^ 1).
__device__ __forceinline__ uint32_t swap_pair(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
}

// Lane l's bit of a wave-uniform mask, as a lane predicate.
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Sum over the wave of a per-lane value (all 64 lanes active), in vector
// instructions only: pairs and quads by quad permutes, rows of 16 by half-row
// and row mirrors, then the rows' sums broadcast into row 3 (row_bcast:15 into
// rows 1 and 3, row_bcast:31 into rows 2 and 3), so lane 63 holds the total.
// Where the scalar unit is the busier one this beats a ballot per bit plane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);            // quad_perm [1,0,3,2]
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);            // quad_perm [2,3,0,1]
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);           // row_half_mirror
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);           // row_mirror
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);     // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);     // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Number of set bits of a wave-uniform mask below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Per-lane state counters of the measurement for q <= 16: byte (c & 7) of word
// (c >> 3) counts this lane's sites in state c (at most 31 rows per lane).
// q <= 8 needs only the first word (count_state_byte).
__device__ __forceinline__ void count_state_byte(uint64_t (&w)[2], bool valid, uint32_t s)
{
    w[0] += (uint64_t)valid << (8u * (s & 7u));
}

__device__ __forceinline__ void count_state_bytes(uint64_t (&w)[2], bool valid, uint32_t s)
{
    const uint64_t one = (uint64_t)valid << (8u * (s & 7u));
    w[0] += (s < 8u) ? one : 0ull;
    w[1] += (s < 8u) ? 0ull : one;
}

// Wave totals of states 1..q-1 from the per-lane bytes, added into hist.
__device__ __forceinline__ void flush_state_bytes(const uint64_t (&w)[2], uint32_t* hist, uint32_t q, uint32_t lane)
{
    for (uint32_t c = 1; c < q; ++c) {
        const uint32_t n = wave_sum((uint32_t)(w[c >> 3] >> (8u * (c & 7u))) & 0xFFu);
        if (lane == 0 && n) atomicAdd(&hist[c], n);
    }
}

// Lanes k and k + 1 (k wave-uniform) of the words v[0..3] set to the halves of
// the wave-uniform values x0, y0 (lane k) and x1, y1.  The lane goes through m0
// (an instruction takes one scalar register), which is given back as it was.
__device__ __forceinline__ void write_rows(uint32_t (&v)[4], uint32_t k, uint64_t x0, uint64_t y0, uint64_t x1, uint64_t y1)
{
    uint32_t m0;
    asm("s_mov_b32 %4, m0\n\t"
        "s_mov_b32 m0, %5\n\t"
        "v_writelane_b32 %0, %6, m0\n\t"
        "v_writelane_b32 %1, %7, m0\n\t"
        "v_writelane_b32 %2, %8, m0\n\t"
        "v_writelane_b32 %3, %9, m0\n\t"
        "s_add_u32 m0, m0, 1\n\t"
        "v_writelane_b32 %0, %10, m0\n\t"
        "v_writelane_b32 %1, %11, m0\n\t"
        "v_writelane_b32 %2, %12, m0\n\t"
        "v_writelane_b32 %3, %13, m0\n\t"
        "s_mov_b32 m0, %4"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "=&s"(m0)
        : "s"(k), "s"((uint32_t)x0), "s"((uint32_t)(x0 >> 32)), "s"((uint32_t)y0), "s"((uint32_t)(y0 >> 32)),
          "s"((uint32_t)x1), "s"((uint32_t)(x1 >> 32)), "s"((uint32_t)y1), "s"((uint32_t)(y1 >> 32))
        : "scc");
}

// The value of lane k (wave-uniform) as a scalar.
__device__ __forceinline__ uint64_t lane_value64(uint64_t v, uint32_t k)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)k);
    return ((uint64_t)hi << 32) | lo;
}

struct TileGeom {
    uint32_t tx, ty, x0, y0, w, h;
};

__device__ __forceinline__ TileGeom tile_geom(const LatDesc& d, uint32_t tile, uint32_t ty_rows)
{
    TileGeom g;
    // tiles per row: L / 64 for a power-of-two L >= 64 (a shift), else a division
    g.ty = d.log2L >= 6 ? tile >> (d.log2L - 6u) : tile / d.ntx;
    g.tx = tile - g.ty * d.ntx;
    g.x0 = g.tx * TX;
    g.y0 = g.ty * ty_rows;
    g.w = min(TX, d.L - g.x0);
    g.h = min(ty_rows, d.L - g.y0);
    return g;
}

// Which lattice (lat) and tile this workgroup (or wave) works on.  Without a
// map the work is the tiles of lattice 0, optionally spread over the XCDs so
// that each gets a contiguous band of tiles.  Mapped work (many lattices of
// uneven cost) keeps the hardware's round-robin dealing, which balances the
// XCDs better than bands do.
__device__ __forceinline__ bool pick(const LatDesc* descs, const WorkItem* map, uint32_t idx,
                                     bool spread, LatDesc& d, uint32_t& tile, uint32_t& lat)
{
    if (map) {
        const WorkItem it = map[idx];
        if (it.lat == INVALID) return false;
        d = descs[it.lat];
        tile = it.tile;
        lat = it.lat;
        return true;
    }
    lat = 0;
    d = descs[0];
    if (idx >= d.ntiles) return false;
    tile = spread ? xcd_tile(idx, d.ntiles) : idx;
    return true;
}

__device__ __forceinline__ void flag_error(uint32_t* err)
{
    __hip_atomic_fetch_or(glb(err), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Index of this wave in its workgroup as a wave-uniform (scalar) value, for
// kernels where work selected by it (descriptor loads) should stay scalar.
__device__ __forceinline__ uint32_t wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

__device__ __forceinline__ void atomic_add_i64(int64_t* p, uint64_t v)
{
    __hip_atomic_fetch_add(glb(reinterpret_cast<unsigned long long*>(p)), (unsigned long long)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------ phase clocks
// Profiling builds only (-DSW_PHASE_CLOCKS; the library is then built apart
// from the product one): each wave sums the shader-clock ticks it spends
// between consecutive marks, per phase, and its lane 0 adds the sums and a
// wave count to a per-kernel table of NCOPY rows of PHASES + 1 counters (rows
// picked by workgroup, to spread the atomics).  In every other build the marks
// compile to nothing.
constexpr uint32_t PHASES = 10;
#ifdef SW_PHASE_CLOCKS
struct PhaseClock {
    uint64_t last;
    uint32_t acc[PHASES];
    __device__ PhaseClock() : last(__builtin_amdgcn_s_memtime())
    {
        for (uint32_t i = 0; i < PHASES; ++i) acc[i] = 0;
    }
    __device__ void mark(uint32_t i)
    {
        const uint64_t now = __builtin_amdgcn_s_memtime();
        acc[i] += (uint32_t)(now - last);
        last = now;
    }
    __device__ void flush(unsigned long long* table)
    {
        if ((threadIdx.x & 63u) != 0) return;
        unsigned long long* row = table + (blockIdx.x % NCOPY) * (PHASES + 1);
        for (uint32_t i = 0; i < PHASES; ++i)
            if (acc[i]) atomicAdd(&row[i], (unsigned long long)acc[i]);
        atomicAdd(&row[PHASES], 1ull);
    }
};
#define SW_PHASE_START(pc) PhaseClock pc
#define SW_PHASE(pc, i) pc.mark(i)
#define SW_PHASE_FLUSH(pc, table) pc.flush(table)
#else
#define SW_PHASE_START(pc)
#define SW_PHASE(pc, i) ((void)0)
#define SW_PHASE_FLUSH(pc, table) ((void)0)
#endif

constexpr uint32_t LDS_CAP = 1u << 15;     // cap of union retries in LDS (> sites of a tile)

// ------------------------------------------------------- LDS union-find
// P holds, for every site of the tile (or of a whole lattice of at most
// 128 x 128 sites), a site that is never larger than its own; roots point at
// themselves.  Unions hook the larger root under the smaller one, finds point
// nodes at their roots: every value stored is smaller than its site, so every
// walk that steps only to smaller sites ends.  A walk that stops at a node
// pointing to a larger site has met a corrupted forest and sets `bad`, which the
// kernel reports.
//
// A tile's entries are 16 bits, half the LDS, so more workgroups fit a CU (a
// whole lattice's 32), and name their sites by the byte offset of the site's own
// entry (twice the index, below 2^15), so that a step of a walk needs no shift.
// Vector issue bounds the labelling, and a step of a find is four vector
// instructions this way, eight with indices and 16-bit values that the compiler
// masks again; a hook is one masked exchange instead of a read and a loop of
// compare-and-swaps.  The labelling at L = 16384, q = 2, K_c: 0.630 ms before,
// 0.605 with offsets, 0.575 with the exchange too.
__device__ __forceinline__ uint32_t lds_ld(uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_st(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The entry that a site names, by byte offset (16 bits) or index (32 bits).
__device__ __forceinline__ uint16_t* lds_entry(uint16_t* P, uint32_t at)
{
    return reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(P) + at);
}
__device__ __forceinline__ uint32_t lds_get(uint16_t* P, uint32_t at)
{
    return *(volatile __attribute__((address_space(3))) uint16_t*)lds_entry(P, at);
}
__device__ __forceinline__ void lds_set(uint16_t* P, uint32_t at, uint32_t v)
{
    __hip_atomic_store(lds_entry(P, at), (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t lds_get(uint32_t* P, uint32_t at) { return lds_ld(&P[at]); }
__device__ __forceinline__ void lds_set(uint32_t* P, uint32_t at, uint32_t v) { lds_st(&P[at], v); }

// Two entries at once.  (The compiler masks a 16-bit load's register again when
// its value goes round a loop, hence the instructions themselves.)
__device__ __forceinline__ void lds_get2(uint16_t* P, uint32_t a, uint32_t b, uint32_t& pa, uint32_t& pb)
{
    const uint32_t ea = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds_entry(P, a);
    const uint32_t eb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds_entry(P, b);
    asm volatile("ds_read_u16 %0, %2\n\tds_read_u16 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(pa), "=&v"(pb) : "v"(ea), "v"(eb) : "memory");
}
__device__ __forceinline__ void lds_get2(uint32_t* P, uint32_t a, uint32_t b, uint32_t& pa, uint32_t& pb)
{
    pa = lds_ld(&P[a]);
    pb = lds_ld(&P[b]);
}

// Hangs site hi under lo: lo into its entry, whose value before is returned.
// 32 bits: the smaller of the two stays.  16 bits: a masked exchange on the
// entry's word (LDS has no 16-bit minimum); a smaller value that another hook had
// put there goes back, which keeps walks short (the flip 0.312 ms against 0.317).
// Either way hi may lose a link to a site that it had: the caller joins that site
// with lo, as it does wherever hi was not a root any more.  So all values that an
// entry ever held end in the same cluster, by induction on the site: a lost one
// and its successor are joined among smaller sites.
__device__ __forceinline__ uint32_t lds_hook(uint16_t* P, uint32_t hi, uint32_t lo)
{
    const uint32_t word = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds_entry(P, hi & ~3u);
    const uint32_t sh = (hi & 2u) * 8u;
    uint32_t old;
    asm volatile("ds_mskor_rtn_b32 %0, %1, %2, %3\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(old) : "v"(word), "v"(0xFFFFu << sh), "v"(lo << sh) : "memory");
    old = (old >> sh) & 0xFFFFu;
    if (old < lo) lds_set(P, hi, old);
    return old;
}
__device__ __forceinline__ uint32_t lds_hook(uint32_t* P, uint32_t hi, uint32_t lo)
{
    return __hip_atomic_fetch_min(&P[hi], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Roots of a and b while unions may still run, both walked in the same loop so
// that their LDS round trips overlap.  A walked node is pointed at the root it
// found (an ancestor, so races with other finds and hooks are benign); a chain
// that has ended stays where it is without a predicate.  Splitting the path
// at every step instead takes two more reads and stores a step: the labelling at
// L = 16384 0.670 ms against 0.659; no shortening at all 0.666, but the flip
// then walks longer (0.347 against 0.324).
template <class T>
__device__ __forceinline__ void lds_find2(T* P, uint32_t& a, uint32_t& b, bool& bad)
{
    const uint32_t a0 = a, b0 = b;
    uint32_t pa, pb;
    lds_get2(P, a, b, pa, pb);
    while (pa < a || pb < b) {
        a = min(a, pa);
        b = min(b, pb);
        lds_get2(P, a, b, pa, pb);
    }
    if (a < a0) lds_set(P, a0, a);
    if (b < b0) lds_set(P, b0, b);
    bad |= pa != a || pb != b;
}

template <class T>
__device__ void lds_union(T* P, uint32_t a, uint32_t b, bool& bad)
{
    for (uint32_t it = 0; it < LDS_CAP; ++it) {
        lds_find2(P, a, b, bad);
        if (a == b) return;
        const uint32_t hi = max(a, b), lo = min(a, b);
        const uint32_t old = lds_hook(P, hi, lo);
        if (old == hi) return;
        // hi was hooked meanwhile: join its new parent with lo instead
        a = old;
        b = lo;
    }
    bad = true;
}

}  // namespace swmi
