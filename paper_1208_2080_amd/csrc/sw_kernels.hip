// HIP kernels of one Swendsen-Wang sweep for gfx950, plus their launchers.
//
// One sweep is three launches over the tiles of the lattice (TX = 64 columns
// by TY rows; one workgroup per tile, one column per lane, four waves, eight
// for 128 rows, up to sixteen for 64 rows when tiles are few):
//   k_bond_label  bonds (Sec. 2 step (1)) + tile-local cluster labelling
//                 + measurement of the configuration the bonds were drawn on
//   k_merge       joins tile-local clusters across tile edges (global union-find
//                 with atomicMin, larger root under smaller)
//   k_flip        every cluster takes the state drawn for its smallest site
//                 index (Sec. 2 step (3)); each site follows its in-tile
//                 pointers to a resolved tile-local root
// plus k_measure after the last sweep of a call, and small helpers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sw_device.hpp"
#include "sw_kernels.hpp"
#include "sw_tile.hpp"

namespace swmi {

namespace {

// Every label points at a site index no larger than its own (roots at
// themselves).  Every pointer walk steps only to strictly smaller indices, so
// it ends even in a corrupted forest, and union retries carry caps; a forest
// that breaks the invariant sets the error flag instead of spinning.
constexpr uint32_t UNITE_CAP = 1u << 12;   // cap of union retries in the global forest
constexpr uint32_t SPW = TX + 4;           // LDS row stride of staged spins (bytes)

// ------------------------------------------------------ edge forest (global)
// One node per tile-local cluster that touches a tile edge.  A node's word is
// (key << 32) | parent: parent is a node id, key the smallest site index of the
// parent (a root is its own parent, its key its own smallest site).  Words only
// ever decrease, and ordering words orders keys, so hooking the root with the
// larger word under the one with the smaller (a 64-bit atomicMin) leaves every
// cluster's root at its smallest site.
//
// The finds read through the caches.  A stale word is one the node had
// earlier, still pointing at an ancestor, so chases still end and only ever
// reach true ancestors or stale roots; the hook itself is a device-coherent
// atomicMin that returns the current word, and a hook on a stale root retries
// from that value.  Every step goes to a strictly smaller key, so walks end
// even in a corrupted forest; a step that does not (or leaves the node array)
// sets `bad` and stops.
__device__ __forceinline__ uint32_t node_of(uint64_t w) { return (uint32_t)w; }
__device__ __forceinline__ uint32_t key_of(uint64_t w) { return (uint32_t)(w >> 32); }

__device__ __forceinline__ uint64_t min_coherent64(gptr<uint64_t> p, uint64_t v)
{
    return __hip_atomic_fetch_min(reinterpret_cast<gptr<unsigned long long>>(p), (unsigned long long)v,
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root word of node x whose word w was loaded already (x < n), with path
// splitting (every visited node is pointed at its grandparent when that is a
// real shortcut; any stored word is an ancestor's, so races are benign).
// n: nodes in the array.
__device__ uint64_t n_find_from(gptr<uint64_t> nodes, uint32_t n, uint32_t x, uint64_t w, bool& bad)
{
    for (uint32_t it = 0; it < UNITE_CAP; ++it) {
        const uint32_t p = node_of(w);
        if (p == x) return w;
        if (p >= n) break;
        const uint64_t wp = nodes[p];
        if (key_of(wp) >= key_of(w) && node_of(wp) != p) break;   // keys must fall
        if (wp < w) nodes[x] = wp;
        x = p;
        w = wp;
    }
    bad = true;
    return w;
}

// Read-only root search once the forest is final.
__device__ uint64_t n_root(gptr<const uint64_t> nodes, uint32_t n, uint32_t x, bool& bad)
{
    if (x >= n) {
        bad = true;
        return 0;
    }
    uint64_t w = nodes[x];
    for (uint32_t it = 0; it < UNITE_CAP; ++it) {
        const uint32_t p = node_of(w);
        if (p == x) return w;
        if (p >= n) break;
        const uint64_t wp = nodes[p];
        if (key_of(wp) >= key_of(w) && node_of(wp) != p) break;
        x = p;
        w = wp;
    }
    bad = true;
    return w;
}

// One step of a find (path splitting): from node x with word w to its parent.
// Returns false (and sets bad) if the forest is corrupted.
__device__ __forceinline__ bool n_step(gptr<uint64_t> nodes, uint32_t n, uint32_t& x, uint64_t& w, uint64_t wp,
                                       bool& bad)
{
    const uint32_t p = node_of(w);
    if (key_of(wp) >= key_of(w) && node_of(wp) != p) {   // keys must fall
        bad = true;
        return false;
    }
    if (wp < w) nodes[x] = wp;
    x = p;
    w = wp;
    return true;
}

// Roots of M nodes x[m] (words w[m] already loaded; only the chains whose bit
// is set in `live` are walked), one level of every unfinished chain per step so
// that the loads of all chains overlap.
template <int M>
__device__ void n_find_m(gptr<uint64_t> nodes, uint32_t n, uint32_t (&x)[M], uint64_t (&w)[M], uint32_t live,
                         bool& bad)
{
    for (uint32_t it = 0; it < UNITE_CAP; ++it) {
        bool done = true;
        uint64_t wp[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const bool walk = ((live >> m) & 1u) && node_of(w[m]) != x[m];
            if (walk && node_of(w[m]) >= n) {
                bad = true;
                return;
            }
            wp[m] = walk ? nodes[node_of(w[m])] : w[m];
            done &= !walk;
        }
        if (done) return;
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (((live >> m) & 1u) && node_of(w[m]) != x[m] && !n_step(nodes, n, x[m], w[m], wp[m], bad)) return;
    }
    bad = true;
}

// Every word in the forest, (key << 32) | p, is also the word node p holds
// while it is a root (a node's key is its own).  So a hook can name two roots
// by their words alone: hook(a, b) hangs the node of the larger word under the
// smaller with one atomicMin.  If that node was no longer a root, the atomic
// returns its current word, whose node is the parent it had meanwhile gained
// (and a smaller word stored by the atomic dropped that link), so the hook goes
// on with that word and the smaller one: no reload and no new walk, one round
// trip per attempt.  The larger word falls at every attempt, so the loop ends.
// Two hooks of one lane run in step so that their atomics overlap.
//
// Where all tiles of a lattice merge at the same time, the pieces of a large
// cluster first hang under their upper neighbours, in chains as long as the
// lattice has rows of tiles, and a hook that comes late climbs two of them one
// attempt at a time.  With BOTH it climbs both at once: beside the atomic on the
// larger root it reads the word of the smaller one and goes on from its parent.
// The read may be served by a cache, so that parent may be one it has left
// since; whoever dropped that link joins the two (as above), so it is of the
// same cluster in the end, and a smaller word in any case.  Only from the third
// attempt on: most hooks need no more than two, and the read makes an attempt
// longer (a sweep of small clusters by 0.3 to 1 us: launch_merge picks).
constexpr uint32_t CLIMB_FROM = 2;

template <bool BOTH>
__device__ void n_hook2(gptr<uint64_t> nodes, uint32_t n, uint64_t (&a)[2], uint64_t (&b)[2], bool& bad)
{
    for (uint32_t it = 0; it < UNITE_CAP; ++it) {
        bool done = true;
        uint64_t old[2], hi[2], lo[2], up[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            hi[m] = max(a[m], b[m]);
            lo[m] = min(a[m], b[m]);
            up[m] = lo[m];
        }
        if (BOTH && it >= CLIMB_FROM) {
            // no branch of their own: the loads and the atomics fly together
#pragma unroll
            for (int m = 0; m < 2; ++m)
                up[m] = __hip_atomic_load(nodes + min(node_of(lo[m]), n - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const bool act = hi[m] != lo[m];
            if (act && node_of(hi[m]) >= n) {
                bad = true;
                return;
            }
            old[m] = act ? min_coherent64(nodes + node_of(hi[m]), lo[m]) : hi[m];
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            a[m] = old[m] == hi[m] ? lo[m] : old[m];
            b[m] = BOTH && old[m] != hi[m] ? min(lo[m], up[m]) : lo[m];
            done &= old[m] == hi[m];
        }
        if (done) return;
    }
    bad = true;
}

// ------------------------------------------------------------ spin staging
// Spins of a tile and its halo in LDS: rows 0..h (row h is the row below the
// tile, periodic), columns 0..w-1 plus column w = the column right of the tile
// (periodic).  Row stride SPW bytes.
//
// A thread loads four columns of a few rows at once (a dword at any address:
// rows of a lattice whose size is no multiple of four start anywhere); the last
// word of a width that is no multiple of four is loaded from the row's last
// four columns and shifted.  Every load is issued before the first store: the
// wave waits for memory once, where a load and its store row by row waited once
// a row (23 % of a wave's life at 64-row tiles, L = 16384).
template <int TY, uint32_t NT>
__device__ __forceinline__ void stage_spins(uint8_t* sp, const LatDesc& d, const TileGeom& g, uint32_t tid)
{
    typedef uint32_t __attribute__((aligned(1))) any_u32;
    const uint32_t L = d.L, w = g.w, h = g.h;
    const uint32_t yb = (g.y0 + h == L) ? 0u : g.y0 + h;          // row below the tile
    const uint32_t xh = (g.x0 + w == L) ? 0u : g.x0 + w;          // column right of the tile
    const gptr<const uint8_t> s = glb(d.s);
    const gptr<const uint8_t> tile0 = s + (size_t)g.y0 * L + g.x0;
    constexpr uint32_t HB = (TY + NT) / NT;                       // halo bytes per thread
    uint8_t hb[HB];
#pragma unroll
    for (uint32_t k = 0; k < HB; ++k) {
        const uint32_t r = min(tid + k * NT, h);
        hb[k] = s[(size_t)(r < h ? g.y0 + r : yb) * L + xh];
    }
    if (w >= 4) {
        constexpr uint32_t PER = TY * 16 / NT;                    // words per thread
        const uint32_t c = tid & 15u, r0 = tid >> 4;
        const uint32_t col = min(4 * c, w - 4), sh = 8u * (4 * c - col);   // (sh >= 32: no such word)
        uint32_t v[PER], vb;
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k)
            v[k] = *reinterpret_cast<gptr<const any_u32>>(tile0 + (size_t)min(r0 + k * (NT / 16), h - 1) * L + col);
        vb = *reinterpret_cast<gptr<const any_u32>>(s + (size_t)yb * L + g.x0 + col);
        __builtin_amdgcn_sched_barrier(0);
        if (sh < 32) {
#pragma unroll
            for (uint32_t k = 0; k < PER; ++k) {
                const uint32_t r = r0 + k * (NT / 16);
                if (r < h) *reinterpret_cast<uint32_t*>(sp + r * SPW + 4 * c) = v[k] >> sh;
            }
            if (r0 == 0) *reinterpret_cast<uint32_t*>(sp + h * SPW + 4 * c) = vb >> sh;
        }
        // the halo column's byte may share a word with the last columns: it is
        // stored after them
        if (w & 3u) __syncthreads();
    } else {
        const uint32_t c = tid & 63u;
        for (uint32_t r = tid >> 6; r <= h; r += NT / 64)
            if (c < w) sp[r * SPW + c] = s[(size_t)(r < h ? g.y0 + r : yb) * L + g.x0 + c];
    }
#pragma unroll
    for (uint32_t k = 0; k < HB; ++k) {
        const uint32_t r = tid + k * NT;
        if (r <= h) sp[r * SPW + w] = hb[k];
    }
}

// State counts of the tile's sites from the staged spins, four at a time: for
// q <= 16 the counts of sites whose state has all the bits of m set, m = 1..15
// (population counts of the ands of the words' bit planes), into hist[m]; the
// states' own counts follow from those by inclusion and exclusion
// (states_of_subsets).  For q = 2 that is one and and one count per word, where
// counting each site in its lane took four instructions a site.  q > 16: one
// LDS atomic per site.  At most 16 sites per lane, so two counts fit a word.
template <int TY, uint32_t NT>
__device__ __forceinline__ void count_tile_states(const uint8_t* sp, const TileGeom& g, uint32_t q, uint32_t* hist,
                                                  uint32_t tid)
{
    static_assert(TY * TX / NT <= 16, "two counts per word");
    const uint32_t c = tid & 15u, lane = tid & 63u;
    const uint32_t nb = g.w > 4 * c ? min(4u, g.w - 4 * c) : 0u;   // columns of word c inside the tile
    const uint32_t one = nb ? 0x01010101u >> (8u * (4u - nb)) : 0u;
    auto words = [&](auto f) {
#pragma unroll
        for (uint32_t rr = 0; rr < (uint32_t)TY; rr += NT / 16) {
            const uint32_t r = rr + (tid >> 4);
            if (r < g.h) f(*reinterpret_cast<const uint32_t*>(sp + r * SPW + 4 * c));
        }
    };
    auto add = [&](uint32_t v, uint32_t m) {   // two counts (m, m + 1) of the wave
        const uint32_t n = wave_sum(v);
        if (lane == 0 && n) {
            atomicAdd(&hist[m], n & 0xFFFFu);
            if (n >> 16) atomicAdd(&hist[m + 1], n >> 16);
        }
    };
    if (q == 2) {
        uint32_t n1 = 0;
        words([&](uint32_t v) { n1 += (uint32_t)__popc(v & one); });
        add(n1, 1);
    } else if (q <= 4) {
        uint32_t n1 = 0, n2 = 0, n3 = 0;
        words([&](uint32_t v) {
            const uint32_t b0 = v & one, b1 = (v >> 1) & one;
            n1 += (uint32_t)__popc(b0);
            n2 += (uint32_t)__popc(b1);
            n3 += (uint32_t)__popc(b0 & b1);
        });
        add(n1 | (n2 << 16), 1);
        add(n3, 3);
    } else if (q <= 16) {
        uint32_t n[16] = {};
        words([&](uint32_t v) {
            uint32_t b[16];
            b[1] = v & one;
            b[2] = (v >> 1) & one;
            b[4] = (v >> 2) & one;
            b[8] = (v >> 3) & one;
#pragma unroll
            for (uint32_t m = 1; m < 16; ++m) {
                const uint32_t top = m & (0u - m);   // a single bit of m
                if (m != top) b[m] = b[top] & b[m ^ top];
                if (m < 8 || q > 8) n[m] += (uint32_t)__popc(b[m]);
            }
        });
        add(n[1] | (n[2] << 16), 1);
        add(n[3] | (n[4] << 16), 3);
        add(n[5] | (n[6] << 16), 5);
        add(n[7] | (n[8] << 16), 7);
        if (q > 8) {
            add(n[9] | (n[10] << 16), 9);
            add(n[11] | (n[12] << 16), 11);
            add(n[13] | (n[14] << 16), 13);
            add(n[15], 15);
        }
    } else {
        words([&](uint32_t v) {
            for (uint32_t j = 0; j < nb; ++j) {
                const uint32_t st = (v >> (8 * j)) & 0xFFu;
                if (st) atomicAdd(&hist[st], 1u);
            }
        });
    }
}

// Sites in state c >= 1 from the counts of count_tile_states.
__device__ __forceinline__ uint32_t states_of_subsets(const uint32_t* hist, uint32_t q, uint32_t c)
{
    if (q == 2 || q > 16) return hist[c];
    const uint32_t top = q <= 4 ? 4u : q <= 8 ? 8u : 16u;
    uint32_t n = 0;
    for (uint32_t m = c; m < top; ++m)
        if ((m & c) == c) n += (__popc(m ^ c) & 1) ? 0u - hist[m] : hist[m];
    return n;
}

// Add a workgroup's measurement into a ring record (NCOPY partial copies).
__device__ __forceinline__ int64_t* ring_record(const LatDesc& d, uint32_t sweep, uint32_t copy)
{
    return d.ring + ((size_t)(sweep % d.cap) * NCOPY + copy) * ring_stride(d.q);   // cast at the access
}

// Per-wave queue of pending unions (pairs of provisional labels, 16 bits
// each).  Row labelling never reads the union-find, so unions can wait and
// then run with every lane busy instead of one lane of a diverged wave.
// Union queue slots per wave (a two-row step queues at most 128); a little
// smaller for 128-row tiles so that three of their workgroups fit a CU's LDS.
template <int TY>
constexpr uint32_t qcap_of() { return TY == 128 ? 224u : 256u; }

struct UnionQueue {
    uint32_t* q;       // the wave's slots in LDS
    uint32_t n;        // wave-uniform fill
};

// Run the queued unions, one per lane.
__device__ __forceinline__ void drain(UnionQueue& uq, uint16_t* P, uint32_t lane, bool& bad)
{
    for (uint32_t j = lane; j < uq.n; j += 64) {
        const uint32_t e = lds_ld(&uq.q[j]);
        lds_union(P, e & 0xFFFFu, e >> 16, bad);
    }
    uq.n = 0;
}

// Queue the unions (a, b) of the lanes in `mask` where a != b (at most 64; the
// caller keeps at least 64 slots free).
__device__ __forceinline__ void enqueue(UnionQueue& uq, uint64_t mask, uint32_t a, uint32_t b)
{
    const uint64_t m = ballot(a != b) & mask;
    if (lane_in(m)) lds_st(&uq.q[uq.n + lanes_below(m)], a | (b << 16));
    uq.n = __builtin_amdgcn_readfirstlane(uq.n + popc64(m));
}

// Provisional labels of one tile row, Hoshen-Kopelman style.  hx: +x bonds
// inside the tile; V: +y bonds from the row above (0 on a strip's first row);
// lp: this lane's label of the row above.  Every run of +x bonds takes one
// label: the label above one of its +y bonds, or, with none, its first site
// (a new root).  The runs are numbered from the left, and one LDS slot
// per run carries the choice to all its sites.  Any further +y bond into the
// run from a differently labelled site queues a union.  Every site's own
// union-find entry points at its label (itself for a new root), so the forest
// spans all sites and no separate array of provisional labels is kept.
// Vector instructions bound the kernel (scalar ones issue beside them), so what
// can be a mask is one: stores are masked by the lanes that have something to
// store rather than sent to a scratch slot.
__device__ __forceinline__ uint32_t row_labels(uint16_t* P, uint32_t* rl, UnionQueue& uq, uint32_t fresh,
                                               uint64_t validm, uint64_t hx, uint64_t V, uint64_t hprev, uint32_t lp)
{
    const uint64_t C = hx << 1;                 // bit x: bond (x-1) -> x
    const uint64_t S = ~C & validm;             // first sites of runs (site 0 always is one)
    // run index of x: the sites left of x whose +x bond is missing
    uint32_t* const slot = &rl[lanes_below(~hx)];
    // lanes talk through the slots, so these accesses must not be folded away;
    // a run's first site offers itself and every +y bond offers the label
    // above, in one store: any offer may win (unions below cover the rest)
    const uint32_t offer = lane_in(V) ? lp : fresh;
    if (lane_in(S | V)) lds_st(slot, offer);
    const uint32_t lab = lds_ld(slot);
    lds_set(P, fresh, lab);   // columns outside the tile write entries no one reads
    // bonds x-1 and x from the same run above into the same run here add nothing
    const uint64_t R = (V & C) & ((V & hprev) << 1);
    enqueue(uq, V & ~R, lp, lab);
    return lab;
}

}  // namespace

#ifdef SW_PHASE_CLOCKS
// Phase-clock tables of the profiling build: [kernel][NCOPY][PHASES + 1], the
// kernels being the bond-and-label kernel (Potts), the merge, the flip
// (Potts), the labelling of preset bonds and the flip that reflects (XY).
constexpr uint32_t PHASE_KERNELS = 5;
static __device__ unsigned long long g_phase_table[PHASE_KERNELS * NCOPY * (PHASES + 1)];
__device__ __forceinline__ unsigned long long* phase_table(uint32_t kernel)
{
    return g_phase_table + (size_t)kernel * NCOPY * (PHASES + 1);
}

// Profiling builds only (C linkage, so the namespace does not matter): the
// phase-clock tables summed over their rows into
// host [PHASE_KERNELS][PHASES + 1] (ticks per phase, then waves), and cleared
// when `clear` is nonzero.  Synchronises the device.
extern "C" int sw_phase_clocks(unsigned long long* host, int clear)
{
    static unsigned long long t[PHASE_KERNELS * NCOPY * (PHASES + 1)];
    if (hipDeviceSynchronize() != hipSuccess) return -1;
    if (hipMemcpyFromSymbol(t, HIP_SYMBOL(g_phase_table), sizeof(t)) != hipSuccess) return -1;
    for (uint32_t k = 0; k < PHASE_KERNELS; ++k)
        for (uint32_t i = 0; i <= PHASES; ++i) {
            unsigned long long sum = 0;
            for (uint32_t c = 0; c < NCOPY; ++c) sum += t[(k * NCOPY + c) * (PHASES + 1) + i];
            host[k * (PHASES + 1) + i] = sum;
        }
    if (clear) {
        for (auto& v : t) v = 0;
        if (hipMemcpyToSymbol(HIP_SYMBOL(g_phase_table), t, sizeof(t)) != hipSuccess) return -1;
    }
    return 0;
}
#endif

// ---------------------------------------------------------------------------
// Bonds + tile-local labels (+ measurement of the incoming configuration).
//
// Each wave owns a strip of TY/NW consecutive rows and labels it two rows at a
// time; strips are then stitched along their seams through the same LDS
// union-find, which always hangs the larger label under the smaller, so the
// final label of every tile-local cluster is its smallest site.
//
// Random words: with L even, one Philox call serves the pair of sites
// (2m, 2m+1) of one row; lane 2m draws for row r and lane 2m+1 for row r+1,
// and the two lanes swap the halves the other one needs.
//
// What bounds it: vector issue (1300 instructions a wave of 16 rows at eight
// waves a SIMD, about four cycles each; 8 x 88 of them the row loop, of which
// Philox 37).  L = 16384, q = 2 at K_c: 0.575 ms (0.74 with 1870 vector
// instructions, loads staged row by row and paths split at every step of a find;
// 0.66 with 1580, before the edge sites were taken one a thread and the forest
// held byte offsets).
//
// flags bit 0: also measure the configuration the bonds are drawn on (the
// result of the previous sweep, t - 1).
// PRESET: the bonds are already in the bond plane (drawn by the XY model's own
// kernel); the kernel then only labels, and measures nothing.
template <int TY, uint32_t NW, bool PRESET = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(8))) void k_bond_label(const LatDesc* descs, const WorkItem* map, uint32_t k,
                                                   uint32_t flags)
{
    constexpr uint32_t NT = 64 * NW;
    constexpr uint32_t RPW = TY / NW;  // rows per wave (even)
    static_assert(RPW % 2 == 0, "rows are labelled two at a time");
    constexpr uint32_t QCAP = qcap_of<TY>();
    __shared__ __align__(16) uint16_t P[TY * TX];   // union-find over the tile's sites
    __shared__ __align__(16) uint8_t sp[(TY + 1) * SPW];
    __shared__ uint64_t rb[TY][2];     // per row: +x bond word, +y bond word
    // per wave: the label of every run of a row; once a wave has left its
    // strip, its row holds the labels of the strip's last row (the seam)
    __shared__ uint32_t RL[NW][64];
    uint32_t(*const seam)[64] = RL;
    __shared__ uint32_t UQ[NW][QCAP];  // per wave: pending unions
    __shared__ uint32_t hist[256];
    __shared__ uint32_t tot[3];        // unequal pairs, active bonds, edge-forest nodes

    LatDesc d;
    uint32_t tile, lat;
    if (!pick(descs, map, blockIdx.x, true, d, tile, lat)) return;
    SW_PHASE_START(pc);
    const TileGeom g = tile_geom(d, tile, TY);
    const uint32_t t = *glb(d.counter) + k;
    const bool meas = !PRESET && d.cap != 0;
    const bool meas_prev = meas && (flags & 1u);
    const uint32_t tid = threadIdx.x, wave = wave_id(), lane = tid & 63u;
    const uint32_t L = d.L, w = g.w, h = g.h, x0 = g.x0, y0 = g.y0;

    if (tid < 256) hist[tid] = 0;
    if (tid < 3) tot[tid] = 0;
    uint64_t preset[2] = {0ull, 0ull};   // PRESET: lane k holds row r0 + k's bond words
    if constexpr (PRESET) {
        const gptr<const uint64_t> bin = glb(d.bonds) + (size_t)tile * 2 * TY;
        const uint32_t r = wave * RPW + lane;
        if (lane < RPW) {
            if (r < h) {
                preset[0] = bin[r];
                preset[1] = bin[TY + r];
            }
            rb[r][0] = preset[0];
            rb[r][1] = preset[1];
        }
    } else {
        stage_spins<TY, NT>(sp, d, g, tid);
    }
    __syncthreads();
    SW_PHASE(pc, 0);   // staging
    if (meas_prev) count_tile_states<TY, NT>(sp, g, d.q, hist, tid);

    const uint32_t x = lane;
    const bool vx = x < w;
    const uint64_t validm = (w == 64) ? ~0ull : ((1ull << w) - 1ull);
    const uint64_t cross = 1ull << (w - 1);   // the +x bond of column w-1 leaves the tile
    const uint32_t r0 = wave * RPW, r1 = min(h, r0 + RPW);
    const uint64_t bondm = d.thr_nz ? validm : 0ull;   // K = 0: no bond at all
    const bool even_L = (L & 1u) == 0;
    uint32_t* rl = RL[wave];
    UnionQueue uq{UQ[wave], 0u};
    uint32_t n_eq = 0;   // equal-spin pairs of the strip (wave-uniform)
    uint32_t lp = 0;
    const PhiloxKeys ks = philox_keys_v(d.key0, d.key1);
    bool bad = false;   // this lane met a corrupted forest
    uint64_t hprev = 0, vprev = 0;

    // Full strips of full-width tiles (K > 0), the common case: no lane or row
    // masks, always two rows, one Philox call per lane and pass, the bond words
    // gathered into lanes (one row per lane) and stored once per strip.
    // ODD: L is odd.  Row r then starts at an even site index (y0 + r and x0 are
    // even) and row r+1 at an odd one, so the pairs of row r are the columns
    // (2m, 2m+1) and those of row r+1 the columns (2m+1, 2m+2): an even lane
    // draws for row r, an odd lane for row r+1, and either way the pair's second
    // half belongs to the lane on the right.  Column 0 of row r+1 is the second
    // half of a pair that starts left of the tile; lane k draws it for pass k
    // before the loop.  (Two calls per lane and pass, as for ragged tiles below,
    // cost an odd lattice a third: 32 uneven lattices, half of them odd, 237 us
    // a labelling against 171 at the even lattices' rate.)
    auto full_rows = [&](auto odd_tag) {
        constexpr bool ODD = decltype(odd_tag)::value;
        uint32_t words[4] = {0u, 0u, 0u, 0u};   // lane k holds row r0 + k's bond words
        const bool odd = x & 1u;
        // site indices in 32 bits: exact for every row of the lattice (N <= 2^32)
        const uint32_t base = (y0 + r0) * L + x0;
        const uint32_t pair = ODD ? ((odd ? base + L : base) >> 1) + ((x + 1u) >> 1)
                                  : ((odd ? base + L : base) + (x & ~1u)) >> 1;
        uint64_t m0 = PHILOX_M0 * pair;
        const uint64_t m0_step = PHILOX_M0 * L;   // two rows on, pairs are L further
        uint32_t ez = 0, ew = 0;
        if constexpr (ODD) {
            const u32x4 e = philox4x32_10((base + (2u * min(lane, RPW / 2 - 1u) + 1u) * L) >> 1, 0u, t, 0u, ks);
            ez = e.z;
            ew = e.w;
        }
#pragma unroll 1
        for (uint32_t k = 0; k < RPW; k += 2) {
            const uint32_t r = r0 + k;
            if (uq.n > QCAP - 128) drain(uq, P, lane, bad);
            const uint8_t* row = sp + r * SPW;
            const uint32_t s0 = row[x], s0r = row[x + 1];
            const uint32_t s1 = row[SPW + x], s1r = row[SPW + x + 1];
            const uint32_t s2 = row[2 * SPW + x];
            const u32x4 q4 = philox4x32_10_from(m0, t, 0u, ks);
            m0 += m0_step;
            uint32_t wx0, wy0, wx1, wy1;
            if constexpr (ODD) {
                // the left lane's second half; lane 0 the one drawn ahead
                const uint32_t lz = (uint32_t)__builtin_amdgcn_update_dpp(__builtin_amdgcn_readlane((int)ez, (int)(k / 2)),
                                                                          (int)q4.z, 0x138, 0xF, 0xF, false);   // wave_shr:1
                const uint32_t lw = (uint32_t)__builtin_amdgcn_update_dpp(__builtin_amdgcn_readlane((int)ew, (int)(k / 2)),
                                                                          (int)q4.w, 0x138, 0xF, 0xF, false);
                wx0 = odd ? lz : q4.x;
                wy0 = odd ? lw : q4.y;
                wx1 = odd ? q4.x : lz;
                wy1 = odd ? q4.y : lw;
            } else {
                const uint32_t recv0 = swap_pair(odd ? q4.x : q4.z);
                const uint32_t recv1 = swap_pair(odd ? q4.y : q4.w);
                wx0 = odd ? recv0 : q4.x;
                wy0 = odd ? recv1 : q4.y;
                wx1 = odd ? q4.z : recv0;
                wy1 = odd ? q4.w : recv1;
            }
            // equal-spin masks and draw masks as wave ballots; a bond needs both
            const uint64_t EX0 = ballot(s0 == s0r), EY0 = ballot(s0 == s1);
            const uint64_t EX1 = ballot(s1 == s1r), EY1 = ballot(s1 == s2);
            const uint64_t BX0 = EX0 & ballot(wx0 <= d.thr_m1), BY0 = EY0 & ballot(wy0 <= d.thr_m1);
            const uint64_t BX1 = EX1 & ballot(wx1 <= d.thr_m1), BY1 = EY1 & ballot(wy1 <= d.thr_m1);
            n_eq += popc64(EX0) + popc64(EY0) + popc64(EX1) + popc64(EY1);
            write_rows(words, k, BX0, BY0, BX1, BY1);

            const uint64_t hx0 = BX0 & ~cross, hx1 = BX1 & ~cross;
            const uint32_t fresh = 2 * (r * TX + x);
            lp = row_labels(P, rl, uq, fresh, ~0ull, hx0, vprev, hprev, lp);
            lp = row_labels(P, rl, uq, fresh + 2 * TX, ~0ull, hx1, BY0, hx0, lp);
            hprev = hx1;
            vprev = BY1;
        }
        if (lane < RPW) {
            rb[r0 + lane][0] = ((uint64_t)words[1] << 32) | words[0];
            rb[r0 + lane][1] = ((uint64_t)words[3] << 32) | words[2];
        }
    };
    // Ragged tiles and K = 0: masks for the columns and rows outside, one Philox
    // call per row and lane where L is odd.
    auto ragged_rows = [&]() {
#pragma unroll 1
        for (uint32_t r = r0; r < r1; r += 2) {
            const bool two = r + 1 < r1;
            if (uq.n > QCAP - 128) drain(uq, P, lane, bad);
            const uint8_t* row = sp + r * SPW;
            const uint32_t s0 = row[x], s0r = row[x + 1];
            const uint32_t s1 = row[SPW + x], s1r = row[SPW + x + 1];
            const uint32_t s2 = two ? row[2 * SPW + x] : 0u;

            // a draw for row r+1 past the last row wraps but is never used
            const uint32_t base0 = (y0 + r) * L + x0;
            uint32_t wx0, wy0, wx1, wy1;
            if (even_L) {
                const bool odd = x & 1u;
                const uint32_t pair = ((odd ? base0 + L : base0) + (x & ~1u)) >> 1;
                const u32x4 q4 = philox4x32_10(pair, 0u, t, 0u, ks);
                const uint32_t recv0 = swap_pair(odd ? q4.x : q4.z);
                const uint32_t recv1 = swap_pair(odd ? q4.y : q4.w);
                wx0 = odd ? recv0 : q4.x;
                wy0 = odd ? recv1 : q4.y;
                wx1 = odd ? q4.z : recv0;
                wy1 = odd ? q4.w : recv1;
            } else {
                const uint32_t ga = base0 + x, gb = base0 + L + x;
                const u32x4 qa = philox4x32_10(ga >> 1, 0u, t, 0u, ks);
                const u32x4 qb = philox4x32_10(gb >> 1, 0u, t, 0u, ks);
                wx0 = (ga & 1u) ? qa.z : qa.x;
                wy0 = (ga & 1u) ? qa.w : qa.y;
                wx1 = (gb & 1u) ? qb.z : qb.x;
                wy1 = (gb & 1u) ? qb.w : qb.y;
            }
            const uint64_t EX0 = ballot(s0 == s0r) & validm, EY0 = ballot(s0 == s1) & validm;
            const uint64_t BX0 = EX0 & ballot(wx0 <= d.thr_m1) & bondm;
            const uint64_t BY0 = EY0 & ballot(wy0 <= d.thr_m1) & bondm;
            uint64_t EX1 = 0, EY1 = 0, BX1 = 0, BY1 = 0;
            if (two) {
                EX1 = ballot(s1 == s1r) & validm;
                EY1 = ballot(s1 == s2) & validm;
                BX1 = EX1 & ballot(wx1 <= d.thr_m1) & bondm;
                BY1 = EY1 & ballot(wy1 <= d.thr_m1) & bondm;
            }
            n_eq += popc64(EX0) + popc64(EY0) + popc64(EX1) + popc64(EY1);
            if (lane == 0) {
                rb[r][0] = BX0;
                rb[r][1] = BY0;
                if (two) {
                    rb[r + 1][0] = BX1;
                    rb[r + 1][1] = BY1;
                }
            }

            const uint64_t hx0 = BX0 & ~cross;
            const uint32_t fresh = 2 * (r * TX + x);
            lp = row_labels(P, rl, uq, fresh, validm, hx0, vprev, hprev, lp);
            hprev = hx0;
            vprev = BY0;
            if (two) {
                const uint64_t hx1 = BX1 & ~cross;
                lp = row_labels(P, rl, uq, fresh + 2 * TX, validm, hx1, vprev, hprev, lp);
                hprev = hx1;
                vprev = BY1;
            }
        }
    };
    // the same row labelling over bond words that are there already
    auto preset_rows = [&]() {
        for (uint32_t r = r0; r < r1; ++r) {
            if (uq.n > QCAP - 64) drain(uq, P, lane, bad);
            const uint64_t hx = lane_value64(preset[0], r - r0) & ~cross;
            lp = row_labels(P, rl, uq, 2 * (r * TX + x), validm, hx, vprev, hprev, lp);
            hprev = hx;
            vprev = lane_value64(preset[1], r - r0);
        }
    };
    const bool full = w == TX && r1 - r0 == RPW && d.thr_nz;
    if constexpr (PRESET) preset_rows();
    else if (full && even_L) full_rows(std::false_type{});
    else if (full) full_rows(std::true_type{});
    else ragged_rows();
    SW_PHASE(pc, 1);   // rows: draws, ballots, row labels, queue drains, equal pairs
    seam[wave][lane] = lp;
    // every site of the strip owns two bonds
    if (meas_prev && lane == 0 && r0 < r1) atomicAdd(&tot[0], 2u * w * (r1 - r0) - n_eq);
    SW_PHASE(pc, 2);   // measurement sums of the strip
    __syncthreads();
    SW_PHASE(pc, 3);   // barrier

    // Seams: +y bonds from the last row of the strip above into this strip.
    if (wave > 0 && r0 < h) {
        const uint32_t ru = r0 - 1;
        const uint64_t V = rb[ru][1];
        const uint64_t hu = rb[ru][0] & ~cross, hc = rb[r0][0] & ~cross;
        const uint64_t R = V & (V << 1) & (hc << 1) & (hu << 1);
        const uint32_t up = seam[wave - 1][lane];
        // the site's entry is its label or, after path halving, an ancestor of it
        const uint32_t first_prov = lds_get(P, 2 * (r0 * TX + x));
        if (uq.n > QCAP - 64) drain(uq, P, lane, bad);
        enqueue(uq, V & ~R, up, first_prov);
    }
    drain(uq, P, lane, bad);
    SW_PHASE(pc, 4);   // seams and the last drain

    // Tile record: bond words (tile-major), crossing-bond masks.
    gptr<uint32_t> rec = glb(d.edges) + (size_t)tile * edge_words(TY);
    gptr<uint64_t> bw = glb(d.bonds) + (size_t)tile * 2 * TY;
    for (uint32_t j0 = 0; j0 < 2 * TY; j0 += NT) {
        const uint32_t j = j0 + tid, r = j % TY;
        const uint64_t word = (j < 2 * TY && r < h) ? rb[r][j / TY] : 0ull;
        if (!PRESET && j < 2 * TY && r < h) bw[j] = word;
        if (meas) {
            const uint32_t n = wave_sum(popc64(word));   // active bonds
            if (lane == 0 && n) atomicAdd(&tot[1], n);
        }
    }
    if (wave == 0) {
        for (uint32_t j = 0; j < TY; j += 64) {
            const uint32_t r = j + lane;
            const bool bit = r < h && ((rb[r][0] >> (w - 1)) & 1ull);
            const uint64_t m = ballot(bit);
            if (lane == 0) {
                rec[j / 32] = (uint32_t)m;
                rec[j / 32 + 1] = (uint32_t)(m >> 32);
            }
        }
        if (lane == 0) {
            if (TY < 128) {
                rec[2] = 0;
                rec[3] = 0;
            }
            const uint64_t b = rb[h - 1][1];
            rec[4] = (uint32_t)b;
            rec[5] = (uint32_t)(b >> 32);
        }
    }
    __syncthreads();
    SW_PHASE(pc, 5);   // bond words out, edge record, barrier

    // Edge sites find their tile-local roots, one a thread, in the order of the
    // edge record's slots (a tile has no more of them than threads; with the left
    // and right sites of a strip taken by its own wave, and the top and bottom
    // rows by the first and last, the waves walked up to four times each with
    // mostly idle lanes: 0.658 ms a labelling against 0.626, L = 16384).
    // The first lane to reach a root claims it as a node of the tile's edge
    // forest: it takes the next slot (in no particular order: a node's word
    // carries its key), writes the node's word (a root of its own, keyed by its
    // site index) and makes the root's LDS entry ROOT16 + 2 (slot + 1), which halved
    // like an offset, as a signed number, is NODE16 + slot: that the labels
    // and the edge record carry on.  One wave claims while others still walk: only
    // roots are ever tagged, and a walk that meets a tagged entry stops there, at
    // the root it was looking for.
    // a site index fits 32 bits (N <= 2^32) and y, L fit 24 bits
    auto global_index = [&](uint32_t la) { return __umul24(y0 + la / TX, L) + x0 + la % TX; };
    const uint32_t node0 = tile * nslot(TY);
    auto edge_root = [&](uint32_t at) {
        uint32_t p = lds_get(P, at);
        while (!(p & ROOT16) && p < at) {
            at = p;
            p = lds_get(P, at);
        }
        bad |= !(p & ROOT16) && p != at;
        return at;
    };
    // A claim of root r sets the ROOT16 bit of its entry with one LDS atomic
    // OR on the entry's 32-bit word: the lane that finds the bit clear is the
    // first and wins; an entry tagged already keeps its value (a slot stored
    // by another winner is never overwritten).  Then the wave's winners take
    // consecutive slots with one LDS atomic and make their roots' entries
    // ROOT16 + 2 (slot + 1).
    auto claim = [&](bool want, uint32_t r) {
        if (!want) return false;
        const uint32_t sh = (r & 2u) * 8u;
        const uint32_t old = atomicOr(reinterpret_cast<uint32_t*>(lds_entry(P, r & ~3u)), ROOT16 << sh);
        return ((old >> sh) & 0xFFFFu) == r;
    };
    static_assert(nslot(TY) <= NT, "one thread per edge site");
    uint32_t site = 0, root = 0;
    bool edge = false;
    if (wave * 64 < nslot(TY)) {
        if (tid < 2 * TY) {
            const uint32_t r = tid < TY ? tid : tid - TY;
            edge = r < h;
            site = r * TX + (tid < TY ? w - 1 : 0u);
        } else {
            const uint32_t c = (tid - 2 * TY) % TX;
            edge = c < w && tid < nslot(TY);
            site = (tid < 2 * TY + TX ? (h - 1) * TX : 0u) + c;
        }
        if (edge) root = edge_root(2 * site);
        const bool won = claim(edge, root);
        const uint64_t m = ballot(won);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(&tot[2], popc64(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (won) {
            const uint32_t slot = base + lanes_below(m);
            glb(d.nodes)[node0 + slot] = ((uint64_t)global_index(root >> 1) << 32) | (node0 + slot);
            if (!PRESET && d.csize) glb(d.csize)[node0 + slot] = 0;   // for the flip to gather in
            lds_set(P, root, ROOT16 + 2 * (slot + 1));
        }
    }
    __syncthreads();
    SW_PHASE(pc, 6);   // edge roots, node claims, barrier
    if (tid == 0) rec[6] = tot[2];   // nodes of the tile

    // Tile labels out (16 bits), per site: the tile-local index of its
    // union-find grandparent (a smaller site of its tile-local cluster; the
    // flip follows these pointers inside the tile), or, for a tile-local root,
    // ROOT16 or NODE16 + its slot (the entry halved: see above).  A grandparent that is a node is not
    // copied (its entry carries a slot, not an index): the parent is.  Tagged
    // entries are larger than every index, so two minima do it: the entry of
    // min(entry, own index) (its own entry again for a root), then the smaller
    // of the two entries; a root inside the tile ends at its own index.
    // Entries of columns outside the tile are never stored (full-width tiles,
    // the common case, need no mask at all).
    auto halved = [](uint32_t entry) { return (uint16_t)((int16_t)entry >> 1); };
    auto out_label = [&](uint32_t at, uint32_t p, uint32_t gp) {
        return p == at ? (uint16_t)ROOT16 : halved(min(p, gp));
    };
    if (w == TX && r1 - r0 == RPW) {
        // a full strip: all parent reads first, then all grandparent reads, so
        // the LDS round trips overlap; each row is stored from its own
        // wave-uniform (scalar) base, the lane's column as the only vector part
        uint32_t p[RPW], gp[RPW];
#pragma unroll
        for (uint32_t k = 0; k < RPW; ++k) p[k] = P[(r0 + k) * TX + x];   // (16-bit entries)
#pragma unroll
        for (uint32_t k = 0; k < RPW; ++k) gp[k] = *lds_entry(P, min(p[k], 2 * ((r0 + k) * TX + x)));
        gptr<uint16_t> out = glb(d.tlab) + (size_t)(y0 + r0) * L + x0 + x;   // this lane's site, row by row
#pragma unroll
        for (uint32_t k = 0; k < RPW; ++k, out += L) {
            const uint32_t at = 2 * ((r0 + k) * TX + x);
            *out = out_label(at, p[k], gp[k]);
        }
    } else if (vx) {
        for (uint32_t r = r0; r < r1; ++r) {
            const uint32_t at = 2 * (r * TX + x), p = P[r * TX + x];
            glb(d.tlab)[(size_t)(y0 + r) * L + x0 + x] = out_label(at, p, *lds_entry(P, min(p, at)));
        }
    }
    SW_PHASE(pc, 7);   // tile labels out
    // The edge record's slots, for the merge.
    if (edge) ((gptr<uint16_t>)(rec + 8))[tid] = halved(*lds_entry(P, root)) - NODE16;
    if (bad) flag_error(d.err);

    // the workgroup's sums into the ring, by wave 0 alone (the slot's modulo is
    // scalar work the other waves need not repeat)
    if (meas && wave == 0) {
        const uint32_t copy = blockIdx.x % NCOPY;
        const uint32_t slot = t % d.cap, prev = slot ? slot - 1u : d.cap - 1u;
        int64_t* const rc = d.ring + ((size_t)slot * NCOPY + copy) * ring_stride(d.q);
        if (lane == 0) atomic_add_i64(&rc[1], tot[1]);
        if (meas_prev) {
            int64_t* const rp = d.ring + ((size_t)prev * NCOPY + copy) * ring_stride(d.q);
            if (lane == 0) atomic_add_i64(&rp[0], tot[0]);
            for (uint32_t c = lane; c < d.q; c += 64) {
                const uint32_t n = c ? states_of_subsets(hist, d.q, c) : 0u;
                if (n) atomic_add_i64(&rp[1 + c], n);
            }
        }
    }
    SW_PHASE(pc, 8);   // slots, ring sums
    SW_PHASE_FLUSH(pc, phase_table(PRESET ? 3u : 0u));
}

// ---------------------------------------------------------------------------
// Join tile-local clusters across tile edges.  One wave per tile handles the
// crossing bonds of its right and bottom edges (periodic neighbours): each
// joins the edge-forest nodes of the two sites' tile-local roots.
//
// bump: sweeps to advance each lattice's counter by (0: leave it), done by the
// wave of its tile 0, which also notes the labels' form.  This kernel alone does not read the counter, so a
// step's graph needs no launch of its own to move on to the next sweep; the
// kernels after it in the step see the counter already moved.
template <int TY, bool BOTH>
__global__ __launch_bounds__(256) void k_merge(const LatDesc* descs, const WorkItem* map, uint32_t nitems, uint32_t bump)
{
    const uint32_t wave = wave_id(), lane = threadIdx.x & 63u;
    const uint32_t idx = blockIdx.x * 4 + wave;
    __shared__ uint8_t pairs[4][2][256];
    if (idx >= nitems) return;
    LatDesc d;
    uint32_t tile, lat;
    if (!pick(descs, map, idx, false, d, tile, lat)) return;
    SW_PHASE_START(pc);
    if (bump && tile == 0 && lane == 0) {
        *glb(d.counter) += bump;
        *glb(d.labels) = LABELS_TILE;
    }
    const TileGeom g = tile_geom(d, tile, TY);
    const uint32_t EW = edge_words(TY), NS = nslot(TY);
    const uint32_t n = d.ntiles * NS;
    const uint32_t t_right = g.ty * d.ntx + ((g.tx + 1 == d.ntx) ? 0u : g.tx + 1);
    const uint32_t t_below = ((g.ty + 1 == d.nty) ? 0u : g.ty + 1) * d.ntx + g.tx;
    const gptr<uint32_t> rec = glb(d.edges) + (size_t)tile * EW;
    const gptr<const uint16_t> sl = (gptr<const uint16_t>)(rec + 8);
    const gptr<const uint16_t> slR = (gptr<const uint16_t>)(glb(d.edges) + (size_t)t_right * EW + 8);
    const gptr<const uint16_t> slB = (gptr<const uint16_t>)(glb(d.edges) + (size_t)t_below * EW + 8);
    const gptr<uint64_t> nodes = glb(d.nodes);

    // Lane l takes the crossing bond of row l of the right edge (row l of the
    // right neighbour's left column) and of column l of the bottom edge
    // (column l of the top row of the tile below); crossing bonds between the
    // same two clusters are joined once: every hook is an atomic at memory, and
    // those at one address wait for each other (at q = 2, K_c, dropping equal
    // pairs that are not neighbours too takes the kernel from 0.141 to 0.131 ms
    // at L = 16384, from 0.074 to 0.063 at 8192).  The nodes' words are all
    // loaded before the first union, so their round trips overlap.
    bool bad = false;
    uint32_t pa = INVALID, pb = INVALID;
    for (uint32_t j = 0; j < TY; j += 64) {
        const uint32_t r = j + lane, x = lane;
        // the crossing bits and the slots at both ends of every edge site are
        // loaded together (all inside the records; slots of sites without a
        // crossing bond are not used)
        const uint32_t wr = rec[r >> 5], wb = rec[4 + (x >> 5)];
        const uint32_t sa1 = sl[r], sb1 = slR[TY + r];
        const uint32_t sa2 = sl[2 * TY + x], sb2 = slB[2 * TY + TX + x];
        const bool right = r < g.h && ((wr >> (r & 31u)) & 1u);
        const bool below = j == 0 && x < g.w && ((wb >> (x & 31u)) & 1u);
        SW_PHASE(pc, 0);   // edge record and slots
        uint32_t a1 = INVALID, b1 = INVALID, a2 = INVALID, b2 = INVALID;
        if (right) {
            a1 = tile * NS + sa1;
            b1 = t_right * NS + sb1;
        }
        if (below) {
            a2 = tile * NS + sa2;
            b2 = t_below * NS + sb2;
        }
        uint32_t ua = __shfl_up(a1, 1), ub = __shfl_up(b1, 1);
        uint32_t va = __shfl_up(a2, 1), vb = __shfl_up(b2, 1);
        if (lane == 0) {
            ua = pa;
            ub = pb;
            va = INVALID;
            vb = INVALID;
        }
        pa = __shfl(a1, 63);
        pb = __shfl(b1, 63);
        bool u1 = right && !(ua == a1 && ub == b1) && a1 < n && b1 < n;
        bool u2 = below && !(va == a2 && vb == b2) && a2 < n && b2 < n;
        // lanes further apart: the last lane of a table slot's pairs stands for
        // those equal to its own
        {
            const uint32_t k1 = sa1 | (sb1 << 16), k2 = sa2 | (sb2 << 16);
            uint8_t* const t1 = &pairs[wave][0][(k1 * 0x9E3779B1u) >> 24];
            uint8_t* const t2 = &pairs[wave][1][(k2 * 0x9E3779B1u) >> 24];
            // (other lanes' stores are read: these accesses must not be folded away)
            if (u1) __hip_atomic_store(t1, (uint8_t)lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (u2) __hip_atomic_store(t2, (uint8_t)lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const uint32_t w1 = u1 ? __hip_atomic_load(t1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : lane;
            const uint32_t w2 = u2 ? __hip_atomic_load(t2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : lane;
            // (by all lanes: a permute reads nothing from a lane that is masked off)
            const uint32_t q1 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(w1 * 4), (int)k1);
            const uint32_t q2 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(w2 * 4), (int)k2);
            u1 = u1 && (w1 == lane || q1 != k1);
            u2 = u2 && (w2 == lane || q2 != k2);
        }
        bad |= (right && !(a1 < n && b1 < n)) || (below && !(a2 < n && b2 < n));
        // both unions' four walks in step, then both hooks
        uint32_t xs[4] = {a1, b1, a2, b2};
        uint64_t ws[4] = {u1 ? nodes[a1] : 0ull, u1 ? nodes[b1] : 0ull, u2 ? nodes[a2] : 0ull, u2 ? nodes[b2] : 0ull};
        n_find_m<4>(nodes, n, xs, ws, (u1 ? 3u : 0u) | (u2 ? 12u : 0u), bad);
        SW_PHASE(pc, 1);   // node words, walks to the roots
        if (bad) break;
        uint64_t ha[2] = {ws[0], ws[2]}, hb[2] = {ws[1], ws[3]};
        n_hook2<BOTH>(nodes, n, ha, hb, bad);
        SW_PHASE(pc, 2);   // hooks
    }
    if (bad) flag_error(d.err);
    SW_PHASE_FLUSH(pc, phase_table(1u));
}

// ---------------------------------------------------------------------------
// Cluster-size sums of a sweep's clusters, for the improved estimators of the
// moments of the magnetisation (given the clusters, the mean of |M|^2 over the
// clusters' independent uniform states is sum |C|^2, and that of |M|^4 a
// combination of (sum |C|^2)^2 and sum |C|^4).  The flip takes them along: it
// walks every site to its tile-local root anyway.  |C| <= 2^30, so |C|^2 fits
// 64 bits and the sums of |C|^4 take 128 (two words, carried by hand).

// v added to the 128-bit number (lo, hi), atomically.
template <int SCOPE, class P>
__device__ __forceinline__ void add_u128(P lo, P hi, unsigned __int128 v)
{
    const unsigned long long vl = (unsigned long long)v, vh = (unsigned long long)(v >> 64);
    if (!vl && !vh) return;
    const unsigned long long old = __hip_atomic_fetch_add(lo, vl, __ATOMIC_RELAXED, SCOPE);
    const unsigned long long up = vh + ((old + vl) < old ? 1u : 0u);
    if (up) __hip_atomic_fetch_add(hi, up, __ATOMIC_RELAXED, SCOPE);
}

// The workgroup's sums (in LDS) into ring record t, partial copy 0.
__device__ __forceinline__ void cs_flush(const LatDesc& d, uint32_t t, const unsigned long long* sums)
{
    const gptr<unsigned long long> rec =
        (gptr<unsigned long long>)(glb(d.ring) + (size_t)(t % d.cap) * NCOPY * ring_stride(d.q) + cs_word(d.q));
    if (sums[0]) __hip_atomic_fetch_add(rec, sums[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    add_u128<__HIP_MEMORY_SCOPE_AGENT>(rec + 1, rec + 2, ((unsigned __int128)sums[2] << 64) | sums[1]);
}

// ---------------------------------------------------------------------------
// Flip: every site takes the state drawn for the smallest site index of its
// cluster.  Inside the tile the labels form a forest of tile-local indices
// whose terminals are the tile-local roots.  The tile's edge-forest nodes are
// loaded together at the start (node j by lane j / NW of wave j % NW) and
// search their roots (halving the paths they walk); then each wave draws, in
// compacted lanes, the states of its nodes (keyed by their roots) and of the
// roots of clusters inside the tile it found (keyed by their own sites).
// Wave w owns rows w, w+NW, w+2NW, ... (lane = column); its labels are all
// loaded first.  LDS entries are 16 bits (so more workgroups fit a CU): a
// tile-local index, NODE16 + slot for a node, ROOT16 | RES16 | state for a
// resolved root inside the tile.
// Bound by the latency of its loads at eight workgroups a CU (L = 16384, q = 2
// at K_c: 0.312 ms, 0.91 GB; 0.35 and 0.39 at seven and six workgroups; 14 % fewer
// vector instructions, node words a round trip earlier or wider label loads
// change nothing); the XY form by HBM (2.7 GB in 0.585 ms).
// XY: the draw per cluster is a reflection bit instead of a state, and each
// site of a reflected cluster has its angle reflected across the line
// perpendicular to the sweep's direction.  A lane takes four neighbouring columns
// of every fourth row, so that labels and angles move 8 and 16 bytes a lane
// (0.605 ms with a column a lane; four of them without a reflected site are not
// touched).  Potts gains nothing from that (0.308 ms against 0.306).
// CS: lattices with cluster sums also have the sites of each tile-local cluster
// counted as they are walked (a run of equal roots along a row adds its length
// with one LDS atomic).  A cluster inside the tile adds |C|^2 and |C|^4; a node
// adds its count c to its root's size with one returning atomic, and of the
// powers what it raises them by, (old + c)^2 - old^2 and (old + c)^4 - old^4:
// over a root's nodes these add up to the powers of its final size, whatever the
// order, so no launch after the flip has to visit the roots.  The 198 tiles of
// 36 replicas of L = 32 ... 256, q = 2 near K_c: 10.0 us a sweep for flip and
// sums, 24.1 with two kernels of their own after the flip (counts, then roots).
template <int TY, uint32_t NW, bool XY = false, bool CS = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(CS ? 4 : 8))) void k_flip(
    const LatDesc* descs, const WorkItem* map, uint32_t k)
{
    constexpr uint32_t NT = 64 * NW;
    constexpr uint32_t PER = TY / NW;       // sites per lane
    constexpr uint32_t W = XY ? 4 : 1;      // neighbouring columns per lane: W rows a step
    constexpr uint32_t STEPS = PER / W;
    static_assert(PER % W == 0, "whole steps");
    constexpr uint32_t RES16 = 0x2000u;     // a resolved root inside the tile
    constexpr uint32_t NKN = 512;           // node table (>= nslot(TY), a power of two)
    constexpr uint32_t NODE_ENTRY = 0x8000u;   // a list entry that names a node
    static_assert(nslot(TY) < NKN && nslot(TY) <= NT && nslot(TY) < RES16, "one thread per node");
    typedef uint64_t __attribute__((aligned(2))) any_u64;   // rows start at any multiple of an entry
    typedef uint32_t __attribute__((ext_vector_type(4), aligned(4))) any_u32x4;
    __shared__ __align__(8) uint16_t E[TY * TX];
    __shared__ uint16_t list[NW][PER * TX + 64 + 64];   // roots inside the tile, nodes, a scratch slot per lane
    __shared__ uint32_t NK[NKN];            // per node (slot + 1): its root's key, then its state
    // CS: sites per root inside the tile (by index), then per node (slot + 1), 16
    // bits each, two a word (a tile has at most 2^13 sites)
    static_assert(TY * TX < 65536, "a tile's sites are counted in 16 bits");
    __shared__ uint32_t C[CS ? (TY * TX + NKN) / 2 : 1];
    __shared__ uint32_t NR[CS ? NKN : 1];   // CS: per node (slot), its root
    __shared__ unsigned long long sums[3];

    LatDesc d;
    uint32_t tile, lat;
    if (!pick(descs, map, blockIdx.x, true, d, tile, lat)) return;
    SW_PHASE_START(pc);
    const TileGeom g = tile_geom(d, tile, TY);
    const uint32_t t = *glb(d.counter) + k;
    const uint32_t tid = threadIdx.x, wave = wave_id(), lane = tid & 63u;
    const uint32_t L = d.L, w = g.w, h = g.h, x0 = g.x0, y0 = g.y0;
    const uint32_t lr = lane / (TX / W), col = lane % (TX / W) * W;   // row of a step, first column
    uint16_t* my_list = list[wave];
    const uint32_t NS = nslot(TY), n_nodes = d.ntiles * NS, node0 = tile * NS;
    const gptr<uint64_t> nodes = glb(d.nodes);
    bool bad = false;

    // The tile's entries are addressed from one wave-uniform base with 32-bit
    // per-lane offsets (a tile spans fewer than 2^32 / 4 sites of the arrays):
    // one vector add per row, where a scalar base per row would cost the busier
    // scalar unit two 64-bit adds.  Step i of this wave covers rows
    // W (wave + NW i) + 0 ... W - 1.
    const uint32_t site0 = (W * wave + lr) * L + col;   // this lane's first site, from the tile origin
    const uint32_t wave_step = W * NW * L;              // sites between a lane's consecutive steps
    const gptr<const char> lab_tile = (gptr<const char>)(glb(d.tlab) + (size_t)y0 * L + x0);
    const gptr<char> s_tile = (gptr<char>)(glb(d.s) + (size_t)y0 * L + x0);
    // the tile's node count, by a vector load ahead of the labels': a scalar one
    // would be waited for before them
    uint32_t lane0 = 0;
    asm("" : "+v"(lane0));
    const uint32_t n_loaded = glb(d.edges)[(size_t)tile * edge_words(TY) + 6 + lane0];
    const bool count = CS && d.csize;
    if (count) {
        for (uint32_t i = tid; i < (TY * TX + NKN) / 2; i += NT) C[i] = 0;
        if (tid < 3) sums[tid] = 0;
    }
    // XY: the sweep's direction (wave-uniform)
    const uint32_t phi = XY ? __builtin_amdgcn_readfirstlane(xy_direction(d, t)) : 0u;

    // Full tiles (the common case) need no masks for columns or rows outside.
    auto body = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        // this lane's site c of step i is inside the tile
        auto in = [&](uint32_t i, uint32_t c) { return FULL || (W * (wave + NW * i) + lr < h && col + c < w); };
        uint32_t v[PER];
        if constexpr (FULL && W == 4) {
            uint64_t q4[STEPS];
#pragma unroll
            for (uint32_t i = 0; i < STEPS; ++i)
                q4[i] = *reinterpret_cast<gptr<const any_u64>>(lab_tile + (site0 + i * wave_step) * 2u);
#pragma unroll
            for (uint32_t i = 0; i < STEPS; ++i)
#pragma unroll
                for (uint32_t c = 0; c < W; ++c) v[i * W + c] = (uint32_t)(q4[i] >> (16 * c)) & 0xFFFFu;
        } else {
            gptr<const uint16_t> lab_p = (gptr<const uint16_t>)lab_tile + site0;
#pragma unroll
            for (uint32_t i = 0; i < STEPS; ++i, lab_p += wave_step)
#pragma unroll
                for (uint32_t c = 0; c < W; ++c) v[i * W + c] = in(i, c) ? (uint32_t)lab_p[c] : 0u;
        }
        const uint32_t n_used = min(n_loaded, NS);
        const uint32_t nj = lane * NW + wave;   // this lane's node
        const bool is_node = nj < n_used;
        const uint64_t nw = is_node ? nodes[node0 + nj] : 0ull;

        // Site c of step i: tile index li(i W + c).  The labels go to E.  A
        // pointer to a larger site is found by the walk below.
        const uint32_t li0 = (W * wave + lr) * TX + col;
        auto li = [&](uint32_t j) { return li0 + (j / W) * (W * NW * TX) + j % W; };
#pragma unroll
        for (uint32_t i = 0; i < STEPS; ++i) {
            if constexpr (W == 4) {   // (entries outside the tile are not read)
                uint64_t q4 = 0;
#pragma unroll
                for (uint32_t c = 0; c < W; ++c) q4 |= (uint64_t)v[i * W + c] << (16 * c);
                *reinterpret_cast<uint64_t*>(&E[li(i * W)]) = q4;
            } else if (in(i, 0)) {
                E[li(i)] = (uint16_t)v[i];
            }
        }
        SW_PHASE(pc, 0);   // labels in
        // The roots (tagged), one ballot per row: that of a cluster inside the tile
        // joins this wave's list, a node's slot must name a node of the tile
        // (labels outside the tile are 0).  Lanes with nothing
        // to list store to their scratch slot instead of branching around the
        // store.
        uint32_t nterm = 0;   // wave-uniform
        uint32_t most = 0;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            const uint64_t m = ballot(v[j] == ROOT16);
            most = max(most, v[j]);
            my_list[lane_in(m) ? nterm + lanes_below(m) : PER * TX + 64 + lane] = (uint16_t)li(j);
            nterm += popc64(m);
        }
        bad |= most >= NODE16 + n_used;
        SW_PHASE(pc, 1);   // roots inside the tile listed
        // this wave's nodes find their roots' keys and join the list
        if (is_node) {
            const uint64_t root = n_find_from(nodes, n_nodes, node0 + nj, nw, bad);
            NK[nj + 1] = key_of(root);
            if (CS) NR[nj] = bad ? node0 + nj : node_of(root);
        }
        const uint32_t n_inside = nterm;
        {
            const uint64_t m = ballot(is_node);
            if (is_node) my_list[nterm + lanes_below(m)] = (uint16_t)(NODE_ENTRY | (nj + 1));
            nterm += popc64(m);
        }
        SW_PHASE(pc, 2);   // node roots found

        // the states, 64 list entries at a time; lanes past the end work on a
        // copy they do not store
        for (uint32_t j0 = 0; j0 < nterm; j0 += 64) {
            const uint32_t j = j0 + lane;
            const bool act = j < nterm;
            const uint32_t e = my_list[act ? j : 0];
            const bool node = (e & NODE_ENTRY) != 0u;
            const uint32_t idx = e & ~NODE_ENTRY;
            const uint32_t key = node ? NK[idx & (NKN - 1u)] : __umul24(y0 + idx / TX, L) + x0 + idx % TX;
            const uint32_t st = XY ? xy_flip_bit(d, key, t) : cluster_state(d, key, t);
            if (act && node) NK[idx & (NKN - 1u)] = st;
            if (act && !node) E[idx & (TY * TX - 1u)] = ROOT16 | RES16 | st;
        }
        SW_PHASE(pc, 3);   // states drawn
        __syncthreads();
        SW_PHASE(pc, 4);   // barrier

        // Every site follows in-tile pointers (each to a smaller tile index, so
        // the walk ends) to a root: resolved inside the tile, or a node whose
        // state is in the table; the new spins are stored at the end.
        // (A root's entry, ROOT16 and up, is larger than every tile index, so
        // `x < cur` alone continues the walk.)  The first step is taken from the
        // label still in its register: a pointer leads to its target, a root's
        // tag back to the site itself (one of two to three steps saved a row).
        auto walk = [&](uint32_t j, uint32_t& at) -> uint32_t {
            uint32_t cur = min(v[j], li(j)), x = E[cur];
            while (x < cur) {
                cur = x;
                x = E[cur];
            }
            bad |= !(x & ROOT16);
            if (CS) at = (x & RES16) ? cur : TY * TX + (x & (NKN - 1u));   // where C counts it
            return (x & RES16) ? x : NK[x & (NKN - 1u)];
        };
        uint32_t at;
        if constexpr (XY) {
            // one bit per row (reflect or not) keeps the loop's registers few
            uint32_t bits = 0;
#pragma unroll
            for (uint32_t j = 0; j < PER; ++j)
                if (in(j / W, j % W)) bits |= (walk(j, at) & 1u) << j;
            SW_PHASE(pc, 5);   // walks
            // the angles of the steps with a reflected site, two steps at a time:
            // their loads in flight together, then their stores
            const gptr<char> a_tile = (gptr<char>)(glb(d.ang) + (size_t)y0 * L + x0);
            constexpr uint32_t B = STEPS < 2 ? STEPS : 2;
#pragma unroll 1
            for (uint32_t i0 = 0; i0 < STEPS; i0 += B) {
                u32x4 av[B];
#pragma unroll
                for (uint32_t i = 0; i < B; ++i) {
                    const uint32_t m = (bits >> ((i0 + i) * W)) & 15u;
                    const gptr<const uint32_t> a = (gptr<const uint32_t>)(a_tile + (site0 + (i0 + i) * wave_step) * 4u);
                    av[i] = u32x4{0u, 0u, 0u, 0u};
                    if (FULL ? m != 0u : m == 15u) {
                        const any_u32x4 q = *reinterpret_cast<gptr<const any_u32x4>>(a);
                        av[i] = u32x4{q[0], q[1], q[2], q[3]};
                    } else if (!FULL && m) {
                        if (m & 1u) av[i].x = a[0];
                        if (m & 2u) av[i].y = a[1];
                        if (m & 4u) av[i].z = a[2];
                        if (m & 8u) av[i].w = a[3];
                    }
                }
#pragma unroll
                for (uint32_t i = 0; i < B; ++i) {
                    const uint32_t m = (bits >> ((i0 + i) * W)) & 15u;
                    const gptr<uint32_t> a = (gptr<uint32_t>)(a_tile + (site0 + (i0 + i) * wave_step) * 4u);
                    if (m & 1u) av[i].x = xy_reflect(av[i].x, phi);
                    if (m & 2u) av[i].y = xy_reflect(av[i].y, phi);
                    if (m & 4u) av[i].z = xy_reflect(av[i].z, phi);
                    if (m & 8u) av[i].w = xy_reflect(av[i].w, phi);
                    if (FULL ? m != 0u : m == 15u) {
                        *reinterpret_cast<gptr<any_u32x4>>(a) = any_u32x4{av[i].x, av[i].y, av[i].z, av[i].w};
                    } else if (!FULL && m) {
                        if (m & 1u) a[0] = av[i].x;
                        if (m & 2u) a[1] = av[i].y;
                        if (m & 4u) a[2] = av[i].z;
                        if (m & 8u) a[3] = av[i].w;
                    }
                }
            }
        } else {
#pragma unroll
            for (uint32_t j = 0; j < PER; ++j) {
                at = INVALID;
                if (in(j, 0)) v[j] = walk(j, at);   // (the new state)
                if (CS && count) {
                    const uint32_t left = (uint32_t)__shfl_up((int)at, 1);
                    const uint64_t heads = ballot(lane == 0 || at != left);
                    const uint64_t right = lane == 63 ? 0ull : heads >> (lane + 1);
                    const uint32_t len = right ? (uint32_t)__builtin_ctzll(right) + 1u : 64u - lane;
                    if (at != INVALID && lane_in(heads)) atomicAdd(&C[at >> 1], len << (16u * (at & 1u)));
                }
            }
            SW_PHASE(pc, 5);   // walks
            gptr<uint8_t> s_p = (gptr<uint8_t>)s_tile + site0;
#pragma unroll
            for (uint32_t j = 0; j < PER; ++j, s_p += wave_step)
                if (in(j, 0)) *s_p = (uint8_t)v[j];
        }
        if constexpr (CS) {
            if (!count) return;
            __syncthreads();
            auto sites = [&](uint32_t i) { return (C[i >> 1] >> (16u * (i & 1u))) & 0xFFFFu; };
            uint64_t s2 = 0;
            unsigned __int128 s4 = 0;
            for (uint32_t j = lane; j < n_inside; j += 64) {
                const uint32_t c = sites(my_list[j] & (TY * TX - 1u));
                const uint64_t c2 = (uint64_t)c * c;
                s2 += c2;
                s4 += c2 * c2;   // (at most 2^52)
            }
            if (wave * 64 < n_used) {
                // the nodes again, one a thread; those of the wave's first root (by
                // number: most often the largest cluster) go in one addition
                const uint32_t root = tid < n_used ? NR[tid] : INVALID;
                uint32_t c = tid < n_used ? sites(TY * TX + tid + 1) : 0u, lead = root;
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) lead = min(lead, (uint32_t)__shfl_xor((int)lead, o));
                const uint64_t same = ballot(root == lead);
                const uint32_t all = wave_sum(root == lead ? c : 0u);
                if (lane_in(same)) c = lanes_below(same) ? 0u : all;
                if (c) {
                    const uint64_t old = __hip_atomic_fetch_add((gptr<unsigned long long>)(glb(d.csize) + root),
                                                                (unsigned long long)c, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT);
                    const uint64_t now = old + c, d2 = now * now - old * old;
                    s2 += d2;
                    s4 += (unsigned __int128)d2 * (now * now + old * old);
                }
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                s2 += (uint64_t)__shfl_xor((unsigned long long)s2, o);
                const uint64_t lo = (uint64_t)__shfl_xor((unsigned long long)s4, o);
                s4 += ((unsigned __int128)__shfl_xor((unsigned long long)(s4 >> 64), o) << 64) | lo;
            }
            if (lane == 0 && s2) {
                __hip_atomic_fetch_add(&sums[0], (unsigned long long)s2, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                add_u128<__HIP_MEMORY_SCOPE_WORKGROUP>(&sums[1], &sums[2], s4);
            }
            __syncthreads();
            if (tid == 0) cs_flush(d, t, sums);
        }
    };
    if (w == TX && h == TY) body(std::true_type{});
    else body(std::false_type{});
    SW_PHASE(pc, 6);   // spins out (Potts) or reflections (XY)
    if (bad) flag_error(d.err);
    SW_PHASE_FLUSH(pc, phase_table(XY ? 4u : 2u));

    // The ring record of the next sweep starts from zero.
    if (d.cap && tile == 0) {
        const uint32_t words = NCOPY * (XY ? XY_STRIDE : ring_stride(d.q));
        gptr<int64_t> rec = glb(d.ring) + (size_t)((t + 1) % d.cap) * words;
        for (uint32_t i = tid; i < words; i += NT) rec[i] = 0;
    }
}

// ---------------------------------------------------------------------------
// Measurement of the current configuration into the ring record of sweep
// counter + k (used after the last sweep of a call).
template <int TY>
__global__ __launch_bounds__(threads_of<TY>()) void k_measure(const LatDesc* descs, const WorkItem* map, uint32_t k,
                                                const uint32_t* n_each)
{
    constexpr uint32_t RPW = TY / waves_of<TY>();
    __shared__ __align__(16) uint8_t sp[(TY + 1) * SPW];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t tot;
    LatDesc d;
    uint32_t tile, lat;
    if (!pick(descs, map, blockIdx.x, true, d, tile, lat)) return;
    if (d.cap == 0) return;
    if (n_each) {
        const uint32_t nl = n_each[lat];
        if (nl == 0) return;
        k = nl - 1;
    }
    const TileGeom g = tile_geom(d, tile, TY);
    const uint32_t t = *glb(d.counter) + k;
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
    const uint32_t w = g.w, h = g.h;
    if (tid < 256) hist[tid] = 0;
    if (tid == 0) tot = 0;
    stage_spins<TY, threads_of<TY>()>(sp, d, g, tid);
    __syncthreads();
    const uint32_t x = lane;
    const uint64_t validm = (w == 64) ? ~0ull : ((1ull << w) - 1ull);
    const uint32_t r0 = wave * RPW, r1 = min(h, r0 + RPW);
    count_tile_states<TY, threads_of<TY>()>(sp, g, d.q, hist, tid);
    uint32_t n_unsat = 0;   // wave-uniform
    for (uint32_t r = r0; r < r1; ++r) {
        const uint8_t* row = sp + r * SPW;
        const uint32_t s = row[x], sr = row[x + 1], sd = row[SPW + x];
        n_unsat += popc64(ballot(s != sr) & validm) + popc64(ballot(s != sd) & validm);
    }
    if (lane == 0) atomicAdd(&tot, n_unsat);
    __syncthreads();
    int64_t* rp = ring_record(d, t, blockIdx.x % NCOPY);
    if (tid == 0) atomic_add_i64(&rp[0], tot);
    if (tid >= 1 && tid < d.q) {
        const uint32_t n = states_of_subsets(hist, d.q, tid);
        if (n) atomic_add_i64(&rp[1 + tid], n);
    }
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init(const LatDesc* descs, uint32_t lat, uint32_t random_start)
{
    const LatDesc d = descs[lat];
    const size_t N = (size_t)d.L * d.L;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        glb(d.s)[i] = random_start
                     ? (uint8_t)state_of_draw(philox4x32_10((uint32_t)i, 0u, 0u, 2u, d.key0, d.key1).x, d.q)
                     : (uint8_t)0;
    }
}

// The last sweep's labels of rows [ya, yb) resolved to the smallest site index
// of each cluster, written from the base of the label region (row ya first):
// one workgroup per tile walks its sites' pointers in LDS to their tile-local
// roots and those, if they are nodes, to the edge forest's roots.  The tile
// labels (upper half of the region) are only read, so that (yb - ya) L <= N/2
// keeps the output clear of them.  With `out` the labels go there instead, all
// rows at once, and a region that holds site indices already is copied (a lattice
// of L = 128 swept by tiles: labels read in 32 us; in two bands and three copies 95,
// and 34 when it was always swept whole).
template <int TY>
__global__ __launch_bounds__(threads_of<TY>()) void k_resolve(const LatDesc* descs, uint32_t lat, uint32_t ya,
                                                              uint32_t yb, uint32_t* to)
{
    constexpr uint32_t NT = threads_of<TY>();
    __shared__ uint16_t E[TY * TX];
    const LatDesc d = descs[lat];
    const uint32_t tile = blockIdx.x;
    if (tile >= d.ntiles) return;
    const TileGeom g = tile_geom(d, tile, TY);
    if (g.y0 >= yb || g.y0 + g.h <= ya) return;
    const uint32_t NS = nslot(TY), n_nodes = d.ntiles * NS, node0 = tile * NS;
    const gptr<const uint16_t> lab = glb(d.tlab);
    const gptr<uint32_t> out = glb(to ? to : d.lab);
    if (to && *glb(d.labels) != LABELS_TILE) {
        for (uint32_t li = threadIdx.x; li < TY * TX; li += NT) {
            const uint32_t r = li / TX, c = li % TX, y = g.y0 + r;
            if (r < g.h && c < g.w && y >= ya && y < yb)
                out[(size_t)(y - ya) * d.L + g.x0 + c] = glb(d.lab)[(size_t)y * d.L + g.x0 + c];
        }
        return;
    }
    bool bad = false;
    for (uint32_t li = threadIdx.x; li < TY * TX; li += NT) {
        const uint32_t r = li / TX, c = li % TX;
        E[li] = (r < g.h && c < g.w) ? lab[(size_t)(g.y0 + r) * d.L + g.x0 + c] : ROOT16;
    }
    __syncthreads();
    for (uint32_t li = threadIdx.x; li < TY * TX; li += NT) {
        const uint32_t r = li / TX, c = li % TX, y = g.y0 + r;
        if (r >= g.h || c >= g.w || y < ya || y >= yb) continue;
        uint32_t cur = li, v = E[cur];
        while (v < cur) {   // (a tagged entry is larger than every index)
            cur = v;
            v = E[cur];
        }
        uint32_t root = INVALID;
        if (!(v & ROOT16)) {
            bad = true;
        } else if (v == ROOT16) {
            root = (g.y0 + cur / TX) * d.L + g.x0 + cur % TX;
        } else {
            root = key_of(n_root(glb(d.nodes), n_nodes, node0 + (v - NODE16), bad));
        }
        out[(size_t)(y - ya) * d.L + g.x0 + c] = root;
    }
    if (bad) flag_error(d.err);
}

// One thread per (record, word): the sum of the word over the record's NCOPY
// partial copies.
__global__ __launch_bounds__(256) void k_ring_sum(const int64_t* ring, int64_t* out, uint32_t slots, uint32_t slot0,
                                                  uint32_t n, uint32_t W, uint32_t stride, const uint32_t* err)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * W) return;
    if (i == 0 && err) glb(out)[(size_t)n * W] = *glb(err);
    const uint32_t rec = i / W, w = i - rec * W;
    const uint32_t slot = (uint32_t)(((uint64_t)slot0 + rec) % slots);
    const size_t R = stride;
    const gptr<const int64_t> copy0 = glb(ring) + (size_t)slot * NCOPY * R;
    const gptr<const int64_t> base = copy0 + w;
    int64_t sum = 0;
    if (copy0[W] != 0) {
        sum = base[0];   // the whole record is in copy 0
    } else {
#pragma unroll 8
        for (uint32_t c = 0; c < NCOPY; ++c) sum += base[(size_t)c * R];
    }
    glb(out)[i] = sum;
}

// Bytes of src copied to out by words (src 4-byte aligned, out too), then the
// error flag.
__global__ __launch_bounds__(256) void k_read_out(const uint32_t* src, uint32_t bytes, uint32_t* out, const uint32_t* err)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x, words = bytes >> 2;
    if (i < words) glb(out)[i] = glb(src)[i];
    if (i == 0) {
        const gptr<const uint8_t> tail = (gptr<const uint8_t>)(glb(src) + words);
        const gptr<uint8_t> to = (gptr<uint8_t>)(glb(out) + words);
        for (uint32_t j = 0; j < (bytes & 3u); ++j) to[j] = tail[j];
        glb(out)[(bytes + 3u) >> 2] = *glb(err);
    }
}

// Advance sweep counters: lattice i by n (or by n_each[i] when given), after
// sweeps by tiles (or sweeps of a batch, whose labels are not read).
__global__ void k_bump(const LatDesc* descs, uint32_t count, const uint32_t* n_each, uint32_t n)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) {
        const uint32_t add = n_each ? n_each[i] : n;
        if (add) {
            *glb(descs[i].counter) += add;
            *glb(descs[i].labels) = LABELS_TILE;
        }
    }
}

// Set-up of a lattice whose descriptor and state live in caller-independent
// scratch (the no-allocation entry point): descriptor copied in, error flag
// cleared, sweep counter set, ring records zeroed.  A plain kernel rather than
// copies and fills, so the whole call can be captured in a graph.
__global__ __launch_bounds__(256) void k_static_setup(LatDesc d, LatDesc* d_out, DevState* st, uint32_t counter,
                                                      int64_t* ring, uint32_t ring_words)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        *d_out = d;
        st->err = 0;
        st->counter = counter;
    }
    for (uint32_t j = i; j < ring_words; j += gridDim.x * blockDim.x) glb(ring)[j] = 0;
}

// One finished ring record as an observable row [n_unsat, n_active, n_0, ...,
// n_{q-1}] (n_0 = N minus the other counts), summed over its NCOPY partial
// copies; optionally the error flag into *status.  One workgroup of 256.
__global__ __launch_bounds__(256) void k_emit_row(const int64_t* ring, uint32_t slots, uint32_t slot, uint32_t q,
                                                  uint64_t N, int64_t* row, const uint32_t* err, uint32_t* status)
{
    __shared__ int64_t word[256];
    const uint32_t w = threadIdx.x;
    if (row) {
        const size_t R = ring_stride(q);
        int64_t sum = 0;
        if (w <= q) {
            const gptr<const int64_t> base = glb(ring) + (size_t)(slot % slots) * NCOPY * R + w;
            for (uint32_t c = 0; c < NCOPY; ++c) sum += base[(size_t)c * R];
        }
        word[w] = sum;
        __syncthreads();
        if (w == 0) {
            int64_t rest = 0;
            for (uint32_t c = 1; c < q; ++c) rest += word[1 + c];
            glb(row)[0] = word[0];
            glb(row)[1] = word[1];
            glb(row)[2] = (int64_t)N - rest;
        } else if (w < q) {
            glb(row)[2 + w] = word[1 + w];
        }
    }
    if (status && w == 0) *glb(status) = *glb(err);
}

// ---------------------------------------------------------------- launchers
namespace {
uint32_t init_grid(size_t N)
{
    const size_t b = (N + 255) / 256;
    return (uint32_t)(b < 65536 ? (b ? b : 1) : 65536);
}
}  // namespace

// BLOCK(T): threads per workgroup of the kernel instantiated for T rows.
#define SWMI_TY_DISPATCH_B(TYV, KERNEL, GRID, BLOCK, ...)                                                    \
    switch (TYV) {                                                                                         \
    case 32: hipLaunchKernelGGL(KERNEL<32>, dim3(GRID), dim3(BLOCK(32)), 0, w.stream, __VA_ARGS__); break;    \
    case 64: hipLaunchKernelGGL(KERNEL<64>, dim3(GRID), dim3(BLOCK(64)), 0, w.stream, __VA_ARGS__); break;    \
    case 128: hipLaunchKernelGGL(KERNEL<128>, dim3(GRID), dim3(BLOCK(128)), 0, w.stream, __VA_ARGS__); break; \
    default: return hipErrorInvalidValue;                                                                  \
    }
#define SWMI_TILE_BLOCK(T) threads_of<T>()
#define SWMI_TY_DISPATCH(TYV, KERNEL, GRID, ...) SWMI_TY_DISPATCH_B(TYV, KERNEL, GRID, SWMI_TILE_BLOCK, __VA_ARGS__)

// Waves of a tile's workgroup.  A wave walks its strip of rows one after another,
// so with few tiles, where a sweep is one workgroup's latency, shorter strips
// on more waves are faster; with many tiles they repeat the work at the strips'
// seams and leave fewer workgroups per CU to cover each other's barriers.
// Whole sweeps measured at 64-row tiles, q = 2 (us; labelling with 4 / 16 waves,
// then flip with 4 / 8 / 16 waves):
//   16 tiles (L = 200)     27.4 / 25.1    27.4 / 25.7 / 24.8
//   256 tiles (L = 1001)   35.4 / 32.5    35.4 / 33.7 / 32.7
//   529 tiles (L = 1448)   38.9 / 42.9    38.9 / 37.3 / 38.4
//   1024 tiles (L = 2048)  44.1 / 50.6    44.1 / 43.2 / 46.2
//   2116 tiles (L = 2900)  65.2 / 84.6    65.2 / 66.7 / 72.2
// so the lines lie at one workgroup per CU (256 tiles) and, for the flip, four.
// Labelling and flip both with 4 / 8 / 16 waves, for the other kernels and for
// mapped work (us):
//   XY, K = 1.12   256 tiles 42.3 / 38.3 / 37.0, 289 48.2 / 44.4 / 45.0, 529 55.4 / 52.7 / 56.5,
//                  1024 64.3 / 62.9 / 70.0, 1089 71.6 / 72.3 / 79.3
//   cluster sums   256 tiles 45.0 / 40.7 / 39.7, 289 47.2 / 43.2 / 44.1,
//                  1024 82.8 / 82.2 / 84.3, 1089 88.3 / 89.6 / 96.3
//   batches of L = 128   256 tiles 30.3 / 26.8 / 26.0, 400 33.1 / 30.5 / 31.8,
//                  1024 42.0 / 41.7 / 49.6, 1600 53.3 / 57.3 / 73.3
// so the same lines hold for them (eight waves for the labelling of 257 to about
// 500 tiles too would take 2 to 3 % off a sweep there).

template <int TY, bool PRESET>
hipError_t start_bond_label(const Work& w, uint32_t k, uint32_t flags)
{
    auto go = [&](auto nw) {
        constexpr uint32_t NW = decltype(nw)::value;
        return start_kernel(w, k_bond_label<TY, NW, PRESET>, dim3(w.nitems), dim3(64 * NW), w.descs, w.map, k, flags);
    };
    if constexpr (TY == 64) {
        if (w.nitems <= CUS) return go(std::integral_constant<uint32_t, 16>{});
        return go(std::integral_constant<uint32_t, 4>{});
    } else {
        return go(std::integral_constant<uint32_t, waves_of<TY>()>{});
    }
}

template <int TY, bool XY>
hipError_t start_flip(const Work& w, uint32_t k)
{
    auto go = [&](auto nw) {
        constexpr uint32_t NW = decltype(nw)::value;
        const dim3 grid(w.nitems), block(64 * NW);
        if (!XY && w.cluster)
            return start_kernel(w, k_flip<TY, NW, XY, !XY>, grid, block, w.descs, w.map, k);
        return start_kernel(w, k_flip<TY, NW, XY>, grid, block, w.descs, w.map, k);
    };
    if constexpr (TY == 64) {
        if (w.nitems <= CUS) return go(std::integral_constant<uint32_t, 16>{});
        if (w.nitems <= 4 * CUS) return go(std::integral_constant<uint32_t, 8>{});
        return go(std::integral_constant<uint32_t, 4>{});
    } else {
        return go(std::integral_constant<uint32_t, waves_of<TY>()>{});
    }
}

hipError_t launch_bond_label(const Work& w, uint32_t k, uint32_t flags)
{
    if (w.nitems == 0) return hipSuccess;
    switch (w.ty) {
    case 32: return start_bond_label<32, false>(w, k, flags);
    case 64: return start_bond_label<64, false>(w, k, flags);
    case 128: return start_bond_label<128, false>(w, k, flags);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_label_preset(const Work& w)
{
    if (w.nitems == 0) return hipSuccess;
    switch (w.ty) {
    case 32: return start_bond_label<32, true>(w, 0, 0);
    case 64: return start_bond_label<64, true>(w, 0, 0);
    case 128: return start_bond_label<128, true>(w, 0, 0);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_flip(const Work& w, uint32_t k)
{
    if (w.nitems == 0) return hipSuccess;
    switch (w.ty) {
    case 32: return start_flip<32, false>(w, k);
    case 64: return start_flip<64, false>(w, k);
    case 128: return start_flip<128, false>(w, k);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_flip_xy(const Work& w, uint32_t k)
{
    if (w.nitems == 0) return hipSuccess;
    switch (w.ty) {
    case 32: return start_flip<32, true>(w, k);
    case 64: return start_flip<64, true>(w, k);
    case 128: return start_flip<128, true>(w, k);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_merge(const Work& w, uint32_t bump)
{
    if (w.nitems == 0) return hipSuccess;
    // Hooks that climb both chains at once (n_hook2) for a lattice by itself of
    // 12 x 12 to 160 x 160 tiles, at a coupling where clusters span it: smaller
    // clusters make short chains, fewer tiles too, and more tiles do not all run
    // at the same time and are bound by the rate of atomics instead, as are the
    // many lattices of mapped work.  A whole sweep, us, one chain / both:
    //   q = 2, K_c     L = 512 27.5 / 27.3, 777 33.0 / 31.4, 1001 35.4 / 32.7,
    //                  2048 56.4 / 46.5, 4096 121 / 101, 6000 234 / 188
    //   q = 2, 2048    0.95 K_c 37.1 / 37.7, 0.99 40.2 / 41.4, 1.01 51.8 / 46.9
    //   q = 8, 2048    0.99 K_c 36.3 / 36.6, 1.00 37.4 / 37.8, 1.01 52.4 / 45.2
    //   XY, 2048       K = 1.01 60.8 / 61.9, 1.05 67.8 / 65.6, 1.12 72.2 / 65.9
    // the merge alone, q = 2, K_c, 8192 77 / 48, 10000 81 / 68, 11585 87 / 94, 16384
    // 133 / 141; 32 uneven jobs 292 / 300.  Far above the transition, whole sweeps:
    //   q = 2, 4096    K = 1.6 104.5 / 91.1, 2.0 100.7 / 94.8, 2.2 99.2 / 99.1,
    //                  2.4 97.9 / 101.6, 4 96.0 / 102.0 (q = 4, 8, 20 alike)
    //   q = 2, 2048    K = 2.0 45.5 / 44.0, 2.2 44.7 / 44.8, 2.4 44.1 / 45.3
    //   q = 2, 8192    K = 2.2 289 / 266, 2.7 280 / 273, 4 274 / 277
    //   XY, 2048       K = 2 69.5 / 63.0, 6 67.2 / 64.2, 30 64.6 / 64.3
    const bool both = w.spans && !w.map && w.nitems >= 144 && w.nitems <= 25600;
    auto go = [&](auto ty) {
        constexpr int TY = decltype(ty)::value;
        const dim3 grid((w.nitems + 3) / 4), block(256);
        return both ? start_kernel(w, k_merge<TY, true>, grid, block, w.descs, w.map, w.nitems, bump)
                    : start_kernel(w, k_merge<TY, false>, grid, block, w.descs, w.map, w.nitems, bump);
    };
    switch (w.ty) {
    case 32: return go(std::integral_constant<int, 32>{});
    case 64: return go(std::integral_constant<int, 64>{});
    case 128: return go(std::integral_constant<int, 128>{});
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_measure(const Work& w, uint32_t k)
{
    if (w.nitems == 0) return hipSuccess;
    SWMI_TY_DISPATCH(w.ty, k_measure, w.nitems, w.descs, w.map, k, (const uint32_t*)nullptr);
    return hipGetLastError();
}

hipError_t launch_measure_each(const Work& w, const uint32_t* n_each)
{
    if (w.nitems == 0) return hipSuccess;
    if (!w.map) return hipErrorInvalidValue;
    SWMI_TY_DISPATCH(w.ty, k_measure, w.nitems, w.descs, w.map, 0u, n_each);
    return hipGetLastError();
}

hipError_t launch_init(const LatDesc* descs, uint32_t lat, size_t N, uint32_t random_start, hipStream_t s)
{
    hipLaunchKernelGGL(k_init, dim3(init_grid(N)), dim3(256), 0, s, descs, lat, random_start);
    return hipGetLastError();
}

hipError_t launch_resolve(const LatDesc* descs, uint32_t lat, uint32_t ntiles, uint32_t ty, uint32_t ya, uint32_t yb,
                          uint32_t* to, hipStream_t s)
{
    switch (ty) {
    case 32: hipLaunchKernelGGL(k_resolve<32>, dim3(ntiles), dim3(threads_of<32>()), 0, s, descs, lat, ya, yb, to); break;
    case 64: hipLaunchKernelGGL(k_resolve<64>, dim3(ntiles), dim3(threads_of<64>()), 0, s, descs, lat, ya, yb, to); break;
    case 128:
        hipLaunchKernelGGL(k_resolve<128>, dim3(ntiles), dim3(threads_of<128>()), 0, s, descs, lat, ya, yb, to);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ring_sum(const int64_t* ring, int64_t* out, uint32_t slots, uint32_t slot0, uint32_t n,
                           uint32_t words, uint32_t stride, const uint32_t* err, hipStream_t s)
{
    const uint64_t total = (uint64_t)n * words;
    if (total == 0) return hipSuccess;
    if (total > 0xFFFFFFFFull || slot0 >= slots || n >= slots || words > stride) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ring_sum, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, s, ring, out, slots, slot0, n,
                       words, stride, err);
    return hipGetLastError();
}

hipError_t launch_read_out(const void* src, size_t bytes, void* out, const uint32_t* err, hipStream_t s)
{
    if (bytes == 0 || bytes > (1u << 30)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_read_out, dim3((uint32_t)((bytes / 4 + 256) / 256)), dim3(256), 0, s,
                       static_cast<const uint32_t*>(src), (uint32_t)bytes, static_cast<uint32_t*>(out), err);
    return hipGetLastError();
}

hipError_t launch_static_setup(const LatDesc& d, LatDesc* d_out, DevState* st, uint32_t counter, int64_t* ring,
                               uint32_t ring_words, hipStream_t s)
{
    const uint32_t grid = std::max(1u, std::min(1024u, (ring_words + 255) / 256));
    hipLaunchKernelGGL(k_static_setup, dim3(grid), dim3(256), 0, s, d, d_out, st, counter, ring, ring_words);
    return hipGetLastError();
}

hipError_t launch_emit_row(const int64_t* ring, uint32_t slots, uint32_t slot, uint32_t q, uint64_t N, int64_t* row,
                           const uint32_t* err, uint32_t* status, hipStream_t s)
{
    if (q < 2 || q > 255 || slots == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_emit_row, dim3(1), dim3(256), 0, s, ring, slots, slot, q, N, row, err, status);
    return hipGetLastError();
}

hipError_t launch_bump(const LatDesc* descs, uint32_t count, const uint32_t* n_each, uint32_t n, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bump, dim3((count + 255) / 256), dim3(256), 0, s, descs, count, n_each, n);
    return hipGetLastError();
}

}  // namespace swmi
