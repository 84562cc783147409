// Small lattices swept whole in one workgroup's LDS, many sweeps per launch.
//
// A lattice of at most 128 x 128 sites fits a workgroup's LDS with its spins,
// draws and union-find; one launch then runs any number of sweeps without
// touching global memory between them (no per-sweep launches, which is what
// bounds the tile kernels at these sizes).  Each sweep takes the three steps of
// Sec. 2 with the same random streams and the same cluster keys as the tile
// kernels, so results are bit-identical to them (and to the oracle).
//
// What bounds it is one CU: about 400 SIMD cycles of vector, scalar and LDS
// instructions per 64 sites in the row step below, and in the other steps
// chains of dependent LDS accesses.  (L = 64, q = 2 at K_c: 9.2 us a sweep, of
// which the rows take a quarter, the seams a fifth; 25.2 us for the kernel
// before, which walked every site to its root through the rows' chains and
// had seven barriers.  L = 128: 26.9 us, before 54.9.)  So the work is cut to keep
// chains short: sixteen waves (fewer where there are more lattices than CUs:
// launch_whole) own a strip of whole rows each (one column per lane, 64 columns at
// a time), everything a strip needs is loaded first, and a sweep has four
// barriers:
//   1. bonds and runs: the bonds of a row are wave ballots of its spins and
//      draws; the runs of +x bonds of a row are bit arithmetic on them (no LDS),
//      and a run's first site is its node in the union-find.  The first +y bond
//      into a run makes the run's node point at the node above (bit arithmetic
//      again: a carry through the run's bonds tells first from later ones); the
//      other +y bonds, and the +x bonds across 64-column passes and the periodic
//      edge, are queued and joined 64 at a time.  A run hooked like that takes
//      the label above, so a strip's chains stay one deep.  The configuration the bonds
//      are drawn on is the previous sweep's result and is measured here;
//   2. seams: the +y bonds from the row above a strip (the last strip's for the
//      first: the periodic edge), joined the same way;
//   3. roots: a label that points at itself draws its cluster's state (Philox
//      counter (root, 0, t, 1)), gathered per wave and drawn 64 at a time, and
//      keeps it in its own entry, tagged; the other labels are pointed at
//      their roots;
//   4. every site takes the state, two reads from its label; the draws of the next sweep, which
//      depend on nothing, are made here (one Philox call per pair of sites in
//      the order of the site index, counter (i >> 1, 0, t, 0), so odd sizes
//      cost no more than even ones) and kept as two bits per site.
// After the last sweep the spins go back to global memory, and on request the
// labels (smallest site indices) and the tile-major bond words of that sweep.
#include <hip/hip_runtime.h>

#include "sw_device.hpp"
#include "sw_kernels.hpp"
#include "sw_tile.hpp"

namespace swmi {

namespace {

constexpr uint32_t TAG = 0x8000u;                 // a root's entry once it holds its state

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Sweeps counter .. counter + n - 1.  flags bit 0: write the labels
// and bond words of the last sweep; bit 1: leave the sweep counter (the caller
// advances it), else set it past the last sweep.  ty: tile height of the
// lattice's bond-word layout.
template <int LMAX, uint32_t NW>
__global__ __launch_bounds__(64 * NW) void k_whole(const LatDesc* descs, const uint32_t* list,
                                                    uint32_t n_uniform, const uint32_t* n_each, uint32_t flags,
                                                    uint32_t ty)
{
    constexpr uint32_t NT = 64 * NW;
    constexpr uint32_t CH = (LMAX + 63) / 64;         // 64-column passes of a row
    constexpr uint32_t RP = LMAX / NW;                // rows of a strip, at most
    static_assert(NT >= 256 && (RP & (RP - 1)) == 0 && RP <= 16, "a thread a state; rows by masked lanes");
    constexpr uint32_t NMAX = LMAX * LMAX;
    constexpr uint32_t SPS = LMAX + 4;                // row stride of the spins
    constexpr uint32_t QCAP = 256;
    __shared__ uint8_t s[LMAX * SPS + 64];            // spins (a pass reads 65 columns of any row)
    __shared__ __align__(16) uint8_t D[NMAX + 128];   // per site: bit 0 +x draw below the threshold, bit 1 +y
    __shared__ uint32_t P[NMAX];                      // union-find over the runs' first sites
    __shared__ uint32_t UQ[NW][QCAP];                 // per wave: queued unions (two 16-bit sites), then roots
    __shared__ uint16_t HB[NW][64 * CH];              // per strip: the labels of its last row, by column
    __shared__ uint16_t LN[NW][CH][RP];               // per strip: the node of the last site of each row's pass
    __shared__ uint64_t MB[NW][CH][2];                // per strip: its last row's +y bonds and run links
    __shared__ uint64_t BW[LMAX][CH][2];              // the last sweep's bond words
    __shared__ uint32_t hist[256];
    __shared__ uint32_t tot[2];                       // equal pairs, active bonds

    const uint32_t lat = list ? list[blockIdx.x] : blockIdx.x;
    const LatDesc d = descs[lat];
    const uint32_t n = n_each ? n_each[lat] : n_uniform;
    if (n == 0) return;
    const uint32_t L = d.L, N = L * L, q = d.q;
    const uint32_t tid = threadIdx.x, wave = wave_id(), lane = tid & 63u;
    if (L > (uint32_t)LMAX) {   // (the host sorts lattices by size; never taken)
        if (tid == 0) flag_error(d.err);
        return;
    }
    const uint32_t t0 = *glb(d.counter);
    const bool meas = d.cap != 0;
    bool bad = false;

    // this wave's strip: rows y0 .. y0 + rows - 1 of ns strips
    const uint32_t rps = (L + NW - 1) / NW, ns = (L + rps - 1) / rps;
    const uint32_t y0 = wave * rps, rows = wave < ns ? min(rps, L - y0) : 0u;
    auto columns = [&](uint32_t c) -> uint64_t {   // valid lanes of pass c
        const uint32_t w = L > 64 * c ? min(64u, L - 64 * c) : 0u;
        return w == 64 ? ~0ull : (1ull << w) - 1ull;
    };
    const uint32_t last_c = (L - 1) / 64, last_lane = (L - 1) & 63u;
    auto below = [&](uint32_t y) { return y + 1 == L ? 0u : y + 1; };
    uint32_t xr[CH];   // the column to the right, per pass
#pragma unroll
    for (uint32_t c = 0; c < CH; ++c) xr[c] = 64 * c + lane + 1 == L ? 0u : 64 * c + lane + 1;
    const uint64_t upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);

    for (uint32_t i = tid; i < N; i += NT) {
        const uint32_t y = div_L(d, i), x = i - y * L;
        s[y * SPS + x] = glb(d.s)[i];
    }
    if (tid < 256) hist[tid] = 0;
    if (tid < 2) tot[tid] = 0;

    auto draws = [&](uint32_t t) {
        const uint32_t pairs = (N + 1) >> 1;
        for (uint32_t p = tid; p < pairs; p += NT) {
            const u32x4 w = philox4x32_10(p, 0u, t, 0u, d.key0, d.key1);
            uint32_t b = 0;
            if (d.thr_nz)
                b = (uint32_t)(w.x <= d.thr_m1) | ((uint32_t)(w.y <= d.thr_m1) << 1) |
                    ((uint32_t)(w.z <= d.thr_m1) << 8) | ((uint32_t)(w.w <= d.thr_m1) << 9);
            reinterpret_cast<uint16_t*>(D)[p] = (uint16_t)b;
        }
    };
    draws(t0);
    __syncthreads();

    // equal pairs (per wave) and state counts of the strip's rows, added to tot
    // and hist; the loop below calls count_row for its own loads
    uint32_t n_eq = 0, ones = 0;
    uint64_t packed[2] = {0ull, 0ull};
    const bool q2 = q == 2, q8 = q <= 8, q16 = q <= 16;
    auto count_row = [&](uint64_t vm, uint32_t s0, uint64_t EX, uint64_t EY) {
        n_eq += popc64(EX) + popc64(EY);
        if (q2) {
            ones += popc64(ballot(s0 != 0) & vm);
            return;
        }
        const bool v = lane_in(vm);
        if (q8) count_state_byte(packed, v, s0);
        else if (q16) count_state_bytes(packed, v, s0 & 15u);
        else if (v && s0) atomicAdd(&hist[s0], 1u);
    };
    auto count_flush = [&]() {
        if (lane == 0) {
            atomicAdd(&tot[0], n_eq);
            if (q2) atomicAdd(&hist[1], ones);
        }
        if (q16 && !q2) flush_state_bytes(packed, hist, q, lane);
        n_eq = ones = 0;
        packed[0] = packed[1] = 0ull;
    };
    // the record of sweep t: its counts are in tot[0] and hist, written whole
    // into copy 0 with the whole-record flag
    const uint32_t words = NCOPY * ring_stride(q);
    uint32_t slot = meas ? t0 % d.cap : 0u;   // the next record to write
    auto write_record = [&](uint32_t active) {
        const gptr<int64_t> rec = glb(d.ring) + (size_t)slot * words;
        slot = slot + 1 == d.cap ? 0u : slot + 1;
        if (tid == 0) {
            rec[0] = 2ll * N - tot[0];
            rec[1] = active;
            rec[ring_words(q)] = 1;
        }
        if (tid >= 1 && tid < q) rec[1 + tid] = hist[tid];
    };

    uint32_t active_prev = 0;   // n_active of the previous sweep (every thread)
    for (uint32_t k = 0; k < n; ++k) {
        const uint32_t t = t0 + k;
        const bool meas_prev = meas && k > 0;
        const bool out = (flags & 1u) && k + 1 == n;   // the last sweep's bonds and labels are wanted
        uint32_t qn = 0;   // wave-uniform
        auto drain = [&]() {
            for (uint32_t j0 = 0; j0 < qn; j0 += 64) {
                const uint32_t j = j0 + lane;
                if (j < qn) {
                    const uint32_t e = lds_ld(&UQ[wave][j]);
                    lds_union(P, e & 0xFFFFu, e >> 16, bad);
                }
            }
            qn = 0;
        };
        auto push = [&](uint64_t m, uint32_t a, uint32_t b) {
            if (lane_in(m)) lds_st(&UQ[wave][qn + lanes_below(m)], a | (b << 16));
            qn += popc64(m);
        };
        // ---- 1. bonds, runs, measurement of the incoming configuration
        uint32_t lab[RP][CH];                   // labels of the lane's sites
        uint64_t C0[CH] = {};                   // run links of the strip's first row
        uint64_t Vp[CH] = {}, Cp[CH] = {};      // +y bonds and run links of the row above
        uint32_t n_act = 0, wrap = 0, join = 0;
#pragma unroll
        for (uint32_t j = 0; j < RP; ++j) {
            if (j >= rows) break;
            const uint32_t y = y0 + j;
            if (qn > QCAP - 64 * CH) drain();
#pragma unroll
            for (uint32_t c = 0; c < CH; ++c) {
                const uint32_t x = 64 * c + lane, li = y * L + x;
                const uint64_t vm = columns(c);
                const uint32_t s0 = s[y * SPS + x], sr = s[y * SPS + xr[c]], sd = s[below(y) * SPS + x], dd = D[li];
                const uint64_t EX = ballot(s0 == sr) & vm, EY = ballot(s0 == sd) & vm;
                const uint64_t BX = EX & ballot(dd & 1u), BY = EY & ballot(dd & 2u);
                if (meas_prev) count_row(vm, s0, EX, EY);
                n_act += popc64(BX) + popc64(BY);
                const uint64_t C = (BX << 1) & vm;   // bit x: linked to x - 1
                const uint64_t S = ~C & vm;          // first sites of runs
                const uint32_t h = y * L + 64 * c + 63u - (uint32_t)__builtin_clzll((S & upto) | 1ull);
                if (j == 0) {
                    C0[c] = C;
                    if (lane_in(S)) lds_st(&P[li], li);
                    lab[j][c] = h;
                } else {
                    const uint64_t V = Vp[c];
                    // sites above whose run here has a +y bond further left: a
                    // carry from a bond runs to the end of its run
                    const uint64_t X = (V << 1) & C;
                    const uint64_t later = (C & ~(C + X)) | X;
                    // a run's label: its first site, or the label above its first
                    // +y bond; its first site's entry carries the choice to all
                    // its sites (LDS accesses of a wave are done in order)
                    const uint32_t lp = lab[j > 0 ? j - 1 : 0][c];
                    if (lane_in(S)) lds_st(&P[li], li);
                    if (lane_in(V & ~later)) lds_st(&P[h], lp);
                    const uint32_t l = lds_ld(&P[h]);
                    lab[j][c] = l;
                    // bonds x-1 and x from one run above into one run here add nothing
                    push(V & later & ~((V << 1) & C & Cp[c]) & ballot(l != lp), lp, l);
                }
                // across the passes and the periodic edge: one bit a row, joined below
                if (c == last_c) wrap |= (uint32_t)((BX >> last_lane) & 1u) << j;
                else if (c < last_c) join |= (uint32_t)(BX >> 63) << j;
                if (lane == (c == last_c ? last_lane : 63u)) LN[wave][c][j] = (uint16_t)h;
                Vp[c] = BY;
                Cp[c] = C;
                if (j + 1 == rows) {
                    HB[wave][x] = (uint16_t)lab[j][c];
                    if (lane == 0) {
                        MB[wave][c][0] = BY;
                        MB[wave][c][1] = C;
                    }
                }
                if (out && lane == 0) {
                    BW[y][c][0] = BX;
                    BW[y][c][1] = BY;
                }
            }
        }
        {
            // (a run's first site is its node: column 0 and column 64 start runs,
            // the node of a row's last site was kept by its lane; the rows may
            // have left the queue full)
            if (qn > QCAP - CH * RP) drain();
            const uint32_t row = (y0 + lane) * L;
            push(wrap, LN[wave][last_c][lane & (RP - 1)], row);
            if (CH > 1) push(join, LN[wave][0][lane & (RP - 1)], row + 64);
        }
        drain();
        if (meas) {
            if (meas_prev) count_flush();
            if (lane == 0 && n_act) atomicAdd(&tot[1], n_act);
        }
        __syncthreads();
        // ---- 2. seams
        uint32_t active = 0;
        if (meas) {
            active = tot[1];
            if (meas_prev) write_record(active_prev);
        }
        if (rows) {
            const uint32_t pw = wave ? wave - 1 : ns - 1;
#pragma unroll
            for (uint32_t c = 0; c < CH; ++c) {
                const uint64_t mv = MB[pw][c][0], mc = MB[pw][c][1];
                const uint32_t up = HB[pw][64 * c + lane];
                const uint64_t V = uniform64(mv), Cu = uniform64(mc);
                push(V & ~((V << 1) & C0[c] & Cu) & ballot(up != lab[0][c]), up, lab[0][c]);
            }
            drain();
        }
        __syncthreads();
        // ---- 3. roots draw their clusters' states; every other label's entry is
        // pointed at its root (labels are first sites of runs that took no label
        // from above, so their own lanes know them)
        {
            auto draw = [&]() {
                for (uint32_t j0 = 0; j0 < qn; j0 += 64) {
                    const uint32_t j = j0 + lane;
                    if (j < qn) {
                        const uint32_t r = lds_ld(&UQ[wave][j]);
                        lds_st(&P[r], TAG | state_of_draw(philox4x32_10(r, 0u, t, 1u, d.key0, d.key1).x, q));
                    }
                }
                qn = 0;
            };
            uint32_t p[RP][CH];
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j)
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c) {
                    const uint32_t li = (y0 + j) * L + 64 * c + lane;
                    p[j][c] = (j < rows && lane_in(columns(c)) && lab[j][c] == li) ? lds_ld(&P[li]) : 0xFFFFFFFFu;
                }
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j) {
                if (j >= rows) break;
                if (qn > QCAP - 64 * CH) draw();
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c) {
                    const uint32_t li = (y0 + j) * L + 64 * c + lane;
                    const uint64_t m = ballot(p[j][c] == li);
                    if (lane_in(m)) lds_st(&UQ[wave][qn + lanes_below(m)], li);
                    qn += popc64(m);
                }
            }
            draw();
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j) {
                if (j >= rows) break;
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c) {
                    const uint32_t li = (y0 + j) * L + 64 * c + lane;
                    uint32_t r = p[j][c];
                    if (r < li) {   // (not a root; entries only point at smaller sites)
                        uint32_t up = lds_ld(&P[r]);
                        while (up < r) {
                            r = up;
                            up = lds_ld(&P[r]);
                        }
                        bad |= up != r && !(up & TAG);
                        lds_st(&P[li], r);
                    }
                }
            }
        }
        __syncthreads();
        // ---- 4. every site takes its cluster's state: its label's entry is the
        // root's state or the root, whose entry is the state
        {
            uint32_t e[RP][CH], st[RP][CH];
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j)
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c) {
                    const bool in = j < rows && lane_in(columns(c));
                    e[j][c] = in ? lab[j][c] : 0u;
                    st[j][c] = lds_ld(&P[e[j][c]]);
                }
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j)
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c)
                    if (!(st[j][c] & TAG)) {
                        e[j][c] = st[j][c];
                        st[j][c] = lds_ld(&P[e[j][c]]);
                    }
#pragma unroll
            for (uint32_t j = 0; j < RP; ++j) {
                if (j >= rows) break;
#pragma unroll
                for (uint32_t c = 0; c < CH; ++c) {
                    const uint32_t y = y0 + j, x = 64 * c + lane;
                    if (x < L) {
                        const uint8_t v = (uint8_t)st[j][c];
                        bad |= !(st[j][c] & TAG);
                        s[y * SPS + x] = v;
                        if (out) glb(d.lab)[y * L + x] = e[j][c];
                    }
                }
            }
            if (k + 1 < n) draws(t + 1);
            if (meas) {
                if (tid < 256) hist[tid] = 0;
                if (tid < 2) tot[tid] = 0;
            }
            active_prev = active;
        }
        __syncthreads();
    }

    if (meas) {
        // the last sweep's result
        for (uint32_t j = 0; j < rows; ++j)
            for (uint32_t c = 0; c <= last_c; ++c) {
                const uint32_t y = y0 + j, x = 64 * c + lane;
                const uint64_t vm = columns(c);
                const uint32_t s0 = s[y * SPS + x], sr = s[y * SPS + (x + 1 == L ? 0u : x + 1)], sd = s[below(y) * SPS + x];
                count_row(vm, s0, ballot(s0 == sr) & vm, ballot(s0 == sd) & vm);
            }
        count_flush();
        __syncthreads();
        write_record(active_prev);
        // the record after it starts from zero (the tile kernels add into it)
        const gptr<int64_t> rec = glb(d.ring) + (size_t)slot * words;
        for (uint32_t i = tid; i < words; i += NT) rec[i] = 0;
    }
    for (uint32_t i = tid; i < N; i += NT) {
        const uint32_t y = div_L(d, i), x = i - y * L;
        glb(d.s)[i] = s[y * SPS + x];
    }
    if (flags & 1u) {
        for (uint32_t i = tid; i < L * CH * 2; i += NT) {
            const uint32_t y = i / (CH * 2), c = (i / 2) % CH, pl = i & 1u;
            if (c <= last_c) glb(d.bonds)[((size_t)((y / ty) * d.ntx + c) * 2 + pl) * ty + y % ty] = BW[y][c][pl];
        }
    }
    if (bad) flag_error(d.err);
    if (tid == 0 && (flags & 1u)) *glb(d.labels) = LABELS_SITE;
    if (tid == 0 && !(flags & 2u)) *glb(d.counter) = t0 + n;
}

}  // namespace

hipError_t launch_whole(const LatDesc* descs, const uint32_t* list, uint32_t count, uint32_t lmax,
                        uint32_t n_uniform, const uint32_t* n_each, uint32_t flags, uint32_t ty, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    const auto go = [&](auto kernel, uint32_t nw) {
        hipLaunchKernelGGL(kernel, dim3(count), dim3(64 * nw), 0, s, descs, list, n_uniform, n_each, flags, ty);
        return hipGetLastError();
    };
    if (lmax > WHOLE_LMAX) return hipErrorInvalidValue;
    if (lmax > 64) return go(k_whole<128, 16>, 16);
    // Sixteen waves (80 registers) fill a CU's share alone; with more lattices than
    // CUs, eight waves let two be swept side by side and four waves four, each
    // longer than by itself.  us a sweep with 16 / 8 / 4 waves, and with the kernel
    // of 256 threads that was before:
    //   256 lattices    L = 8 4.1 / 4.5 / 6.0 (6.1)      L = 64 10.0 / 12.4 / 20.2 (26)
    //   512             L = 8 7.8 / 5.2 / 6.7 (6.9)      L = 64 19.6 / 16.3 / 23.3 (31)
    //   640             L = 8 11.5 / 8.7 / 7.3 (7.9)     L = 64 28.7 / 24.9 / 26.5 (38)
    //   4096            L = 8 59.6 / 37.2 / 29.1 (37)    L = 64 150 / 111 / 108 (180)
    if (count <= CUS) return go(k_whole<64, 16>, 16);
    if (count <= 2 * CUS) return go(k_whole<64, 8>, 8);
    return go(k_whole<64, 4>, 4);
}

}  // namespace swmi
