// The classical XY model swept by the same SW multi-cluster machinery, with
// Wolff's embedded clusters (the extension named in Sec. 5 of the paper): a
// random direction r = (cos phi, sin phi) per sweep, the projections
// c_i = cos(theta_i - phi), a bond between neighbours with c_i c_j > 0 active
// with probability 1 - exp(-2K c_i c_j), and every cluster reflected across
// the line perpendicular to r with probability 1/2.
//
// Only the bond step and the measurement are the model's own (this file);
// the labelling runs the Potts labeller over the bond words written here, the
// cross-tile merge is shared unchanged, and the flip is the Potts flip's
// per-cluster walk with a reflection bit in place of a new state.
//
// Angles are uint32 fractions of a full turn (unit 2^-32).  sin and cos of an
// angle take off its nearest quarter turn in integer arithmetic (exact) and
// evaluate the rest, at most an eighth of a turn, in FP64 by Taylor
// polynomials, then rotate by the quarter turns; a site's projection on the
// direction and the cos and sin of its bonds' angle differences follow from
// products of those values.  The bond test is the FP64 rule u < -expm1(-y),
// with an FP32 estimate deciding whenever u is far enough from the threshold.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sw_device.hpp"
#include "sw_kernels.hpp"
#include "sw_tile.hpp"

namespace swmi {

namespace {

constexpr double PI_2_31 = 3.14159265358979323846264338327950288 / 2147483648.0;   // pi / 2^31

// a * b + k rounded once, for a constant k, as the three-operand FP64 fused
// multiply-add (left to itself the compiler copies k into the destination of
// the two-operand multiply-accumulate first, one more instruction per step).
__device__ __forceinline__ double fma_k(double a, double b, double k)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
}

// v with its sign changed if bit 31 of k is set.
__device__ __forceinline__ double flip_sign(double v, uint32_t k)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v) ^ ((uint64_t)(k & 0x80000000u) << 32);
    return __longlong_as_double((long long)b);
}

// sin and cos of the angle a (a fraction a / 2^32 of a turn).  With k the
// nearest quarter turn and d = a - k 2^30 in [-2^29, 2^29), x = d pi / 2^31
// lies in [-pi/4, pi/4); the Taylor series of sin to x^17 and of cos to x^18
// leave out less than 1e-19 there.
__device__ __forceinline__ void sincos_turn(uint32_t a, double& s, double& c)
{
    const uint32_t k = a + 0x20000000u;   // the quarter turn in the top two bits
    const int32_t d = (int32_t)(a - (k & 0xC0000000u));
    const double x = (double)d * PI_2_31;
    const double x2 = x * x;
    // sin x = x + x^3 (-1/3! + x^2 (1/5! - ...)), cos x = 1 + x^2 (-1/2! + x^2 (1/4! - ...))
    double ps = 1.0 / 355687428096000.0;           // 1/17!
    ps = fma_k(ps, x2, -1.0 / 1307674368000.0);      // 1/15!
    ps = fma_k(ps, x2, 1.0 / 6227020800.0);          // 1/13!
    ps = fma_k(ps, x2, -1.0 / 39916800.0);           // 1/11!
    ps = fma_k(ps, x2, 1.0 / 362880.0);              // 1/9!
    ps = fma_k(ps, x2, -1.0 / 5040.0);               // 1/7!
    ps = fma_k(ps, x2, 1.0 / 120.0);                 // 1/5!
    ps = fma_k(ps, x2, -1.0 / 6.0);                  // 1/3!
    const double sx = fma(x * x2, ps, x);
    double pc = 1.0 / 6402373705728000.0;          // 1/18!
    pc = fma_k(pc, x2, -1.0 / 20922789888000.0);     // 1/16!
    pc = fma_k(pc, x2, 1.0 / 87178291200.0);         // 1/14!
    pc = fma_k(pc, x2, -1.0 / 479001600.0);          // 1/12!
    pc = fma_k(pc, x2, 1.0 / 3628800.0);             // 1/10!
    pc = fma_k(pc, x2, -1.0 / 40320.0);              // 1/8!
    pc = fma_k(pc, x2, 1.0 / 720.0);                 // 1/6!
    pc = fma_k(pc, x2, -1.0 / 24.0);                 // 1/4!
    pc = fma_k(pc, x2, 0.5);                         // the 1/2! term, subtracted below
    const double cx = fma(-x2, pc, 1.0);
    // rotate by k quarter turns: sin and cos change places for odd k; sin changes
    // sign for k = 2, 3 and cos for k = 1, 2 (sign bits taken from k itself)
    const bool odd = k & 0x40000000u;
    const double ss = odd ? cx : sx, cc = odd ? sx : cx;
    s = flip_sign(ss, k);
    c = flip_sign(cc, k + 0x40000000u);
}

// Observable sums: a term v (|v| <= 1) counts as v 2^30 rounded to an integer (to
// nearest, ties to even).  1.5 2^52 + v 2^30, rounded once, is that integer in
// the low bits of a double whose spacing there is one, so the bits of such
// doubles can be added as 64-bit integers; FX_ZERO is the bits of a zero term.
// Two instructions a term (multiply, round, add in FP64: three).
constexpr double FX_BASE = 6755399441055744.0;   // 1.5 * 2^52
constexpr uint64_t FX_ZERO = 0x4338000000000000ull;

__device__ __forceinline__ void fx30_add(uint64_t& acc, double v, double two30)
{
    acc += (uint64_t)__double_as_longlong(fma_k(v, two30, FX_BASE));
}

// The projection cos(theta - phi) = cos theta cos phi + sin theta sin phi,
// rounded product by product (no fused multiply-add): for a spin exactly a
// quarter turn from phi the two products are equal and opposite (the quarter
// turn only permutes and negates the polynomial values), so it is exactly 0.
__device__ __forceinline__ double projection(double s, double c, double sphi, double cphi)
{
    return __dadd_rn(__dmul_rn(c, cphi), __dmul_rn(s, sphi));
}

// The bond rule u < 1 - exp(-y), y >= 0 (may be +inf), decided as in FP64: an
// FP32 estimate of u - (1 - exp(-y)) from the top 32 bits of u is within 10^-6
// of the FP64 value (the exponential's own error, its argument's and three
// roundings are a few 10^-7, the bits left out of u 2^-32), so when it is larger
// than BOND_MARGIN in magnitude its sign decides, else FP64 expm1 does (one
// test in 10^5).
constexpr float BOND_MARGIN = 1.0f / 262144.0f;

__device__ __forceinline__ bool bond_exact(uint32_t wa, uint32_t wb, double y)
{
    const double u = (double)((((uint64_t)wa) << 21) | (wb >> 11)) * 0x1p-53;
    return u < -expm1(-y);
}

// The value of the lane whose number times four is addr.
__device__ __forceinline__ double lane_value(double v, uint32_t addr)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)addr, (int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)addr, (int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ long long wave_sum_i64(long long v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, o), hi = (uint32_t)__shfl_xor((int)(uint32_t)((uint64_t)v >> 32), o);
        v += (long long)(((uint64_t)hi << 32) | lo);
    }
    return v;
}

__device__ __forceinline__ int64_t* xy_record(const LatDesc& d, uint32_t sweep, uint32_t copy)
{
    return d.ring + ((size_t)(sweep % d.cap) * NCOPY + copy) * XY_STRIDE;
}

// ---------------------------------------------------------------------------
// Bonds of sweep t = counter + k, and/or the measurement of a configuration.
//
// flags bit 0: also measure the incoming configuration (the result of sweep
// t - 1) into record t - 1; bit 1: only measure the current configuration
// into record t (no bonds; k = 0xFFFFFFFF names the last sweep done).
//
// One workgroup per tile, one column per lane, each wave a strip of rows.
// Every site evaluates sin and cos of its own angle once; its projection, the
// pair terms cos and sin(theta_i - theta_j) of its +x and +y bonds and its
// magnetisation terms are products of those with the direction's and the
// neighbours' (the right-hand lane's, the next row's; the column right of the
// tile is evaluated once per tile).  A site's +x and +y bonds use one Philox
// call (counter (i, 0, t, 4)): words 0, 1 make the 53-bit uniform of the +x
// bond, words 2, 3 that of the +y bond.  The bond words go to the tile-major
// bond plane the labeller reads.
//
// Bound by vector issue: 138 instructions per row of 64 sites (36 Philox, 35
// sin and cos, 20 the two bond tests, 20 the six sums), 1.12 ms at L = 16384
// with measurement; 172 and 1.50 ms with the tests' estimates formed in FP64
// from 53-bit uniforms, projections computed twice and three instructions per
// term of the sums.
template <int TY, uint32_t NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4))) void k_xy_bonds(const LatDesc* descs, const WorkItem* map, uint32_t k,
                                                               uint32_t flags)
{
    constexpr uint32_t RPW = TY / NW;
    __shared__ unsigned long long acc[XY_WORDS];   // n_active, Ex, Ey, Ix, Iy, Mx, My
    __shared__ double sedge[TY], cedge[TY];        // sin, cos of the column right of the tile

    LatDesc d;
    uint32_t tile, lat;
    if (!pick(descs, map, blockIdx.x, true, d, tile, lat)) return;
    const TileGeom g = tile_geom(d, tile, TY);
    const uint32_t t = *glb(d.counter) + k;
    const bool only_measure = (flags & 2u) != 0;
    const bool meas = d.cap != 0 && (flags & 3u) != 0;
    const uint32_t tid = threadIdx.x, wave = wave_id(), lane = tid & 63u;
    const uint32_t L = d.L, w = g.w, h = g.h, x0 = g.x0, y0 = g.y0;
    const gptr<uint32_t> ang = glb(d.ang);
    const uint32_t xe = (x0 + w == L) ? 0u : x0 + w;   // the column right of the tile

    if (tid < XY_WORDS) acc[tid] = 0ull;
    if (tid < h) {
        double se, ce;
        sincos_turn(ang[(y0 + tid) * L + xe], se, ce);
        sedge[tid] = se;
        cedge[tid] = ce;
    }
    __syncthreads();

    double sphi, cphi;
    sincos_turn(xy_direction(d, t), sphi, cphi);
    const bool vx = lane < w;
    const bool edge = lane == w - 1;
    const uint32_t x = x0 + (vx ? lane : 0u);
    const uint32_t r0 = wave * RPW, r1 = min(h, r0 + RPW);
    const uint64_t validm = (w == 64) ? ~0ull : ((1ull << w) - 1ull);
    const double k2 = d.k2;
    const PhiloxKeys ks = philox_keys_v(d.key0, d.key1);
    const gptr<uint64_t> bw = glb(d.bonds) + (size_t)tile * 2 * TY;
    uint32_t n_active = 0;   // wave-uniform
    uint64_t ex = 0, ey = 0, ix = 0, iy = 0, mx = 0, my = 0;
    const float kf = (float)(-k2 * 1.4426950408889634074);   // -2K log2 e
    const uint32_t right = ((lane + 1u) & 63u) * 4u;
    double two30 = 1073741824.0;
    asm("" : "+v"(two30));   // in vector registers: fx30_add's other constant takes the scalar operand

    if (r0 < r1) {
        // tile row rr of this column (row h is the first row of the tile below,
        // or row 0 of the lattice), from a wave-uniform base
        auto row_angle = [&](uint32_t rr) { return (ang + (size_t)((y0 + rr == L) ? 0u : y0 + rr) * L)[x]; };
        double si, ci;
        sincos_turn(row_angle(r0), si, ci);
        double pi_ = projection(si, ci, sphi, cphi);
        // site indices fit 32 bits (N <= 2^32)
        uint64_t m0 = PHILOX_M0 * (uint32_t)((y0 + r0) * L + x);
        const uint64_t m0_step = PHILOX_M0 * L;
        // the rows below are loaded two iterations ahead of their use
        uint32_t a1 = row_angle(r0 + 1), a2 = (r0 + 2 <= r1) ? row_angle(r0 + 2) : 0u;
        for (uint32_t r = r0; r < r1; ++r) {
            const uint32_t ad = a1;
            a1 = a2;
            if (r + 3 <= r1) a2 = row_angle(r + 3);
            const double s_right = lane_value(si, right), c_right = lane_value(ci, right);
            double sd, cd;
            sincos_turn(ad, sd, cd);
            const double sr = edge ? sedge[r] : s_right, cr = edge ? cedge[r] : c_right;
            if (!only_measure) {
                const double pr = projection(sr, cr, sphi, cphi);
                const double pd = projection(sd, cd, sphi, cphi);
                const u32x4 q = philox4x32_10_from(m0, t, 4u, ks);
                m0 += m0_step;
                // the estimates: c_i c_j keeps its sign and is no denormal in FP32
                // (a nonzero projection is above 2^-56); 2K may overflow to
                // infinity there, where exp(-y) is 0 in FP64 too
                const float fi = (float)pi_, fr = (float)pr, fd = (float)pd, ki = kf * fi;
                const float tx = fmaf((float)q.x, 0x1p-32f, __builtin_amdgcn_exp2f(ki * fr)) - 1.0f;
                const float ty = fmaf((float)q.z, 0x1p-32f, __builtin_amdgcn_exp2f(ki * fd)) - 1.0f;
                const uint64_t sx = ballot(fi * fr > 0.0f) & validm, sy = ballot(fi * fd > 0.0f) & validm;
                uint64_t BX = sx & ballot(tx < 0.0f), BY = sy & ballot(ty < 0.0f);
                const uint64_t nx = sx & ballot(!(fabsf(tx) >= BOND_MARGIN)), ny = sy & ballot(!(fabsf(ty) >= BOND_MARGIN));
                if (nx | ny) {
                    const double kc = k2 * pi_;
                    BX = (BX & ~nx) | (nx & ballot(bond_exact(q.x, q.y, kc * pr)));
                    BY = (BY & ~ny) | (ny & ballot(bond_exact(q.z, q.w, kc * pd)));
                }
                if (lane == 0) {
                    bw[r] = BX;
                    bw[TY + r] = BY;
                }
                n_active += popc64(BX) + popc64(BY);
                pi_ = pd;
            }
            if (meas) {
                // cos and sin of theta_i - theta_j from the two sites' sin and cos
                fx30_add(ex, fma(ci, cr, si * sr), two30);
                fx30_add(ix, fma(si, cr, -(ci * sr)), two30);
                fx30_add(ey, fma(ci, cd, si * sd), two30);
                fx30_add(iy, fma(si, cd, -(ci * sd)), two30);
                fx30_add(mx, ci, two30);
                fx30_add(my, si, two30);
            }
            si = sd;
            ci = cd;
        }
    }

    if (meas) {
        const uint64_t zero = (uint64_t)(r0 < r1 ? r1 - r0 : 0u) * FX_ZERO;
        const uint64_t v[6] = {ex, ey, ix, iy, mx, my};
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const long long sum = wave_sum_i64(vx ? (long long)(v[j] - zero) : 0ll);
            if (lane == 0 && sum) atomicAdd(&acc[1 + j], (unsigned long long)sum);
        }
    }
    if (!only_measure && lane == 0 && n_active) atomicAdd(&acc[0], (unsigned long long)n_active);
    __syncthreads();
    if (d.cap) {
        const uint32_t copy = blockIdx.x % NCOPY;
        if (!only_measure && tid == 0 && acc[0]) atomic_add_i64(&xy_record(d, t, copy)[0], acc[0]);
        if (meas && tid >= 1 && tid < XY_WORDS && acc[tid])
            atomic_add_i64(&xy_record(d, only_measure ? t : t - 1, copy)[tid], acc[tid]);
    }
}

// Initial angles: Philox counter (i, 0, 0, 6), word 0, or all zero.
__global__ __launch_bounds__(256) void k_xy_init(const LatDesc* descs, uint32_t random_start)
{
    const LatDesc d = descs[0];
    const size_t N = (size_t)d.L * d.L;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (size_t)gridDim.x * 256)
        glb(d.ang)[i] = random_start ? philox4x32_10((uint32_t)i, 0u, 0u, 6u, d.key0, d.key1).x : 0u;
}

}  // namespace

// Eight waves a tile where there is at most one tile per CU (a wave's strip of
// rows is then the kernel's latency), four elsewhere: whole XY sweeps at 64-row
// tiles with 4 / 8 waves take 45.9 / 41.3 us at 16 tiles, 52.1 / 47.7 at 169,
// 67.7 / 68.3 at 529, 138.8 / 146.8 at 2116 (each strip evaluates one row more
// than it owns; 16 waves: 41.0 and 47.5 us at 16 and 169 tiles).
constexpr uint32_t XY_FEW_TILES = 256;

template <int TY>
static hipError_t start_xy_bonds(const Work& w, uint32_t k, uint32_t flags)
{
    auto go = [&](auto nw) {
        constexpr uint32_t NW = decltype(nw)::value;
        return start_kernel(w, k_xy_bonds<TY, NW>, dim3(w.nitems), dim3(64 * NW), w.descs, w.map, k, flags);
    };
    if constexpr (TY == 64) {
        if (w.nitems <= XY_FEW_TILES) return go(std::integral_constant<uint32_t, 8>{});
        return go(std::integral_constant<uint32_t, 4>{});
    } else {
        return go(std::integral_constant<uint32_t, waves_of<TY>()>{});
    }
}

hipError_t launch_xy_bonds(const Work& w, uint32_t k, uint32_t flags)
{
    if (w.nitems == 0) return hipSuccess;
    switch (w.ty) {
    case 32: return start_xy_bonds<32>(w, k, flags);
    case 64: return start_xy_bonds<64>(w, k, flags);
    case 128: return start_xy_bonds<128>(w, k, flags);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_xy_init(const LatDesc* descs, size_t N, uint32_t random_start, hipStream_t s)
{
    const size_t b = (N + 255) / 256;
    const uint32_t grid = (uint32_t)(b < 65536 ? (b ? b : 1) : 65536);
    hipLaunchKernelGGL(k_xy_init, dim3(grid), dim3(256), 0, s, descs, random_start);
    return hipGetLastError();
}

}  // namespace swmi
