// 3-D paths of libsf: transmittance ray marching through a density grid
// (Sec. 5 "Offline rendering": density lookups with trilinear / tricubic
// filters and their stochastic one-lookup forms), emission ray marching
// through a temperature grid (Sec. 5 "Filtering nonlinear physical
// properties") and filtered point lookups.
//
// One lane marches one ray.  The stochastic kernel is the hot path: per step
// it forms the raster position, hashes (ray, sample, step, seed), picks one
// tap per axis by inverse CDF on the separable weights (Sec. 4.1 FRS) and
// gathers ONE voxel; the optical depth is a compensated binary32 sum.
#include <type_traits>

#include "volume_dev.hpp"

#pragma clang fp contract(off)

namespace sfk {

// Black-body emission (Sec. 5, "Filtering nonlinear physical properties"):
// spectral radiance in W sr^-1 m^-2 nm^-1 at 700, 546.1 and 435.8 nm of a
// temperature T in kelvin, B = A_l / (e^x - 1) with x = c2 / (lambda T).
// e^x is evaluated as exp2(K_l / T) on the transcendental unit; below
// x = 1/2 a degree-7 Taylor polynomial of e^x - 1 replaces the subtraction.
// T <= 0 emits nothing, NaN stays NaN.  Binary32 values (not decisions):
// the relative error is about (x + 3) ulp.
struct PlanckConst {
    static constexpr double h = 6.62607015e-34, c = 299792458.0, k = 1.380649e-23;
    static constexpr double A(double nm)
    {
        return 2.0 * h * c * c / (nm * 1e-9 * nm * 1e-9 * nm * 1e-9 * nm * 1e-9 * nm * 1e-9) * 1e-9;
    }
    static constexpr double K(double nm) { return h * c / (nm * 1e-9 * k) * 1.4426950408889634074; }
};

// e^x - 1 of y = x log2(e) below y = 0.72 (x = 1/2).
__device__ __forceinline__ float expm1_small(float y)
{
    const float x = y * 0.69314718f;
    float p = __builtin_fmaf(x, 1.0f / 5040.0f, 1.0f / 720.0f);
    p = __builtin_fmaf(x, p, 1.0f / 120.0f);
    p = __builtin_fmaf(x, p, 1.0f / 24.0f);
    p = __builtin_fmaf(x, p, 1.0f / 6.0f);
    p = __builtin_fmaf(x, p, 0.5f);
    p = __builtin_fmaf(x, p, 1.0f);
    return x * p;
}

// PLANCK_HOT: at and above it a band may need the polynomial.
constexpr float PLANCK_HOT = 41000.0f;

// The three bands side by side, not a branch per band (three exponentials one
// after the other under three execution masks): 1 Mi rays x 256 steps of the
// 512^3 fire, exact after, tricubic 14.2 ms with the branches and 10.5 without,
// trilinear 2.62 and 2.04; stochastic marches wait for their voxel either way
// (trilinear 535 and 528 us, tricubic 613 and 628).  The polynomial is needed
// only beyond 41,000 K: one test for the wavefront, on the band that needs it
// first (COOL: none, T is known to lie in [0, PLANCK_HOT)).
template <bool COOL = false>
__device__ __forceinline__ void planck3(float T, float B[3])
{
    constexpr float A[3] = {(float)PlanckConst::A(700.0), (float)PlanckConst::A(546.1), (float)PlanckConst::A(435.8)};
    constexpr float K[3] = {(float)PlanckConst::K(700.0), (float)PlanckConst::K(546.1), (float)PlanckConst::K(435.8)};
    constexpr float SMALL = 0.72134752f;
    float r = __builtin_amdgcn_rcpf(T);
    r = __builtin_fmaf(__builtin_fmaf(-T, r, 1.0f), r, r);   // one Newton step
    float y[3], em1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        y[k] = K[k] * r;   // x log2(e)
        em1[k] = __builtin_amdgcn_exp2f(y[k]) - 1.0f;   // +inf beyond y = 128: B = 0
    }
    static_assert(K[0] > 1.001f * SMALL * PLANCK_HOT && K[0] < K[1] && K[1] < K[2], "no polynomial below PLANCK_HOT");
    if (!COOL && __any(y[0] < SMALL)) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            em1[k] = y[k] < SMALL ? expm1_small(y[k]) : em1[k];
    }
    const bool cold = T < 0x1p-126f;   // subnormal too: its reciprocal is infinite
#pragma unroll
    for (int k = 0; k < 3; ++k)
        B[k] = cold ? 0.0f : A[k] * __builtin_amdgcn_rcpf(em1[k]);
}

// ---------------------------------------------------------------- ray march
template <int F, bool HALF, int VAR, bool DBG, bool OCC, bool P2>
__global__ __launch_bounds__(64 * MAX_SPLIT_WAVES) void k_ray_stoch(RaymarchCall c, SplitArgs sp)
{
    static_assert(!(DBG && OCC), "the tap dump records every step, so it never skips bricks");
    __shared__ float2 part[MAX_SPLIT_WAVES][64];
    RaySplit r(sp);
    const int64_t i = r.i;
    RayGeom g = {};
    int st = 3;   // no ray
    if (i < c.n)
        st = ray_setup_dev(c.vol.wmin, c.vol.scale, c.rays + 8 * i, c.steps, g);
    r.share(sp, sp.log_apart == sp.log_split || rays_together(g, st == 0, c.steps), c.steps);
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(c.vol.base), 0,
                                                                  (int)c.vol.bytes, kBufferFlags);
    // optical depth and the mean over samples as compensated binary32 sums:
    // tau within 2u tau of its exact value, so T = e^(-dt tau) within about
    // (2 tau + 3) u relative of the exact transmittance of the picked voxels
    __amdgpu_buffer_rsrc_t rm;
    if constexpr (OCC)
        rm = occ_rsrc(c.vol);
    CompSum Tsum;
    Tsum.init();
    for (int s = 0; s < c.spp; ++s) {
        CompSum tau;
        tau.init();
        if (st == 0) {
            StepHash h;
            h.init((uint32_t)i, (uint32_t)s, c.seed);
            // software pipeline: a step's voxel is added one step later, so its
            // load overlaps the next step's arithmetic
            uint32_t pend = 0;
            float kh = (float)r.first + 0.5f;
            const float dk = (float)r.stride;
            if constexpr (OCC) {
                // With the brick mask, the brick word of the next step is loaded
                // during step k as well, ahead of step k's voxel, and every step
                // loads a voxel (a step in an empty brick loads past the grid's
                // end and adds the 0.0 it reads, which leaves the compensated
                // sum unchanged): every pass then finds the same two loads in
                // flight in the same order, and a step waits only for loads
                // issued one step earlier.  Two steps per pass, so that the
                // state of step k + 1 is formed in place of step k - 1's.
                constexpr uint32_t kOut = HALF ? 0xfffffffeu : 0xfffffffcu;
                struct At {
                    float p[3];
                    int i0[3];
                    uint32_t word, bit;   // brick word and bit index
                };
                auto step = [&](int k, const At &cur, At &nxt) {
                    const bool empty = __builtin_amdgcn_ubfe(cur.word, cur.bit, 1u) != 0u;
                    kh += dk;
                    step_pos(g, kh, nxt.p, nxt.i0);
                    nxt.word = brick_word(rm, c.vol, nxt.i0, nxt.bit);
                    tau.add(bits_value<HALF>(pend));   // step k - 1
                    uint32_t off = kOut;
                    if (!empty) {
                        float t[3];
                        int o[3];
                        step_frac(cur.p, cur.i0, t);
                        pick3<F, VAR>(t, h.at((uint32_t)k), o);
                        off = voxel_offset_or_outside<HALF, P2>(c.vol, cur.i0[0] + o[0], cur.i0[1] + o[1],
                                                                 cur.i0[2] + o[2]);
                    }
                    pend = voxel_bits<HALF>(rs, off);  // step k
                };
                At a, b;
                step_pos(g, kh, a.p, a.i0);
                a.word = brick_word(rm, c.vol, a.i0, a.bit);
                // a first load of zero behind the first brick word (its offset
                // depends on the brick index so that it is not moved ahead)
                __builtin_amdgcn_sched_barrier(0);
                pend = voxel_bits<HALF>(rs, kOut | (a.bit >> 31));
                int k = r.first;
                for (; k + r.stride < c.steps; k += 2 * r.stride) {
                    step(k, a, b);
                    step(k + r.stride, b, a);
                }
                if (k < c.steps)
                    step(k, a, b);
                tau.add(bits_value<HALF>(pend));
            } else {
                for (int k = r.first; k < c.steps; k += r.stride, kh += dk) {
                    int i0[3], o[3];
                    float p[3], t[3];
                    step_pos(g, kh, p, i0);
                    step_frac(p, i0, t);
                    pick3<F, VAR>(t, h.at((uint32_t)k), o);
                    int x = i0[0] + o[0], y = i0[1] + o[1], z = i0[2] + o[2];
                    if constexpr (DBG) {
                        int32_t *tp = c.taps + (((int64_t)i * c.spp + s) * c.steps + k) * 3;
                        tp[0] = x;
                        tp[1] = y;
                        tp[2] = z;
                    }
                    const uint32_t off = voxel_offset_or_outside<HALF, P2>(c.vol, x, y, z);
                    tau.add(bits_value<HALF>(pend));     // step k-1
                    pend = voxel_bits<HALF>(rs, off);    // step k (0 outside the grid)
                }
                tau.add(bits_value<HALF>(pend));
            }
        }
        if (sp.log_split) {
            // the wavefronts' sums meet in order
            part[r.wave][r.lane] = make_float2(tau.s, tau.c);
            __syncthreads();
            if (r.part == 0)
                for (int q = 1; q < r.parts; ++q) {
                    const float2 t = part[r.wave + q][r.lane];
                    tau.add(t.x);
                    tau.c += t.y;
                }
            __syncthreads();
        }
        Tsum.add(expf(-(g.dt * tau.value())));
    }
    if (r.part != 0 || st == 3)
        return;
    if (st != 0) {
        c.T[i] = st == 1 ? 1.0f : __builtin_nanf("");
        if constexpr (DBG) {
            int64_t per = (int64_t)3 * c.spp * c.steps;
            for (int64_t k = 0; k < per; ++k)
                c.taps[per * i + k] = SF_TAP_NONE;
        }
        return;
    }
    c.T[i] = Tsum.value() / (float)c.spp;
}

// ------------------------------------------------- every tap of every step
// The deterministic marches read all taps of a step.  Neighbouring rays read
// overlapping boxes of voxels, and so do neighbouring steps of a ray (a step
// is about two voxels long, its taps span four), so reading each ray's rows
// by itself is bound by the L1: 33 cache accesses per 64-lane row load, 16
// such loads per tricubic step.  A wavefront therefore copies the box that
// holds the taps of all its rays over up to STAGE_STEPS steps into LDS, as
// binary32, and takes the taps from there.  A box that does not fit
// (incoherent rays, sparse pixels) is tried over fewer steps and then given
// up: those steps' taps are read from the grid, all loads of a step (or two
// of its four planes) on their way before the first is used.  Values and order
// of summation are the same either way.
// One tap per step is always read from the grid (1 Mi rays x 256 steps, 256^3
// binary16 cloud: 265 us, from boxes 768).  A box of eight taps per ray has to
// serve four steps to be worth its wait, one of 64 taps a single one.
// Units of 16 bytes per wavefront and wavefronts per SIMD, within 160 KiB per
// CU: for two taps per axis 480 and five (1 Mi rays x 256 steps, before, 512^3
// cloud: binary32 905 us, 320 and eight 1,382, 640 and four 938; binary16 946,
// 1,176 and 990), for four 640 and four.
template <int F>
constexpr int STAGE_UNITS = F == NEAREST ? 0 : (Taps<F>::n == 2 ? 480 : 640);
template <int F>
constexpr int STAGE_WAVES = F == NEAREST ? 8 : (Taps<F>::n == 2 ? 5 : 4);
constexpr int STAGE_STEPS = 4;
template <int F>
constexpr int STAGE_LEAST = Taps<F>::n == 2 ? 4 : 1;   // steps worth a box
constexpr int STAGE_PAUSE = 8;     // steps read from the grid before a box is tried again

__device__ __forceinline__ int wave_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_max(int v) { return ~wave_min(~v); }

// Taps of one step read from the grid: load() issues the loads of the rows of
// planes c0.., value() makes the NT numbers of what came back for one row.
// PLANES: planes to issue before the first row is used (the wait for the loads
// is what such a step takes).
template <int F, bool HALF>
struct GridVoxels {
    static constexpr bool GRID = true;
    static constexpr int NT = Taps<F>::n, PLANES = NT == 4 ? 2 : NT;
    struct Raw {
        uint32_t w[NT];
    };
    const VolArgs &v;
    __amdgpu_buffer_rsrc_t rs;
    int x, y, z;     // first tap
    __device__ __forceinline__ GridVoxels(const VolArgs &vol, __amdgpu_buffer_rsrc_t r, const int i0[3])
        : v(vol), rs(r), x(i0[0] + Taps<F>::first), y(i0[1] + Taps<F>::first), z(i0[2] + Taps<F>::first)
    {
    }
    template <int P>
    __device__ __forceinline__ void load(int c0, Raw (&raw)[P][NT]) const
    {
#pragma unroll
        for (int cz = 0; cz < P; ++cz)
#pragma unroll
            for (int by = 0; by < NT; ++by)
#pragma unroll
                for (int a = 0; a < NT; ++a)
                    raw[cz][by].w[a] = voxel_bits<HALF>(
                        rs, voxel_offset_or_outside<HALF, false>(v, x + a, y + by, z + c0 + cz));
    }
    __device__ __forceinline__ void value(const Raw &r, float *t) const
    {
#pragma unroll
        for (int a = 0; a < NT; ++a)
            t[a] = bits_value<HALF>(r.w[a]);
    }
};

// Binary16 rows of four: one load per row where all of a step's taps lie
// inside the grid (rows4_inside), else voxel by voxel into the same words, so
// that the lanes of a wavefront at the grid's faces share what follows.
template <int MODE>
struct GridRows {
    static constexpr bool GRID = true;
    static constexpr int NT = 4, PLANES = MODE == BEFORE ? 4 : 2;
    typedef voxel_words Raw;
    const VolArgs &v;
    __amdgpu_buffer_rsrc_t rs;
    int x, y, z;     // first tap
    bool inside;
    __device__ __forceinline__ GridRows(const VolArgs &vol, __amdgpu_buffer_rsrc_t r, const int i0[3])
        : v(vol), rs(r), x(i0[0] - 1), y(i0[1] - 1), z(i0[2] - 1), inside(rows4_inside(vol, i0))
    {
    }
    template <int P>
    __device__ __forceinline__ void load(int c0, Raw (&raw)[P][4]) const
    {
        if (inside) {
            const uint32_t ys = (uint32_t)v.nx, zs = (uint32_t)v.ny * (uint32_t)v.nx;
            const uint32_t e0 = (uint32_t)(z + c0) * zs + (uint32_t)y * ys + (uint32_t)x;
#pragma unroll
            for (int cz = 0; cz < P; ++cz)
#pragma unroll
                for (int by = 0; by < 4; ++by)
                    raw[cz][by] = row4_load(rs, e0 + (uint32_t)cz * zs + (uint32_t)by * ys);
        } else {
#pragma unroll
            for (int cz = 0; cz < P; ++cz)
#pragma unroll
                for (int by = 0; by < 4; ++by) {
                    uint32_t h[4];
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        h[a] = voxel_bits<true>(
                            rs, voxel_offset_or_outside<true, false>(v, x + a, y + by, z + c0 + cz));
                    raw[cz][by] = {{h[0] | h[1] << 16, h[2] | h[3] << 16, 0u}, 0u};
                }
        }
    }
    __device__ __forceinline__ void value(const Raw &r, float *t) const { row4_values(r, t); }
};

template <int F, bool HALF, int MODE>
using GridTaps = std::conditional_t<HALF && Taps<F>::n == 4, GridRows<MODE>, GridVoxels<F, HALF>>;

// The staged box: nzb planes of nyb rows of u units of four voxels, from
// voxel (x0, y0, z0).  A plane takes an odd number of units, so that the
// planes' rows spread over the LDS banks.  Uniform over the wavefront.
struct StageBox {
    int x0, y0, z0, nyb, nzb, u, plane;
};

// Units of a box of nx x ny x nz voxels; more than MOST for a wider one.
template <int MOST>
__device__ __forceinline__ int box_units(int nx, int ny, int nz)
{
    const int u = (nx + 3) >> 2;
    const int plane = u <= MOST && ny <= MOST ? u * ny | 1 : MOST + 1;
    return plane <= MOST && nz <= MOST ? plane * nz : MOST + 1;
}

// Taps of one step read from the staged box.
template <int F>
struct StageTaps {
    static constexpr bool GRID = false;
    static constexpr int NT = Taps<F>::n, PLANES = 1;
    const float *p;
    int ys, zs;   // voxels per row and per plane
    __device__ __forceinline__ StageTaps(const float *vox, const StageBox &b, const int i0[3])
    {
        ys = 4 * b.u;
        zs = 4 * b.plane;
        p = vox + ((i0[2] + Taps<F>::first - b.z0) * zs + (i0[1] + Taps<F>::first - b.y0) * ys +
                   (i0[0] + Taps<F>::first - b.x0));
    }
    struct Raw {
        float t[NT];
    };
    template <int P>
    __device__ __forceinline__ void load(int c0, Raw (&raw)[P][NT]) const
    {
#pragma unroll
        for (int cz = 0; cz < P; ++cz)
#pragma unroll
            for (int by = 0; by < NT; ++by) {
                const float *r = p + ((c0 + cz) * zs + by * ys);
#pragma unroll
                for (int a = 0; a < NT; ++a)
                    raw[cz][by].t[a] = r[a];
            }
    }
    __device__ __forceinline__ void value(const Raw &r, float *t) const
    {
#pragma unroll
        for (int a = 0; a < NT; ++a)
            t[a] = r.t[a];
    }
};

// row(t, by, cz) for every row of the step's taps in order.
template <int NT, typename T, typename Row>
__device__ __forceinline__ void each_row(const T &taps, Row &&row)
{
    constexpr int PLANES = T::PLANES;
#pragma unroll
    for (int c0 = 0; c0 < NT; c0 += PLANES) {
        typename T::Raw raw[PLANES][NT];
        taps.load(c0, raw);
        if constexpr (T::GRID)
            __builtin_amdgcn_sched_barrier(0);   // all on their way
#pragma unroll
        for (int cz = 0; cz < PLANES; ++cz)
#pragma unroll
            for (int by = 0; by < NT; ++by) {
                float t[NT];
                taps.value(raw[cz][by], t);
                row(t, by, c0 + cz);
            }
    }
}

// Copy the box into LDS (all 64 lanes), voxels outside the grid as 0: each
// lane moves four voxels at a time, STAGE_LOADS loads in flight (a box is
// mostly one or two rounds).  Returns the largest voxel by bit pattern (a
// negative one, -0 and NaN above all others).
template <int F, bool HALF>
__device__ __forceinline__ uint32_t stage_box(const VolArgs &v, float *vox, const StageBox &b)
{
    typedef uint32_t u32x2_2 __attribute__((ext_vector_type(2), aligned(2)));   // rows start at any voxel
    typedef uint32_t u32x4_4 __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int STAGE_LOADS = HALF && Taps<F>::n == 4 ? 8 : 4, W = HALF ? 2 : 4;
    const int units = b.plane * b.nzb;
    // q / plane and rem / u for q < 1024 and divisors up to 641
    const uint32_t invp = (uint32_t)(1048576.0f / (float)b.plane) + 1u, invu = (uint32_t)(1048576.0f / (float)b.u) + 1u;
    const uint8_t *base = static_cast<const uint8_t *>(v.base);
    uint32_t top = 0;
    for (int q0 = threadIdx.x & 63; q0 < units; q0 += STAGE_LOADS * 64) {
        uint32_t w[STAGE_LOADS][W];
#pragma unroll
        for (int i = 0; i < STAGE_LOADS; ++i) {
            const int q = q0 + 64 * i;
#pragma unroll
            for (int k = 0; k < W; ++k)
                w[i][k] = 0u;
            const int zz = (int)(((uint32_t)q * invp) >> 20), rem = q - zz * b.plane;
            const int yy = (int)(((uint32_t)rem * invu) >> 20);
            const int gx = b.x0 + 4 * (rem - yy * b.u), gy = b.y0 + yy, gz = b.z0 + zz;
            if (q < units && yy < b.nyb && (uint32_t)gy < (uint32_t)v.ny && (uint32_t)gz < (uint32_t)v.nz) {
                const uint32_t e = ((uint32_t)gz * (uint32_t)v.ny + (uint32_t)gy) * (uint32_t)v.nx + (uint32_t)gx;
                if (gx >= 0 && gx + 4 <= v.nx) {
                    if constexpr (HALF) {
                        const u32x2_2 h = *reinterpret_cast<const u32x2_2 *>(base + (size_t)e * 2);
                        w[i][0] = h.x, w[i][1] = h.y;
                    } else {
                        const u32x4_4 h = *reinterpret_cast<const u32x4_4 *>(base + (size_t)e * 4);
                        w[i][0] = h.x, w[i][1] = h.y, w[i][2] = h.z, w[i][3] = h.w;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if ((uint32_t)(gx + k) >= (uint32_t)v.nx)
                            continue;
                        if constexpr (HALF)
                            w[i][k >> 1] |= (uint32_t)reinterpret_cast<const uint16_t *>(base)[e + (uint32_t)k]
                                            << (16 * (k & 1));
                        else
                            w[i][k] = reinterpret_cast<const uint32_t *>(base)[e + (uint32_t)k];
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < STAGE_LOADS; ++i) {
            const int q = q0 + 64 * i;
            float4 f;
            if constexpr (HALF)
                f = make_float4(half_bits_to_float((uint16_t)w[i][0]), half_bits_to_float((uint16_t)(w[i][0] >> 16)),
                                half_bits_to_float((uint16_t)w[i][1]), half_bits_to_float((uint16_t)(w[i][1] >> 16)));
            else
                f = make_float4(__uint_as_float(w[i][0]), __uint_as_float(w[i][1]), __uint_as_float(w[i][2]),
                                __uint_as_float(w[i][3]));
            if (q < units)
                reinterpret_cast<float4 *>(vox)[q] = f;
            top = max(max(top, __float_as_uint(f.x)), __float_as_uint(f.y));
            top = max(max(top, __float_as_uint(f.z)), __float_as_uint(f.w));
        }
    }
    return (uint32_t)wave_max((int)(top ^ 0x80000000u)) ^ 0x80000000u;
}

// The march over every tap: eval(wx, wy, wz, taps, largest) once for each
// step of this lane and wavefront that is not in a provably empty brick, in step
// order; `largest` bounds the step's taps from above if they are all
// non-negative, and is infinite otherwise.  Called by all lanes of a wavefront;
// `march` marks those with a ray.
template <int F, bool HALF, int MODE, bool OCC, typename Eval>
__device__ __forceinline__ void march_taps(const VolArgs &v, const RayGeom &g, bool march, bool together, int steps,
                                           const RaySplit &r, float *vox, Eval &&eval)
{
    constexpr int first = Taps<F>::first, last = Taps<F>::first + Taps<F>::n - 1;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(v.base), 0, (int)v.bytes, kBufferFlags);
    __amdgpu_buffer_rsrc_t rm;
    if constexpr (OCC)
        rm = occ_rsrc(v);
    const auto weigh = [&](int i0[3], const float t[3], float wx[4], float wy[4], float wz[4]) {
        if constexpr (F == NEAREST) {
#pragma unroll
            for (int a = 0; a < 3; ++a)
                i0[a] += t[a] >= 0.5f;
        }
        axis_weights<F>(t[0], wx);
        axis_weights<F>(t[1], wy);
        axis_weights<F>(t[2], wz);
    };
    int mtry = STAGE_STEPS;        // steps of the next box
    // Rays that lie apart or take too long steps never try a box, and their
    // wavefronts take the steps one by one, others in blocks of a box.
    bool boxes = false;
    if constexpr (STAGE_UNITS<F> > 0) {
        int e[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            e[a] = Taps<F>::n + (int)((STAGE_LEAST<F> - 1) * __builtin_fminf(__builtin_fabsf(g.G[a]), 1024.0f));
        boxes = together && __any(march && box_units<STAGE_UNITS<F>>(e[0], e[1], e[2]) <= STAGE_UNITS<F>);
    }
    const int block = boxes ? STAGE_STEPS : 1;
    int direct = boxes ? 0 : 0x7fffffff;   // steps to read from the grid before a box is tried
    int pause = STAGE_PAUSE;
    for (int kb = block * r.first; kb < steps; kb += block * r.stride) {
        const int k1 = min(kb + block, steps);
        for (int k = kb; k < k1;) {
            if (STAGE_UNITS<F> == 0 || direct > 0) {
                if (march) {
                    for (int kk = k; kk < k1; ++kk) {
                        int i0[3];
                        float t[3], wx[4], wy[4], wz[4];
                        step_coords(g, (float)kk + 0.5f, i0, t);
                        if constexpr (OCC) {
                            if (brick_empty_clamped(rm, v, i0))
                                continue;
                        }
                        weigh(i0, t, wx, wy, wz);
                        eval(wx, wy, wz, GridTaps<F, HALF, MODE>(v, rs, i0), __builtin_inff());
                    }
                }
                direct -= k1 - k;
                break;
            }
            const int m = min(mtry, k1 - k);
            // brick bits of the m steps; a lane takes part while it has one to read
            uint32_t full = 0;
            if constexpr (OCC) {
                if (march) {
#pragma unroll
                    for (int j = 0; j < STAGE_STEPS; ++j) {
                        if (j < m) {
                            float p[3];
                            int i0[3];
                            step_pos(g, (float)(k + j) + 0.5f, p, i0);
                            full |= brick_empty_clamped(rm, v, i0) ? 0u : 1u << j;
                        }
                    }
                }
            } else {
                full = march ? (1u << m) - 1u : 0u;
            }
            if (!__any(full != 0u)) {   // nothing to read in these steps
                k += m;
                mtry = STAGE_STEPS;
                continue;
            }
            // the box of the wavefront's taps; a lane's cells lie between those
            // of the first and the last step (positions are linear in k)
            StageBox b;
            {
                float p[3];
                int ia[3], ib[3], lo[3], hi[3];
                step_pos(g, (float)k + 0.5f, p, ia);
                step_pos(g, (float)(k + m - 1) + 0.5f, p, ib);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    lo[a] = wave_min(full ? min(ia[a], ib[a]) : 0x3fffffff);
                    hi[a] = wave_max(full ? max(ia[a], ib[a]) : -0x3fffffff);
                }
                const int nx = hi[0] - lo[0] + 1 + last - first, ny = hi[1] - lo[1] + 1 + last - first,
                          nz = hi[2] - lo[2] + 1 + last - first;
                const int units = box_units<STAGE_UNITS<F>>(nx, ny, nz);
                if (units > STAGE_UNITS<F>) {
                    if (m > STAGE_LEAST<F>) {
                        mtry = m >> 1;
                    } else {
                        direct = pause;
                        pause *= 2;
                        mtry = STAGE_STEPS;
                    }
                    continue;
                }
                // as many steps as can be next time if twice the box would fit
                mtry = 2 * units <= STAGE_UNITS<F> ? STAGE_STEPS : m;
                pause = STAGE_PAUSE;
                b.x0 = lo[0] + first, b.y0 = lo[1] + first, b.z0 = lo[2] + first;
                b.nyb = ny, b.nzb = nz, b.u = (nx + 3) >> 2, b.plane = b.u * ny | 1;
            }
            // Lanes read what others of the wavefront wrote: its LDS instructions
            // run in order, the fences keep the compiler to it.
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint32_t top = stage_box<F, HALF>(v, vox, b);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const float largest = top < 0x7f800000u ? __uint_as_float(top) : __builtin_inff();
            for (int j = 0; j < m; ++j) {
                if (!((full >> j) & 1u))
                    continue;
                int i0[3];
                float t[3], wx[4], wy[4], wz[4];
                step_coords(g, (float)(k + j) + 0.5f, i0, t);
                weigh(i0, t, wx, wy, wz);
                eval(wx, wy, wz, StageTaps<F>(vox, b, i0), largest);
            }
            k += m;
        }
    }
}

// Deterministic comparators: all taps of the separable footprint per step.
// BEFORE: exp(-dt sum_k sum_i w_i sigma_i); AFTER: prod_k sum_i w_i e^{-dt sigma_i}.
// Binary32 throughout.  The AFTER product's factors are multiplied as
// binary32 pairs, and a step's factor f_k enters in the form that is known
// to a few ulp of itself: f_k = sum_i w_i e^{-dt sigma_i} when it is below
// 1/2, else 1 - a_k with a_k = sum_i w_i (1 - e^{-dt sigma_i}) (a factor
// close to 1 formed directly would carry the rounding of the binary32
// weights, which sum to 1 +- 3e-7, into every one of 256 factors).  Both
// modes then stay within about 20 u tau of the exact transmittance,
// tau = -ln T, u = 2^-24.
// Where a row's dt sigma_i all lie in [0, 1/16) (and 2^-24 <= dt <= 2^24, so
// that no power of it leaves binary32's range: with dt^4 infinite a zero tap
// would give NaN), 1 - e^{-x} is x times a cubic fitted to
// (1 - e^{-x})/x over that range (within 1.5e-9 of it, binary32 coefficients
// included), and no exponential is taken; where all of a step's do, f_k > 1/2
// and only a_k is formed.  Which form a row takes depends on its own taps
// alone.
// 1 Mi rays x 256 steps through the 512^3 binary16 cloud with a mask of 8^3
// bricks, ms before (each ray reading its own rows or taps) and now: tricubic
// after 8.1 -> 2.1, before 5.3 -> 1.5, trilinear after 2.4 -> 0.91, before
// 2.3 -> 0.78, nearest 0.50 -> 0.46 and 0.47 -> 0.42; both tricubic modes are
// bound by vector instructions (about 570 and 320 per 64-ray step) and the LDS
// reads of the rows together.
template <int F, bool HALF, int MODE, bool OCC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(STAGE_WAVES<F>))) void k_ray_det(RaymarchCall c, SplitArgs sp)
{
    // boxes, then the wavefronts' results
    __shared__ __attribute__((aligned(16))) float stage[4][STAGE_UNITS<F> ? 4 * STAGE_UNITS<F> : 6 * 64];
    RaySplit r(sp);
    const int64_t i = r.i;
    RayGeom g = {};
    int st = 3;   // no ray
    if (i < c.n)
        st = ray_setup_dev(c.vol.wmin, c.vol.scale, c.rays + 8 * i, c.steps, g);
    const bool together = rays_together(g, st == 0, c.steps);
    r.share(sp, together, c.steps);
    constexpr int NT = Taps<F>::n;
    const float dt = g.dt;
    CompSum tau;
    tau.init();
    PairProduct Tp;
    Tp.init();
    const float dt2 = dt * dt;
    const float c2 = dt2 * -0x1.ffffe8p-2f, c3 = (dt2 * dt) * 0x1.5542bcp-3f, c4 = (dt2 * dt2) * -0x1.4d42c4p-5f;
    const float small = dt >= 0x1p-24f && dt <= 0x1p24f ? 0.0625f : 0.0f;
    march_taps<F, HALF, MODE, OCC>(c.vol, g, st == 0, together, c.steps, r, stage[r.wave],
                             [&](const float *wx, const float *wy, const float *wz, auto taps, float largest) {
        float acc = 0.0f;
        if constexpr (MODE == BEFORE) {
            each_row<NT>(taps, [&](const float *t, int by, int cz) {
                float row = 0.0f;
#pragma unroll
                for (int ax = 0; ax < NT; ++ax)
                    row = __builtin_fmaf(wx[ax], t[ax], row);
                acc = __builtin_fmaf(wy[by] * wz[cz], row, acc);
            });
            tau.add(acc);
        } else {
            auto poly_row = [&](const float *t) {
                float row = 0.0f;
#pragma unroll
                for (int ax = 0; ax < NT; ++ax) {
                    float p = __builtin_fmaf(t[ax], c4, c3);
                    p = __builtin_fmaf(t[ax], p, c2);
                    p = __builtin_fmaf(t[ax], p, dt);
                    row = __builtin_fmaf(wx[ax], t[ax] * p, row);
                }
                return row;
            };
            // (`largest` is uniform, and so mostly is the outcome)
            if (!taps.GRID && largest * dt < small) {
                each_row<NT>(taps, [&](const float *t, int by, int cz) {
                    acc = __builtin_fmaf(wy[by] * wz[cz], poly_row(t), acc);
                });
                Tp.mul_one_minus(acc);
                return;
            }
            float accf = 0.0f;
            float wsum = wx[0];
#pragma unroll
            for (int ax = 1; ax < NT; ++ax)
                wsum += wx[ax];
            each_row<NT>(taps, [&](const float *t, int by, int cz) {
                float row = 0.0f, rowf = 0.0f;
                uint32_t top = __float_as_uint(t[0]);
#pragma unroll
                for (int ax = 1; ax < NT; ++ax)
                    top = max(top, __float_as_uint(t[ax]));
                if (top < 0x7f800000u && __uint_as_float(top) * dt < small) {
                    row = poly_row(t);
                    rowf = wsum - row;
                } else {
#pragma unroll
                    for (int ax = 0; ax < NT; ++ax) {
                        float e, m;
                        exp_neg_pair(t[ax] * dt, e, m);
                        row = __builtin_fmaf(wx[ax], m, row);
                        rowf = __builtin_fmaf(wx[ax], e, rowf);
                    }
                }
                const float wyz = wy[by] * wz[cz];
                acc = __builtin_fmaf(wyz, row, acc);
                accf = __builtin_fmaf(wyz, rowf, accf);
            });
            if (accf < 0.5f)
                Tp.mul(accf, 0.0f);
            else
                Tp.mul_one_minus(acc);
        }
    });
    if (sp.log_split) {
        // the wavefronts' results meet in order
        stage[r.wave][2 * r.lane] = MODE == BEFORE ? tau.s : Tp.hi;
        stage[r.wave][2 * r.lane + 1] = MODE == BEFORE ? tau.c : Tp.lo;
        __syncthreads();
        if (r.part == 0)
            for (int q = 1; q < r.parts; ++q) {
                const float a = stage[r.wave + q][2 * r.lane], b = stage[r.wave + q][2 * r.lane + 1];
                if constexpr (MODE == BEFORE) {
                    tau.add(a);
                    tau.c += b;
                } else {
                    Tp.mul(a, b);
                }
            }
    }
    if (r.part != 0 || st == 3)
        return;
    if (st != 0)
        c.T[i] = st == 1 ? 1.0f : __builtin_nanf("");
    else
        c.T[i] = MODE == BEFORE ? expf(-(dt * tau.value())) : Tp.value();
}

// ------------------------------------------------------------ emission march
// An emitting, non-absorbing medium of temperatures: a ray gathers
// dt * sum_k E_k at three wavelengths, E_k the step's emission.  Stochastic:
// E_k = B(T) of the one voxel the step picks (keys, picks and the occupancy
// skip as in the transmittance march; empty bricks emit nothing).  The sums
// are compensated binary32 sums of positive terms.
// Gaussian footprint perpendicular to the ray (Sec. 5: filtering after
// shading under minification): the plane's basis by the branchless
// construction of Duff et al., "Building an Orthonormal Basis, Revisited"
// (JCGT 6(1), 2017), scaled to raster axes A, B; per step the key
// (ray, sample | 2^31, step, seed) gives u0, u1 and Box-Muller with the
// contract ln and cos/sin moves p to fma(g2, B, fma(g1, A, p)).
struct PerpFrame {
    float A[3], B[3];
};

__device__ __forceinline__ PerpFrame perp_frame(const float *r8, const float *scale, float sigma)
{
    const float dx = r8[3], dy = r8[4], dz = r8[5];
    const float sg = __builtin_copysignf(1.0f, dz);
    const float a = -1.0f / (sg + dz);
    const float b = (dx * dy) * a;
    const float e1[3] = {1.0f + ((sg * dx) * dx) * a, sg * b, -sg * dx};
    const float e2[3] = {b, sg + (dy * dy) * a, -dy};
    PerpFrame f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        f.A[i] = (sigma * e1[i]) * scale[i];
        f.B[i] = (sigma * e2[i]) * scale[i];
    }
    return f;
}

// The samples of a ray are spread over G = 2^log_g adjacent lanes (a
// power of two up to 64, inside one wave) and its steps over 2^log_split
// wavefronts; the steps' sums meet in LDS and the samples' in a butterfly, so
// small images still fill the chip.
template <int F, bool HALF, int VAR, bool DBG, bool OCC, bool P2, bool JIT = false>
__global__ __launch_bounds__(64 * MAX_SPLIT_WAVES) void k_emit_stoch(RaymarchCall c, SplitArgs sp, int log_g)
{
    __shared__ float2 part[MAX_SPLIT_WAVES][64];
    RaySplit rg(sp);
    const int G = 1 << log_g;
    const int64_t i = rg.i >> log_g;
    const int lane = rg.lane & (G - 1);
    RayGeom g = {};
    int st = 3;   // no ray (the whole group of lanes shares i)
    if (i < c.n)
        st = ray_setup_dev(c.vol.wmin, c.vol.scale, c.rays + 8 * i, c.steps, g);
    rg.share(sp, sp.log_apart == sp.log_split || rays_together(g, st == 0, c.steps, lane == 0), c.steps);
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(c.vol.base), 0,
                                                                  (int)c.vol.bytes, kBufferFlags);
    __amdgpu_buffer_rsrc_t rm;
    if constexpr (OCC)
        rm = occ_rsrc(c.vol);
    CompSum acc[3];
    acc[0].init();
    acc[1].init();
    acc[2].init();
    PerpFrame pf = {};
    if constexpr (JIT)
        if (st == 0)
            pf = perp_frame(c.rays + 8 * i, c.vol.scale, c.footprint);
    for (int s = st == 0 ? lane : c.spp; s < c.spp; s += G) {
        StepHash h, hj;
        h.init((uint32_t)i, (uint32_t)s, c.seed);
        if constexpr (JIT)
            hj.init((uint32_t)i, (uint32_t)s | 0x80000000u, c.seed);
        uint32_t pend = 0;
        float kh = (float)rg.first + 0.5f;
        const float dk = (float)rg.stride;
        for (int k = rg.first; k < c.steps; k += rg.stride, kh += dk) {
            int i0[3], o[3];
            float t[3];
            if constexpr (JIT) {
                const uint3 wj = hj.at((uint32_t)k);
                const float rr = __builtin_sqrtf(-2.0f * lnc(1.0f - u24(wj.x)));
                float cs, sn;
                sincos2pi(u24(wj.y), cs, sn);
                const float g1 = rr * cs, g2 = rr * sn;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    float p = __builtin_fmaf(kh, g.G[a], g.E[a]);
                    p = __builtin_fmaf(g2, pf.B[a], __builtin_fmaf(g1, pf.A[a], p));
                    const float fl = __builtin_floorf(p);
                    i0[a] = (int)fl;
                    t[a] = p - fl;
                }
            } else {
                step_coords(g, kh, i0, t);
            }
            if constexpr (OCC) {
                if (brick_empty(rm, c.vol, i0))
                    continue;
            }
            pick3<F, VAR>(t, h.at((uint32_t)k), o);
            int x = i0[0] + o[0], y = i0[1] + o[1], z = i0[2] + o[2];
            if constexpr (DBG) {
                int32_t *tp = c.taps + (((int64_t)i * c.spp + s) * c.steps + k) * 3;
                tp[0] = x;
                tp[1] = y;
                tp[2] = z;
            }
            const uint32_t off = voxel_offset_or_outside<HALF, P2>(c.vol, x, y, z);
            float B[3];
            planck3(bits_value<HALF>(pend), B);    // step k-1
            acc[0].add(B[0]);
            acc[1].add(B[1]);
            acc[2].add(B[2]);
            pend = voxel_bits<HALF>(rs, off);      // step k (0 outside the grid)
        }
        float B[3];
        planck3(bits_value<HALF>(pend), B);
        acc[0].add(B[0]);
        acc[1].add(B[1]);
        acc[2].add(B[2]);
    }
    if (sp.log_split) {
        // the wavefronts' sums meet in order, as pairs, a band at a time
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (b)
                __syncthreads();   // the band before is read
            part[rg.wave][rg.lane] = make_float2(acc[b].s, acc[b].c);
            __syncthreads();
            if (rg.part == 0)
                for (int q = 1; q < rg.parts; ++q) {
                    const float2 t = part[rg.wave + q][rg.lane];
                    acc[b].add(t.x);
                    acc[b].c += t.y;
                }
        }
    }
    // the lanes' sums (at most 64, positive) meet in a butterfly
    float e[3] = {acc[0].value(), acc[1].value(), acc[2].value()};
    for (int m = G >> 1; m >= 1; m >>= 1) {
        e[0] += __shfl_xor(e[0], m);
        e[1] += __shfl_xor(e[1], m);
        e[2] += __shfl_xor(e[2], m);
    }
    if (st == 3 || rg.part != 0)
        return;
    if (st != 0) {
        const float v = st == 1 ? 0.0f : __builtin_nanf("");
        if (lane == 0) {
            c.T[3 * i] = v;
            c.T[3 * i + 1] = v;
            c.T[3 * i + 2] = v;
        }
        if constexpr (DBG) {
            const int64_t per = (int64_t)3 * c.steps;
            for (int s = lane; s < c.spp; s += G)
                for (int64_t k = 0; k < per; ++k)
                    c.taps[((int64_t)i * c.spp + s) * per + k] = SF_TAP_NONE;
        }
        return;
    }
    if (lane == 0) {
        const float sc = g.dt / (float)c.spp;
        c.T[3 * i] = e[0] * sc;
        c.T[3 * i + 1] = e[1] * sc;
        c.T[3 * i + 2] = e[2] * sc;
    }
}

// Deterministic emission (march_taps: 1 Mi rays x 256 steps of the 512^3
// binary16 fire with a mask of 8^3 bricks, tricubic after 28.5 -> 10.2 ms,
// bound by the transcendental unit, and before 5.4 -> 1.7 ms): E_k = B(sum_i w_i T_i) before shading,
// sum_i w_i B(T_i) after; binary32 weights and per-step sums of positive
// terms, steps summed with compensation.
template <int F, bool HALF, int MODE, bool OCC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(STAGE_WAVES<F>))) void k_emit_det(RaymarchCall c, SplitArgs sp)
{
    // boxes, then the wavefronts' results
    __shared__ __attribute__((aligned(16))) float stage[4][STAGE_UNITS<F> ? 4 * STAGE_UNITS<F> : 6 * 64];
    RaySplit r(sp);
    const int64_t i = r.i;
    RayGeom g = {};
    int st = 3;   // no ray
    if (i < c.n)
        st = ray_setup_dev(c.vol.wmin, c.vol.scale, c.rays + 8 * i, c.steps, g);
    const bool together = rays_together(g, st == 0, c.steps);
    r.share(sp, together, c.steps);
    constexpr int NT = Taps<F>::n;
    CompSum acc[3];
    acc[0].init();
    acc[1].init();
    acc[2].init();
    march_taps<F, HALF, MODE, OCC>(c.vol, g, st == 0, together, c.steps, r, stage[r.wave],
                             [&](const float *wx, const float *wy, const float *wz, auto taps, float largest) {
        if constexpr (MODE == BEFORE) {
            float T = 0.0f, B[3];
            each_row<NT>(taps, [&](const float *t, int by, int cz) {
                const float wyz = wy[by] * wz[cz];
#pragma unroll
                for (int ax = 0; ax < NT; ++ax)
                    T = __builtin_fmaf(wx[ax] * wyz, t[ax], T);
            });
            planck3(T, B);
            acc[0].add(B[0]);
            acc[1].add(B[1]);
            acc[2].add(B[2]);
        } else {
            float e[3] = {0.0f, 0.0f, 0.0f};
            // a plane at a time and its rows one by one, since all 64 taps side
            // by side take more registers than there are
            auto add_taps = [&](auto cool) {
#pragma unroll 1
                for (int cz = 0; cz < NT; ++cz) {
                    const float wzc = NT == 1 ? wz[0] : (NT == 2 ? (cz == 0 ? wz[0] : wz[1])
                                                  : (cz < 2 ? (cz == 0 ? wz[0] : wz[1]) : (cz == 2 ? wz[2] : wz[3])));
                    typename decltype(taps)::Raw raw[1][NT];
                    taps.load(cz, raw);
#pragma unroll
                    for (int by = 0; by < NT; ++by) {
                        float t[NT];
                        taps.value(raw[0][by], t);
                        const float wyz = wy[by] * wzc;
#pragma unroll
                        for (int ax = 0; ax < NT; ++ax) {
                            const float w = wx[ax] * wyz;
                            float B[3];
                            planck3<decltype(cool)::value>(t[ax], B);
                            e[0] = __builtin_fmaf(w, B[0], e[0]);
                            e[1] = __builtin_fmaf(w, B[1], e[1]);
                            e[2] = __builtin_fmaf(w, B[2], e[2]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            if (!taps.GRID && largest < PLANCK_HOT)
                add_taps(std::true_type{});
            else
                add_taps(std::false_type{});
            acc[0].add(e[0]);
            acc[1].add(e[1]);
            acc[2].add(e[2]);
        }
    });
    if (sp.log_split) {
        // the wavefronts' sums meet in order
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            stage[r.wave][6 * r.lane + 2 * b] = acc[b].s;
            stage[r.wave][6 * r.lane + 2 * b + 1] = acc[b].c;
        }
        __syncthreads();
        if (r.part == 0)
            for (int q = 1; q < r.parts; ++q)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    acc[b].add(stage[r.wave + q][6 * r.lane + 2 * b]);
                    acc[b].c += stage[r.wave + q][6 * r.lane + 2 * b + 1];
                }
    }
    if (r.part != 0 || st == 3)
        return;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        c.T[3 * i + b] = st == 0 ? acc[b].value() * g.dt : (st == 1 ? 0.0f : __builtin_nanf(""));
}

// ------------------------------------------------------------- point lookups
// Point lookups shaded by black-body emission: out is n x 3.
template <int F, bool HALF>
__device__ void filter3d_planck(const Filter3DCall &c, int64_t i, int i0[3], const float t[3],
                                __amdgpu_buffer_rsrc_t rs)
{
    CompSum acc[3];
    acc[0].init();
    acc[1].init();
    acc[2].init();
    if (c.mode == STOCH) {
        for (int s = 0; s < c.spp; ++s) {
            uint4 w4 = pcg4d(make_uint4((uint32_t)i, (uint32_t)s, 0u, c.seed));
            uint3 w = make_uint3(w4.x, w4.y, w4.z);
            int o[3];
            if (c.variant == 0)
                pick3<F, 0>(t, w, o);
            else
                pick3<F, 1>(t, w, o);
            int tx = i0[0] + o[0], ty = i0[1] + o[1], tz = i0[2] + o[2];
            if (c.taps) {
                int32_t *tp = c.taps + ((int64_t)i * c.spp + s) * 3;
                tp[0] = tx;
                tp[1] = ty;
                tp[2] = tz;
            }
            float B[3];
            planck3(voxel<HALF>(rs, c.vol, tx, ty, tz), B);
            for (int k = 0; k < 3; ++k)
                acc[k].add(B[k]);
        }
        for (int k = 0; k < 3; ++k)
            c.out[3 * i + k] = acc[k].value() / (float)c.spp;
        return;
    }
    constexpr int NT = Taps<F>::n;
    constexpr int F0 = Taps<F>::first;
    if constexpr (F == NEAREST) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            i0[a] += t[a] >= 0.5f;
    }
    float wx[4], wy[4], wz[4];
    axis_weights<F>(t[0], wx);
    axis_weights<F>(t[1], wy);
    axis_weights<F>(t[2], wz);
    // binary32 weights; the weighted terms are summed with compensation
    // (before: signed temperatures are allowed, so no positivity is assumed)
    for (int cz = 0; cz < NT; ++cz)
        for (int by = 0; by < NT; ++by)
            for (int ax = 0; ax < NT; ++ax) {
                const float wgt = (wx[ax] * wy[by]) * wz[cz];
                const float T = voxel<HALF>(rs, c.vol, i0[0] + F0 + ax, i0[1] + F0 + by, i0[2] + F0 + cz);
                if (c.mode == BEFORE) {
                    acc[0].add(wgt * T);
                } else {
                    float B[3];
                    planck3(T, B);
                    for (int k = 0; k < 3; ++k)
                        acc[k].add(wgt * B[k]);
                }
            }
    float B[3];
    if (c.mode == BEFORE)
        planck3(acc[0].value(), B);
    for (int k = 0; k < 3; ++k)
        c.out[3 * i + k] = c.mode == BEFORE ? B[k] : acc[k].value();
}

template <int F, bool HALF>
__global__ __launch_bounds__(256) void k_filter3d(Filter3DCall c)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= c.n)
        return;
    float x[3] = {c.pos[3 * i], c.pos[3 * i + 1], c.pos[3 * i + 2]};
    bool ok = __builtin_isfinite(x[0]) & __builtin_isfinite(x[1]) & __builtin_isfinite(x[2]);
    float p[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        p[a] = __builtin_fmaf(x[a] - c.vol.wmin[a], c.vol.scale[a], -0.5f);
        ok &= __builtin_fabsf(p[a]) <= 4194304.0f;
    }
    if (!ok) {
        const int ch = c.shade == SF_SHADE_PLANCK ? 3 : 1;
        for (int k = 0; k < ch; ++k)
            c.out[ch * i + k] = __builtin_nanf("");
        if (c.taps && c.mode == STOCH)
            for (int k = 0; k < 3 * c.spp; ++k)
                c.taps[(int64_t)3 * c.spp * i + k] = SF_TAP_NONE;
        return;
    }
    int i0[3];
    float t[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float fl = __builtin_floorf(p[a]);
        i0[a] = (int)fl;
        t[a] = p[a] - fl;
    }
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(c.vol.base), 0,
                                                                  (int)c.vol.bytes, kBufferFlags);
    const bool trans = c.shade == SF_SHADE_TRANSMITTANCE;
    if (c.shade == SF_SHADE_PLANCK) {
        filter3d_planck<F, HALF>(c, i, i0, t, rs);
        return;
    }
    if (c.mode == STOCH) {
        CompSum acc;
        acc.init();
        for (int s = 0; s < c.spp; ++s) {
            uint4 w4 = pcg4d(make_uint4((uint32_t)i, (uint32_t)s, 0u, c.seed));
            uint3 w = make_uint3(w4.x, w4.y, w4.z);
            int o[3];
            if (c.variant == 0)
                pick3<F, 0>(t, w, o);
            else
                pick3<F, 1>(t, w, o);
            int tx = i0[0] + o[0], ty = i0[1] + o[1], tz = i0[2] + o[2];
            if (c.taps) {
                int32_t *tp = c.taps + ((int64_t)i * c.spp + s) * 3;
                tp[0] = tx;
                tp[1] = ty;
                tp[2] = tz;
            }
            float sg = voxel<HALF>(rs, c.vol, tx, ty, tz);
            acc.add(trans ? expf(-(sg * c.ds)) : sg);
        }
        c.out[i] = acc.value() / (float)c.spp;
        return;
    }
    constexpr int NT = Taps<F>::n;
    constexpr int F0 = Taps<F>::first;
    if constexpr (F == NEAREST) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            i0[a] += t[a] >= 0.5f;
    }
    float wx[4], wy[4], wz[4];
    axis_weights<F>(t[0], wx);
    axis_weights<F>(t[1], wy);
    axis_weights<F>(t[2], wz);
    // binary32 weights, compensated sum (densities may be signed here)
    CompSum sum;
    sum.init();
    for (int cz = 0; cz < NT; ++cz)
        for (int by = 0; by < NT; ++by)
            for (int ax = 0; ax < NT; ++ax) {
                const float wgt = (wx[ax] * wy[by]) * wz[cz];
                const float sg = voxel<HALF>(rs, c.vol, i0[0] + F0 + ax, i0[1] + F0 + by, i0[2] + F0 + cz);
                const float v = (c.mode == BEFORE || !trans) ? sg : expf(-(sg * c.ds));
                sum.add(wgt * v);
            }
    float r = sum.value();
    if (c.mode == BEFORE && trans)
        r = expf(-(r * c.ds));
    c.out[i] = r;
}

// ---------------------------------------------------------- occupancy bricks
// One lane per bit of the mask (OccLayout): a padding bit is 0; a brick's
// bit is 1 when its box grown by 2 voxels on every side holds only zeros (a
// NaN counts as non-zero), the scan stopping at the first other voxel.  A
// wave's 64 bits are gathered with a ballot and written as two words.
template <bool HALF>
__global__ __launch_bounds__(256) void k_build_occ(VolArgs v, uint32_t *occ, int64_t words)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t bits = (int64_t)v.occ_sx * v.occ_sy * v.nbz;
    bool empty = false;
    if (b < bits) {
        const int bx = (int)(b % v.occ_sx), by = (int)((b / v.occ_sx) % v.occ_sy);
        const int bz = (int)(b / ((int64_t)v.occ_sx * v.occ_sy));
        if (bx < v.nbx && by < v.nby) {
            const int B = 1 << v.occ_log2;
            const int x0 = max(bx * B - 2, 0), x1 = min(bx * B + B + 2, v.nx);
            const int y0 = max(by * B - 2, 0), y1 = min(by * B + B + 2, v.ny);
            const int z0 = max(bz * B - 2, 0), z1 = min(bz * B + B + 2, v.nz);
            empty = true;
            for (int z = z0; z < z1 && empty; ++z)
                for (int y = y0; y < y1 && empty; ++y) {
                    const int64_t row = ((int64_t)z * v.ny + y) * v.nx;
                    for (int x = x0; x < x1; ++x) {
                        float val;
                        if constexpr (HALF)
                            val = half_bits_to_float(static_cast<const uint16_t *>(v.base)[row + x]);
                        else
                            val = static_cast<const float *>(v.base)[row + x];
                        empty &= val == 0.0f;
                    }
                }
        }
    }
    const uint64_t m = __ballot(empty);
    if ((threadIdx.x & 63) == 0) {
        const int64_t w0 = b >> 5;   // b is a multiple of 64 here
        if (w0 < words)
            occ[w0] = (uint32_t)m;
        if (w0 + 1 < words)
            occ[w0 + 1] = (uint32_t)(m >> 32);
    }
}

hipError_t launch_build_occupancy(const VolArgs &v, uint32_t *occ, hipStream_t s)
{
    const int64_t words = v.occ_bytes / 4;
    dim3 grid((uint32_t)((words * 32 + 255) / 256)), block(256);
    if (v.fmt == SF_R16F)
        k_build_occ<true><<<grid, block, 0, s>>>(v, occ, words);
    else
        k_build_occ<false><<<grid, block, 0, s>>>(v, occ, words);
    return hipGetLastError();
}

// ---------------------------------------------------------------- launchers
static uint32_t blocks_for(int64_t n) { return (uint32_t)((n + 255) / 256); }

template <int F>
constexpr MarchLanes DET_LANES = F == NEAREST   ? MarchLanes{1 << 19, 1 << 17, 1 << 19, false}
                                 : F == LINEAR ? MarchLanes{1 << 20, 1 << 16, 1 << 19, false}
                                               : MarchLanes{1 << 21, 1 << 18, 1 << 19, false};

template <int F, bool HALF, bool OCC, bool P2>
static void launch_ray_fo(const RaymarchCall &c, hipStream_t s)
{
    if (c.mode == STOCH) {
        const SplitGrid sg(c.n, c.steps, 4, STOCH_LANES);
        if (c.variant)
            k_ray_stoch<F, HALF, 1, false, OCC, P2><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
        else
            k_ray_stoch<F, HALF, 0, false, OCC, P2><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    } else if (c.mode == BEFORE) {
        const SplitGrid sg(c.n, c.steps, 2, DET_LANES<F>);
        k_ray_det<F, HALF, BEFORE, OCC><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    } else {
        const SplitGrid sg(c.n, c.steps, 2, DET_LANES<F>);
        k_ray_det<F, HALF, AFTER, OCC><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    }
}

template <int F, bool HALF>
static hipError_t launch_ray_f(const RaymarchCall &c, hipStream_t s)
{
    const bool p2 = c.vol.lx >= 0;
    if (c.mode == STOCH && c.taps) {
        // the tap dump records every step, so it never skips empty bricks
        const SplitGrid sg(c.n, c.steps, 4, STOCH_LANES);
        if (c.variant)
            k_ray_stoch<F, HALF, 1, true, false, false><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
        else
            k_ray_stoch<F, HALF, 0, true, false, false><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    } else if (c.vol.occ) {
        if (p2)
            launch_ray_fo<F, HALF, true, true>(c, s);
        else
            launch_ray_fo<F, HALF, true, false>(c, s);
    } else {
        if (p2)
            launch_ray_fo<F, HALF, false, true>(c, s);
        else
            launch_ray_fo<F, HALF, false, false>(c, s);
    }
    return hipGetLastError();
}

template <int F, bool HALF, int VAR, bool DBG, bool OCC, bool P2>
static void launch_emit_stoch(const RaymarchCall &c, hipStream_t s)
{
    const int G = lane_group(c.n, c.spp);
    const SplitGrid sg(c.n * G, c.steps, 4,
                       G > 2 ? SHARED_LANES : (c.footprint > 0.0f ? FOOTPRINT_LANES : STOCH_LANES));
    const int lg = __builtin_ctz(G);
    if (c.footprint > 0.0f)
        k_emit_stoch<F, HALF, VAR, DBG, OCC, P2, true><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args, lg);
    else
        k_emit_stoch<F, HALF, VAR, DBG, OCC, P2, false><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args, lg);
}

template <int F, bool HALF, bool OCC, bool P2>
static void launch_emit_fo(const RaymarchCall &c, hipStream_t s)
{
    if (c.mode == STOCH) {
        if (c.variant)
            launch_emit_stoch<F, HALF, 1, false, OCC, P2>(c, s);
        else
            launch_emit_stoch<F, HALF, 0, false, OCC, P2>(c, s);
    } else if (c.mode == BEFORE) {
        const SplitGrid sg(c.n, c.steps, 2, DET_LANES<F>);
        k_emit_det<F, HALF, BEFORE, OCC><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    } else {
        const SplitGrid sg(c.n, c.steps, 2, DET_LANES<F>);
        k_emit_det<F, HALF, AFTER, OCC><<<dim3(sg.blocks), dim3(sg.lanes), 0, s>>>(c, sg.args);
    }
}

template <int F, bool HALF>
static hipError_t launch_emit_f(const RaymarchCall &c, hipStream_t s)
{
    const bool p2 = c.vol.lx >= 0;
    if (c.mode == STOCH && c.taps) {
        if (c.variant)
            launch_emit_stoch<F, HALF, 1, true, false, false>(c, s);
        else
            launch_emit_stoch<F, HALF, 0, true, false, false>(c, s);
    } else if (c.vol.occ) {
        if (p2)
            launch_emit_fo<F, HALF, true, true>(c, s);
        else
            launch_emit_fo<F, HALF, true, false>(c, s);
    } else {
        if (p2)
            launch_emit_fo<F, HALF, false, true>(c, s);
        else
            launch_emit_fo<F, HALF, false, false>(c, s);
    }
    return hipGetLastError();
}

hipError_t launch_emission(const RaymarchCall &c, hipStream_t s)
{
    const bool half = c.vol.fmt == SF_R16F;
    switch (c.filter) {
    case NEAREST:
        return half ? launch_emit_f<NEAREST, true>(c, s) : launch_emit_f<NEAREST, false>(c, s);
    case LINEAR:
        return half ? launch_emit_f<LINEAR, true>(c, s) : launch_emit_f<LINEAR, false>(c, s);
    default:
        return half ? launch_emit_f<BSPLINE3, true>(c, s) : launch_emit_f<BSPLINE3, false>(c, s);
    }
}

hipError_t launch_raymarch(const RaymarchCall &c, hipStream_t s)
{
    const bool half = c.vol.fmt == SF_R16F;
    switch (c.filter) {
    case NEAREST:
        return half ? launch_ray_f<NEAREST, true>(c, s) : launch_ray_f<NEAREST, false>(c, s);
    case LINEAR:
        return half ? launch_ray_f<LINEAR, true>(c, s) : launch_ray_f<LINEAR, false>(c, s);
    default:
        return half ? launch_ray_f<BSPLINE3, true>(c, s) : launch_ray_f<BSPLINE3, false>(c, s);
    }
}

hipError_t launch_filter3d(const Filter3DCall &c, hipStream_t s)
{
    dim3 grid(blocks_for(c.n)), block(256);
    const bool half = c.vol.fmt == SF_R16F;
    switch (c.filter) {
    case NEAREST:
        if (half)
            k_filter3d<NEAREST, true><<<grid, block, 0, s>>>(c);
        else
            k_filter3d<NEAREST, false><<<grid, block, 0, s>>>(c);
        break;
    case LINEAR:
        if (half)
            k_filter3d<LINEAR, true><<<grid, block, 0, s>>>(c);
        else
            k_filter3d<LINEAR, false><<<grid, block, 0, s>>>(c);
        break;
    default:
        if (half)
            k_filter3d<BSPLINE3, true><<<grid, block, 0, s>>>(c);
        else
            k_filter3d<BSPLINE3, false><<<grid, block, 0, s>>>(c);
        break;
    }
    return hipGetLastError();
}

}  // namespace sfk
