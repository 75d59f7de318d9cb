// 2-D texture access helpers shared by the plain, anisotropic and
// compressed-texture kernels: coordinate wrap, raster position, MIP level
// choice, texel fetch, GGX shading and output store.
#pragma once
#include "sf_device.hpp"
#include "sf_internal.hpp"

#pragma clang fp contract(off)

namespace sfk {

__device__ __forceinline__ float wrap_coord(int wrap, float u)
{
    return wrap == SF_WRAP_REPEAT ? u - __builtin_floorf(u) : __builtin_fminf(__builtin_fmaxf(u, 0.0f), 1.0f);
}

// Taps lie in [-2, n+1]: one conditional add or subtract wraps them.
__device__ __forceinline__ int wrap_tap(int wrap, int i, int n)
{
    if (wrap == SF_WRAP_REPEAT) {
        int r = i < 0 ? i + n : (i >= n ? i - n : i);
        return n == 1 ? 0 : r;
    }
    return min(max(i, 0), n - 1);
}

// Any tap index (the FIS Gaussian reaches 25 texels past the point).
__device__ __forceinline__ int wrap_any(int wrap, int i, int n)
{
    if (wrap == SF_WRAP_REPEAT) {
        const int r = i % n;
        return r < 0 ? r + n : r;
    }
    return min(max(i, 0), n - 1);
}

__device__ __forceinline__ void raster(float u, int n, int &i0, float &t)
{
    float p = __builtin_fmaf(u, (float)n, -0.5f);
    float f = __builtin_floorf(p);
    i0 = (int)f;
    t = p - f;
}

__device__ __forceinline__ void levels_of(const Tex2DArgs &tx, float lam, int &l0, int &l1, float &f)
{
    if (tx.mip == SF_MIP_NONE) {
        l0 = l1 = 0;
        f = 0.0f;
        return;
    }
    float lc = __builtin_fminf(__builtin_fmaxf(lam, 0.0f), (float)(tx.levels - 1));
    float fl = __builtin_floorf(lc);
    float fr = lc - fl;
    int a = (int)fl;
    if (tx.mip == SF_MIP_NEAREST) {
        a += fr >= 0.5f;
        a = min(a, tx.levels - 1);
        l0 = l1 = a;
        f = 0.0f;
        return;
    }
    l0 = a;
    l1 = min(a + 1, tx.levels - 1);
    f = fr;
}

// DCT basis c_k(x) = alpha(k) cos((2x+1) k pi / 16) for k = 1, 2 from the
// symmetries of the cosine: |c_1| takes four values mirrored about x = 3.5
// with the sign of x < 4; |c_2| is a for x in {0, 3, 4, 7} and b otherwise,
// negative for x in 2..5.
__device__ __forceinline__ float dct_c1(int x)
{
    const int m = min(x, 7 - x);
    const float v = m == 0 ? 0.49039262533187866f
                           : (m == 1 ? 0.41573479771614075f : (m == 2 ? 0.27778512239456177f : 0.09754516184329987f));
    return x < 4 ? v : -v;
}

__device__ __forceinline__ float dct_c2(int x)
{
    const float v = ((x + 1) >> 1) & 1 ? 0.19134171307086945f : 0.4619397521018982f;
    return ((x + 2) >> 2) & 1 ? -v : v;
}

constexpr float DCT_C0 = 0.3535533845424652f;

// One channel of a DCT block word at block position (x, y).
__device__ __forceinline__ float dct_channel(uint32_t wd, float R, float c1x, float c2x, float c1y, float c2y)
{
    const float q = R * (1.0f / 15.0f);
    float v = (float)(wd & 127u) * ((8.0f / 127.0f) * (DCT_C0 * DCT_C0));
    v = __builtin_fmaf((float)((int)((wd >> 7) & 31u) - 15) * q, c1x * DCT_C0, v);    // (1,0)
    v = __builtin_fmaf((float)((int)((wd >> 12) & 31u) - 15) * q, DCT_C0 * c1y, v);   // (0,1)
    v = __builtin_fmaf((float)((int)((wd >> 17) & 31u) - 15) * q, DCT_C0 * c2y, v);   // (0,2)
    v = __builtin_fmaf((float)((int)((wd >> 22) & 31u) - 15) * q, c1x * c1y, v);      // (1,1)
    v = __builtin_fmaf((float)((int)(wd >> 27) - 15) * q, c2x * DCT_C0, v);           // (2,0)
    return __builtin_fminf(__builtin_fmaxf(v, 0.0f), 1.0f);
}

// Texel (x, y) of a level wl texels wide that starts at lv.
template <int FMT>
__device__ __forceinline__ float4 texel_at(const Tex2DArgs &tx, const uint8_t *lv, int l, int wl, int x, int y)
{
    if constexpr (FMT == SF_DCT8) {
        const int bw = (wl + 7) >> 3;
        const uint4 b = reinterpret_cast<const uint4 *>(lv)[(int64_t)(y >> 3) * bw + (x >> 3)];
        const float4 R = reinterpret_cast<const float4 *>(tx.dct_range)[l];
        const int xi = x & 7, yi = y & 7;
        const float c1x = dct_c1(xi), c2x = dct_c2(xi), c1y = dct_c1(yi), c2y = dct_c2(yi);
        return make_float4(dct_channel(b.x, R.x, c1x, c2x, c1y, c2y), dct_channel(b.y, R.y, c1x, c2x, c1y, c2y),
                           dct_channel(b.z, R.z, c1x, c2x, c1y, c2y), dct_channel(b.w, R.w, c1x, c2x, c1y, c2y));
    } else if constexpr (FMT == SF_RGBA32F) {
        return reinterpret_cast<const float4 *>(lv)[(int64_t)y * wl + x];
    } else {
        const uint32_t px = reinterpret_cast<const uint32_t *>(lv)[(int64_t)y * wl + x];
        const float k = 1.0f / 255.0f;
        return make_float4((float)(px & 0xffu) * k, (float)((px >> 8) & 0xffu) * k, (float)((px >> 16) & 0xffu) * k,
                           (float)(px >> 24) * k);
    }
}

// Texel (x, y) of level l, the texture's levels read from `base` (its own
// base pointer, or a copy of its bytes at the same offsets).
__device__ __forceinline__ float4 texel(const Tex2DArgs &tx, const uint8_t *base, int l, int x, int y)
{
    const int wl = max(1, tx.w >> l);
    const uint8_t *lv = base + tx.off[l];
    if (tx.fmt == SF_DCT8)
        return texel_at<SF_DCT8>(tx, lv, l, wl, x, y);
    if (tx.fmt == SF_RGBA32F)
        return texel_at<SF_RGBA32F>(tx, lv, l, wl, x, y);
    return texel_at<SF_RGBA8_UNORM>(tx, lv, l, wl, x, y);
}

__device__ __forceinline__ float4 texel(const Tex2DArgs &tx, int l, int x, int y) { return texel(tx, tx.base, l, x, y); }

// Texel of a texture whose format the kernel knows, so that the loads of a
// level's taps are in flight together, or (ANY_FORMAT) asks at each texel.
constexpr int ANY_FORMAT = -1;

template <int FMT>
__device__ __forceinline__ float4 texel_of(const Tex2DArgs &tx, int l, int wl, int x, int y)
{
    if constexpr (FMT == ANY_FORMAT)
        return texel(tx, l, x, y);
    else
        return texel_at<FMT>(tx, tx.base + tx.off[l], l, wl, x, y);
}

template <int SHADE>
__device__ __forceinline__ float4 shade(const GgxConst &g, float4 c)
{
    if constexpr (SHADE == SF_SHADE_GGX) {
        float3 v = shade_ggx_dev(g, c);
        return make_float4(v.x, v.y, v.z, 0.0f);
    } else if constexpr (SHADE == SF_SHADE_GGX_NORMAL) {
        float3 v = shade_ggx_normal_dev(g, c);
        return make_float4(v.x, v.y, v.z, 0.0f);
    } else {
        return c;
    }
}

template <int SHADE>
__device__ __forceinline__ void store(float *out, int64_t q, float4 v)
{
    if constexpr (SHADE != SF_SHADE_NONE) {
        out[3 * q] = v.x;
        out[3 * q + 1] = v.y;
        out[3 * q + 2] = v.z;
    } else {
        reinterpret_cast<float4 *>(out)[q] = v;
    }
}

__device__ __forceinline__ bool query_ok(const Tex2DArgs &tx, float3 q)
{
    bool ok = __builtin_isfinite(q.x) & __builtin_isfinite(q.y);
    return ok & (tx.mip == SF_MIP_NONE || __builtin_isfinite(q.z));
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// Weighted sums of taps.  What is summed is linear in the weights, so that
// as little as possible is done per tap and the rest once per sum:
//   TAP_TEXEL   the texel's four channels (RGBA8: bytes, see sum_scaled);
//   TAP_GGX     its albedo channels (likewise) and its specular term, the only
//               part of the GGX + Lambert model that is not linear in the texel;
//   TAP_SHADED  the texel shaded as a whole (normal maps).
enum { TAP_TEXEL = 0, TAP_GGX = 1, TAP_SHADED = 2 };

template <int SHADE, int MODE>
constexpr int tap_kind()
{
    return MODE == BEFORE || SHADE == SF_SHADE_NONE ? TAP_TEXEL : (SHADE == SF_SHADE_GGX ? TAP_GGX : TAP_SHADED);
}

// The specular terms of the 256 roughness bytes, built by a workgroup of 256
// lanes: for RGBA8 textures a tap's specular term is a table read instead of
// two square roots and a reciprocal (the same binary32 numbers).
__device__ __forceinline__ void build_spec_table(const GgxConst &g, float *table)
{
    const float k = 1.0f / 255.0f;
    table[threadIdx.x] = ggx_spec(g, (float)threadIdx.x * k);
    __syncthreads();
}

// Texels of one row as one load from a 4-byte aligned address.
typedef uint32_t rgba8x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t rgba8x4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void tap_add(float w, float x, float y, float z, float a, float4 &s)
{
    s.x = __builtin_fmaf(w, x, s.x);
    s.y = __builtin_fmaf(w, y, s.y);
    s.z = __builtin_fmaf(w, z, s.z);
    s.w = __builtin_fmaf(w, a, s.w);
}

// sum_i w_i tap_i of the reconstruction filter F on level l at the wrapped
// coordinate (uu, vv), rows first.  RGBA8 taps that all lie inside the level
// are read with one load per row, issued before the first is used; others
// wrap and load one by one.  `spec`: the table of
// build_spec_table (RGBA8 with TAP_GGX).
template <int F, int SHADE, int KIND, int FMT>
__device__ __forceinline__ float4 level_sum(const Tex2DArgs &tx, const GgxConst &g, const float *spec, float uu,
                                            float vv, int l)
{
    constexpr int NT = Taps<F>::n;
    constexpr int F0 = Taps<F>::first;
    const int wl = max(1, tx.w >> l), hl = max(1, tx.h >> l);
    const uint8_t *lv = tx.base + tx.off[l];
    int ix, iy;
    float fx, fy, wx[4], wy[4];
    raster(uu, wl, ix, fx);
    raster(vv, hl, iy, fy);
    if constexpr (F == NEAREST) {
        ix += fx >= 0.5f;
        iy += fy >= 0.5f;
    }
    axis_weights<F>(fx, wx);
    axis_weights<F>(fy, wy);
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (FMT == SF_RGBA8_UNORM) {
        uint32_t px[NT][NT];
        const int x0 = ix + F0, y0 = iy + F0;
        if ((x0 >= 0) & (x0 + NT <= wl) & (y0 >= 0) & (y0 + NT <= hl)) {
            const uint32_t *row = reinterpret_cast<const uint32_t *>(lv) + ((int64_t)y0 * wl + x0);
#pragma unroll
            for (int b = 0; b < NT; ++b, row += wl) {
                if constexpr (NT == 4) {
                    const rgba8x4 v = *reinterpret_cast<const rgba8x4 *>(row);
                    px[b][0] = v.x, px[b][1] = v.y, px[b][2] = v.z, px[b][3] = v.w;
                } else if constexpr (NT == 2) {
                    const rgba8x2 v = *reinterpret_cast<const rgba8x2 *>(row);
                    px[b][0] = v.x, px[b][1] = v.y;
                } else {
                    px[b][0] = *row;
                }
            }
        } else {
            int xs[NT];
#pragma unroll
            for (int a = 0; a < NT; ++a)
                xs[a] = wrap_tap(tx.wrap, x0 + a, wl);
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const uint32_t *row = reinterpret_cast<const uint32_t *>(lv) +
                                      (int64_t)wrap_tap(tx.wrap, y0 + b, hl) * wl;
#pragma unroll
                for (int a = 0; a < NT; ++a)
                    px[b][a] = row[xs[a]];
            }
        }
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            float4 row = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                const uint32_t p = px[b][a];
                const float x = (float)(p & 0xffu), y = (float)((p >> 8) & 0xffu), z = (float)((p >> 16) & 0xffu);
                if constexpr (KIND == TAP_TEXEL) {
                    tap_add(wx[a], x, y, z, (float)(p >> 24), row);
                } else if constexpr (KIND == TAP_GGX) {
                    tap_add(wx[a], x, y, z, spec[p >> 24], row);
                } else {
                    const float k = 1.0f / 255.0f;
                    const float4 v = shade<SHADE>(g, make_float4(x * k, y * k, z * k, (float)(p >> 24) * k));
                    tap_add(wx[a], v.x, v.y, v.z, v.w, row);
                }
            }
            tap_add(wy[b], row.x, row.y, row.z, row.w, sum);
        }
    } else {
        // (sixteen shaded DCT blocks in flight take 147 registers: 2,073,600
        // queries 302 us against 253 asking for the format at each texel; filter
        // before shading 221 and 228)
        constexpr int KNOWN = FMT == SF_DCT8 && NT == 4 && KIND != TAP_TEXEL ? ANY_FORMAT : FMT;
        int xs[NT];
#pragma unroll
        for (int a = 0; a < NT; ++a)
            xs[a] = wrap_tap(tx.wrap, ix + F0 + a, wl);
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int y = wrap_tap(tx.wrap, iy + F0 + b, hl);
            float4 row = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                float4 t = texel_of<KNOWN>(tx, l, wl, xs[a], y);
                if constexpr (KIND == TAP_GGX)
                    t.w = ggx_spec(g, t.w);
                else if constexpr (KIND == TAP_SHADED)
                    t = shade<SHADE>(g, t);
                tap_add(wx[a], t.x, t.y, t.z, t.w, row);
            }
            tap_add(wy[b], row.x, row.y, row.z, row.w, sum);
        }
    }
    return sum;
}

// x / 255 within half an ulp (and a little): the product with the reciprocal,
// whose own rounding would bias every value by 2^-24, and the remainder's.
__device__ __forceinline__ float over255(float x)
{
    const float k = 1.0f / 255.0f, q = x * k;
    return __builtin_fmaf(__builtin_fmaf(-255.0f, q, x), k, q);
}

// A sum of taps as texel values (or radiance, once finished by sum_value):
// RGBA8 sums hold bytes.
template <int KIND, int FMT>
__device__ __forceinline__ float4 sum_scaled(float4 s)
{
    if constexpr (FMT != SF_RGBA8_UNORM || KIND == TAP_SHADED)
        return s;
    return make_float4(over255(s.x), over255(s.y), over255(s.z), KIND == TAP_TEXEL ? over255(s.w) : s.w);
}

// The lookup's value from its sum over all taps and levels.
template <int SHADE, int MODE, int FMT>
__device__ __forceinline__ float4 sum_value(const GgxConst &g, float4 sum)
{
    constexpr int KIND = tap_kind<SHADE, MODE>();
    const float4 s = sum_scaled<KIND, FMT>(sum);
    if constexpr (KIND == TAP_GGX) {
        const float3 v = ggx_radiance(g, s.x, s.y, s.z, s.w);
        return make_float4(v.x, v.y, v.z, 0.0f);
    } else if constexpr (KIND == TAP_TEXEL) {
        return shade<SHADE>(g, s);
    } else {
        return s;
    }
}

// The reconstruction filter alone on level l at the wrapped coordinate
// (uu, vv): sum_i w_i t_i with binary32 weights, as the deterministic kernels
// (the split-filtering estimator shades this once per sample).
template <int F, int FMT>
__device__ __forceinline__ float4 recon_level(const Tex2DArgs &tx, const GgxConst &g, float uu, float vv, int l)
{
    return sum_scaled<TAP_TEXEL, FMT>(level_sum<F, SF_SHADE_NONE, TAP_TEXEL, FMT>(tx, g, nullptr, uu, vv, l));
}

}  // namespace sfk
