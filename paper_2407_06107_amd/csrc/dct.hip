// DCT texture compressor (Sec. 5 "Texture compression"): 8x8 blocks, the
// six lowest-frequency coefficients per channel in one 32-bit word.  The
// decoder is part of the texel fetch (tex2d.hpp), so every 2-D filter reads
// SF_DCT8 textures.
//
// Two passes over all levels at once, one thread per block: the first
// takes each channel's largest |AC| over a workgroup's blocks, and a small
// kernel the largest of a level; the second recomputes the coefficients and
// writes the codes.  Every coefficient is one fixed chain of binary32 fused
// multiply-adds, so the codes are reproducible bit for bit.
//
// Both passes are bound by vector instructions (about 1,700 per block, 960
// of them the transform's) and read the pyramid once, from HBM or the
// Infinity Cache.  A 4096^2 pyramid (89 MB) takes 27 + 5 + 22 us: it took
// 267 + 77 us with 64 four-byte loads per block at a stride of 32 bytes
// between lanes, an IEEE division per byte and the maxima taken by atomics.
#include "sf_device.hpp"
#include "sf_internal.hpp"
#include "tex2d.hpp"

#pragma clang fp contract(off)

namespace sfk {

__device__ __forceinline__ float dct_basis(int k, int x) { return k == 0 ? DCT_C0 : (k == 1 ? dct_c1(x) : dct_c2(x)); }

// Level of a global block index at or past the first block of level l.
__device__ __forceinline__ int level_from(const DctEncodeCall &c, int l, int64_t b)
{
    while (l + 1 < c.levels && b >= c.first_block[l + 1])
        ++l;
    return l;
}

// Byte k of a word over 255, correctly rounded (the same number as the IEEE
// division for all 256 bytes): 1/255 as 0x1.01p-8 plus the rest; the product
// with the first part is exact, so the fma rounds once.
template <int K>
__device__ __forceinline__ float unorm8(uint32_t px)
{
    const float x = (float)((px >> (8 * K)) & 0xffu);
    return __builtin_fmaf(x, 0x1.010102p-24f, x * 0x1.01p-8f);
}

// Four texels as one 16-byte load from a 4-byte aligned address.
typedef uint32_t texels4 __attribute__((ext_vector_type(4), aligned(4)));

// The basis over y, read with scalar loads by the loop over rows.
struct BasisRow {
    float c[4];
};
static __constant__ BasisRow kBasis[8] = {
#define SF_BASIS_ROW(y, c1, c2) {{0.3535533845424652f, c1, c2, 0.0f}}
    SF_BASIS_ROW(0, 0.49039262533187866f, 0.4619397521018982f),
    SF_BASIS_ROW(1, 0.41573479771614075f, 0.19134171307086945f),
    SF_BASIS_ROW(2, 0.27778512239456177f, -0.19134171307086945f),
    SF_BASIS_ROW(3, 0.09754516184329987f, -0.4619397521018982f),
    SF_BASIS_ROW(4, -0.09754516184329987f, -0.4619397521018982f),
    SF_BASIS_ROW(5, -0.27778512239456177f, -0.19134171307086945f),
    SF_BASIS_ROW(6, -0.41573479771614075f, 0.19134171307086945f),
    SF_BASIS_ROW(7, -0.49039262533187866f, 0.4619397521018982f),
#undef SF_BASIS_ROW
};

// Eight texels of a row from column x0: two 16-byte loads where they lie
// inside the level (a wavefront then reads whole lines), else texel by texel,
// the level's last one replicated.
__device__ __forceinline__ void load_row(const uint32_t *row, int x0, int wl, bool inside, uint32_t px[8])
{
    if (inside) {
        const texels4 a = *reinterpret_cast<const texels4 *>(row + x0);
        const texels4 b = *reinterpret_cast<const texels4 *>(row + x0 + 4);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            px[x] = a[x];
            px[4 + x] = b[x];
        }
    } else {
#pragma unroll
        for (int x = 0; x < 8; ++x)
            px[x] = row[min(x0 + x, wl - 1)];
    }
}

// Six coefficients, zigzag order (0,0) (1,0) (0,1) (0,2) (1,1) (2,0), of the
// four channels of block (bx, by) of an RGBA8 level.  The coefficients'
// chains run over y, so a row enters them as soon as its own three sums are
// known, and one row is in flight while another is used: eight rows at once
// take 180 registers and leave two wavefronts per SIMD.
__device__ __forceinline__ void block_coeffs(const uint8_t *lv, int wl, int hl, int bx, int by, float C[4][6])
{
    constexpr int U[6] = {0, 1, 0, 0, 1, 2}, V[6] = {0, 0, 1, 2, 1, 0};
    const bool inside = bx * 8 + 8 <= wl;
    const uint32_t *base = reinterpret_cast<const uint32_t *>(lv);
    uint32_t cur[8], nxt[8];
    load_row(base + (int64_t)(by * 8) * wl, bx * 8, wl, inside, cur);
#pragma unroll
    for (int ch = 0; ch < 4; ++ch)
#pragma unroll
        for (int k = 0; k < 6; ++k)
            C[ch][k] = 0.0f;
#pragma unroll 1
    for (int y = 0; y < 8; ++y) {
        // (the last pass loads its own row again)
        load_row(base + (int64_t)min(by * 8 + min(y + 1, 7), hl - 1) * wl, bx * 8, wl, inside, nxt);
        const BasisRow cy = kBasis[y];
        float R[4][3];
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int u = 0; u < 3; ++u)
                R[ch][u] = 0.0f;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const uint32_t w = cur[x];
            const float v[4] = {unorm8<0>(w), unorm8<1>(w), unorm8<2>(w), unorm8<3>(w)};
#pragma unroll
            for (int ch = 0; ch < 4; ++ch)
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    R[ch][u] = __builtin_fmaf(dct_basis(u, x), v[ch], R[ch][u]);
        }
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C[ch][k] = __builtin_fmaf(cy.c[V[k]], R[ch][U[k]], C[ch][k]);
#pragma unroll
        for (int x = 0; x < 8; ++x)
            cur[x] = nxt[x];
    }
}

// First pass: the largest |AC| per channel over each workgroup's blocks of a
// level, kept until the second pass in the 16 bytes of the first of those
// blocks (which no code has been written to yet).  An atomic maximum per
// wavefront and channel on dst_range instead queued 22,000 atomics of a
// 4096^2 pyramid on one line: 190 of the pass's 267 us.  The maxima of a
// launch's only workgroup (256 blocks) are the levels' already, and go to
// c.range without the pass between (64^2 and its levels, a call: 26.4 us with
// it, 22.6 without).
__global__ __launch_bounds__(256) void k_dct_range(DctEncodeCall c)
{
    __shared__ float part[4][4];
    const int64_t b0 = (int64_t)blockIdx.x * 256, total = c.first_block[c.levels];
    const int64_t b = b0 + threadIdx.x;
    const int lfirst = level_from(c, 0, b0);
    const int llast = level_from(c, lfirst, min(b0 + 255, total - 1));
    const bool active = b < total;
    const int l = active ? level_from(c, lfirst, b) : -1;
    float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (active) {
        const int wl = max(1, c.w >> l), hl = max(1, c.h >> l), bw = (wl + 7) >> 3;
        const uint32_t j = (uint32_t)(b - c.first_block[l]);   // a level holds at most 2^26 blocks
        float C[4][6];
        block_coeffs(c.src + c.src_off[l], wl, hl, (int)(j % (uint32_t)bw), (int)(j / (uint32_t)bw), C);
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int k = 1; k < 6; ++k)
                m[ch] = __builtin_fmaxf(m[ch], __builtin_fabsf(C[ch][k]));
    }
    // the levels this workgroup touches: one, but for the last few of a pyramid
    for (int lv = lfirst; lv <= llast; ++lv) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            float v = l == lv ? m[ch] : 0.0f;
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1)
                v = __builtin_fmaxf(v, __shfl_xor(v, s));
            if ((threadIdx.x & 63) == 0)
                part[threadIdx.x >> 6][ch] = v;
        }
        __syncthreads();
        if (threadIdx.x < 4) {
            const int ch = threadIdx.x;
            const int64_t j = max(b0, c.first_block[lv]) - c.first_block[lv];
            float *to = gridDim.x == 1 ? c.range + 4 * lv
                                       : reinterpret_cast<float *>(c.dst + c.dst_off[lv]) + 4 * j;
            to[ch] = __builtin_fmaxf(__builtin_fmaxf(part[0][ch], part[1][ch]),
                                     __builtin_fmaxf(part[2][ch], part[3][ch]));
        }
        __syncthreads();
    }
}

// The maximum of one level's workgroup maxima: its first block, then every
// block of the level whose global index is a multiple of 256.
__global__ __launch_bounds__(1024) void k_dct_range_level(DctEncodeCall c)
{
    __shared__ float part[16][4];
    const int l = blockIdx.x;
    const int64_t f0 = c.first_block[l], f1 = c.first_block[l + 1];
    const float4 *slot = reinterpret_cast<const float4 *>(c.dst + c.dst_off[l]);
    float4 m = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int64_t i = threadIdx.x; f0 + 256 * i < f1 + 255; i += 1024) {
        // i = 0: the level's first block; i >= 1: the i-th multiple of 256 after it
        const int64_t b = i == 0 ? f0 : (f0 / 256 + i) * 256;
        if (b < f1) {
            const float4 v = slot[b - f0];
            m = make_float4(__builtin_fmaxf(m.x, v.x), __builtin_fmaxf(m.y, v.y), __builtin_fmaxf(m.z, v.z),
                            __builtin_fmaxf(m.w, v.w));
        }
    }
    float v[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
    for (int ch = 0; ch < 4; ++ch) {
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1)
            v[ch] = __builtin_fmaxf(v[ch], __shfl_xor(v[ch], s));
        if ((threadIdx.x & 63) == 0)
            part[threadIdx.x >> 6][ch] = v[ch];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        float r = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 16; ++w)
            r = __builtin_fmaxf(r, part[w][threadIdx.x]);
        c.range[4 * l + threadIdx.x] = r;
    }
}

__global__ __launch_bounds__(256) void k_dct_codes(DctEncodeCall c)
{
    const int64_t b0 = (int64_t)blockIdx.x * 256;
    const int64_t b = b0 + threadIdx.x;
    const int lfirst = level_from(c, 0, b0);
    if (b >= c.first_block[c.levels])
        return;
    const int l = level_from(c, lfirst, b);
    const int wl = max(1, c.w >> l), hl = max(1, c.h >> l), bw = (wl + 7) >> 3;
    const uint32_t j = (uint32_t)(b - c.first_block[l]);
    float C[4][6];
    block_coeffs(c.src + c.src_off[l], wl, hl, (int)(j % (uint32_t)bw), (int)(j / (uint32_t)bw), C);
    uint32_t word[4];
#pragma unroll
    for (int ch = 0; ch < 4; ++ch) {
        const float R = c.range[4 * l + ch];
        const float sc = R > 0.0f ? 15.0f / R : 0.0f;
        const int dc = min(max((int)__builtin_floorf(C[ch][0] * 15.875f + 0.5f), 0), 127);
        uint32_t wd = (uint32_t)dc;
#pragma unroll
        for (int k = 1; k < 6; ++k) {
            // R = 0 gives sc = 0 and so the middle code 15
            const int a = min(max((int)__builtin_floorf(C[ch][k] * sc + 0.5f), -15), 15) + 15;
            wd |= (uint32_t)a << (7 + 5 * (k - 1));
        }
        word[ch] = wd;
    }
    reinterpret_cast<uint4 *>(c.dst + c.dst_off[l])[j] = make_uint4(word[0], word[1], word[2], word[3]);
}

hipError_t launch_dct_encode(const DctEncodeCall &c, hipStream_t s)
{
    const int64_t nb = c.first_block[c.levels];
    const dim3 grid((uint32_t)((nb + 255) / 256)), block(256);
    k_dct_range<<<grid, block, 0, s>>>(c);
    if (grid.x > 1)
        k_dct_range_level<<<dim3((uint32_t)c.levels), dim3(1024), 0, s>>>(c);
    k_dct_codes<<<grid, block, 0, s>>>(c);
    return hipGetLastError();
}

}  // namespace sfk
