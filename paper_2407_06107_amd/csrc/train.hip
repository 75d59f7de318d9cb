// Neural training step on the matrix cores (the learned stand-in's
// autodecoder: lattice latents z_c and the MLP D(z) = W3^T relu(W2^T
// relu(W1^T z + b1) + b2) + b3, loss (1/B) sum_s ||D(z_s) - t_s||^2).
//
// BF16 operands, FP32 accumulation, FP32 master copies of latents and
// parameters (and their Adam moments).  One wavefront walks a chunk of the
// batch in pairs of tiles of 16 samples:
//  - forward and backward products are 16-row tiles of hidden units times
//    16 samples as columns (v_mfma_f32_16x16x16_bf16 for the 8/16-input
//    and the <= 4-output layers, v_mfma_f32_16x16x32_bf16 for the 64 x 64
//    layers), so one product's accumulators are, lane for lane, the next
//    product's B operand (the weights' K order is permuted to match);
//  - weight gradients sum over samples, so the pair's activations and
//    pre-activation gradients go through LDS in [sample][feature] order and
//    come back, by the transposing LDS read, as A / B operands whose K
//    dimension is the pair's 32 samples; the wavefront's dW accumulators stay
//    in registers over its whole chunk;
//  - bias gradients and the loss are per-lane sums reduced once at the end;
//  - each sample's latent gradient (16 x 16 tile: channels x samples) gets
//    its Adam step at once (batch entries own distinct latents).
// Four wavefronts share a workgroup's LDS copy of the weights in fragment
// order and add their parameter gradients there before one row per workgroup
// goes to memory; the rows are then summed in a fixed order and Adam moves the
// parameters (the same second stage as the FP32 path).
//
// The products of one tile are a chain of nine, each waiting for the last, and
// a wavefront with its gradient accumulators holds a SIMD's registers alone
// (two per SIMD spill, and a spilled register's reload waits for the latents on
// their way: 61 us below).  So a wavefront takes two tiles side by side: one's
// products run while the other's are waited for, and the weight gradients take
// half the instructions.  What is left is memory: 64-byte rows at random of
// three tables read and written, which move whole 128-byte lines.
// Kernel, 262,144 samples of 16 channels: 59.6 us with one tile at a time,
// weights gathered from memory by each wavefront, 16-bit LDS reads and a row of
// gradients per wavefront; 47 us now.  With the gradient sum, by batch: 262,144
// 68.4 -> 51.2 us, 65,536 37.5 -> 23.3, 5,000 23.0 -> 15.0; 65,536 samples of
// 8 channels and 4 outputs 39.3 -> 23.3.  Loading two pairs ahead instead of
// one gave 49.6, 24.3 and 16.2 (and 24.7, with spills).
#include "sf_device.hpp"
#include "sf_internal.hpp"

#pragma clang fp contract(off)

namespace sfk {

namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr int H = 64;

// B-operand K position 8g + j of K step ks of a 16x16x32 product whose B
// operand is the previous product's accumulators (tiles 2ks, 2ks+1, rows
// 4g..4g+3): hidden unit 16 (2 ks + j/4) + 4 g + j%4.
__device__ __forceinline__ int kp(int ks, int g, int j) { return 16 * (2 * ks + (j >> 2)) + 4 * g + (j & 3); }

__device__ __forceinline__ uint32_t pk(float a, float b)
{
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint32_t relu2(uint32_t w)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, w), (s16x2)0));
}

__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v)
{
    return __builtin_bit_cast(bf16x4, make_uint2(pk(v[0], v[1]), pk(v[2], v[3])));
}

// two accumulator tiles -> one 8-wide B operand; RELU rectifies the rounded
// values (the same numbers as rounding the rectified ones)
template <bool RELU>
__device__ __forceinline__ uint4 pack8(f32x4 lo, f32x4 hi)
{
    uint4 w = make_uint4(pk(lo[0], lo[1]), pk(lo[2], lo[3]), pk(hi[0], hi[1]), pk(hi[2], hi[3]));
    if constexpr (RELU) {
        w.x = relu2(w.x);
        w.y = relu2(w.y);
        w.z = relu2(w.z);
        w.w = relu2(w.w);
    }
    return w;
}

__device__ __forceinline__ bf16x8 as8(uint4 w) { return __builtin_bit_cast(bf16x8, w); }

__device__ __forceinline__ __bf16 bw(const float *P, int i) { return (__bf16)P[i]; }

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// LDS rows of 16-bit values, [sample][feature]: rows 8-byte aligned, their
// strides spread over the banks.
constexpr int RS = H + 8, RS16 = 16 + 4;

// Four samples of a K = samples product's A / B fragment: feature column
// f0 + n, samples 4g..4g+3.  The transposing read hands lane n of a group of
// 16 column n of the four rows that the group's lanes address in quarters.
template <int STRIDE>
__device__ __forceinline__ bf16x4 col4(const uint16_t *s, int g, int n, int f0)
{
    const uint16_t *p = s + (4 * g + (n >> 2)) * STRIDE + f0 + 4 * (n & 3);
    return __builtin_bit_cast(
        bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p));
}

// v plus the lane's neighbour under a DPP control.
template <int CTRL>
__device__ __forceinline__ float add_dpp(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// Sum over the 16 lanes of a row (in every lane): rotations within the row.
__device__ __forceinline__ float sum16(float v)
{
    v = add_dpp<0x121>(v);   // row_ror:1
    v = add_dpp<0x122>(v);
    v = add_dpp<0x124>(v);
    v = add_dpp<0x128>(v);
    return v;
}

}  // namespace

// LDS instructions of one wavefront run in order; this keeps the compiler
// from moving reads of what other lanes wrote across the writes.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A wavefront's tile in LDS, [sample][feature].
struct TileLds {
    uint16_t H1[16 * RS], A2[16 * RS], A1[16 * RS], H2[16 * RS], Z[16 * RS16], Y[16 * RS16];
};

// Packed parameters (and the loss behind them) in LDS: rows of 64 take 65
// words, so that neither the fragments' column reads nor the gradients' row
// writes meet in a bank.
template <int C, int O>
struct Pad {
    static constexpr int w1 = 0, b1 = C * (H + 1), w2 = b1 + H, b2 = w2 + H * (H + 1), w3 = b2 + H, b3 = w3 + H * O,
                         loss = b3 + O, n = loss + 1;
    // place of packed parameter i (or of the loss)
    static __device__ __forceinline__ int at(int i)
    {
        constexpr int p1 = C * H, p2 = p1 + H, p3 = p2 + H * H;
        return i + (i < p1 ? i / H : (i < p2 ? C : (i < p3 ? C + (i - p2) / H : C + H)));
    }
};

template <int C, int O>
__global__ __launch_bounds__(64 * TRAIN_WAVES) __attribute__((amdgpu_waves_per_eu(1))) void
k_train_mfma(TrainCall t, int64_t chunk, float *partials)
{
    static_assert(C == 8 || C == 16, "8 or 16 latent channels");
    static_assert(O >= 1 && O <= 4, "at most 4 outputs");
    using L = Pad<C, O>;
    constexpr int NP = C * H + H + H * H + H + H * O + O + 1;   // parameters and the loss
    // The weights as fragments (BF16 of the FP32 master parameters): W2
    // forward and backward, W1 forward and W3 backward, W3 forward and W1
    // backward, and the hidden layers' biases; each wavefront's tile, before
    // the tiles the parameters, and after them a row of gradients per wavefront.
    struct Work {
        uint4 W2[2][8][64], W13[4][64];
        uint2 small[2][4][64];
        f32x4 bias[2][4][4];
        union {
            TileLds tile[TRAIN_WAVES][2];
            float par[Pad<C, O>::n];
        };
    };
    __shared__ __attribute__((aligned(16))) union {
        Work w;
        float sum[TRAIN_WAVES][Pad<C, O>::n];
    } sh;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63, n = l & 15, g = l >> 4;

    // The parameters come in whole lines, then each lane picks its fragments
    // from LDS: picked from memory by each wavefront they took 14 us.
    constexpr int NR = (NP + 64 * TRAIN_WAVES - 1) / (64 * TRAIN_WAVES);   // rounds of the workgroup over them
    {
        float w[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k)
            w[k] = t.params[min((int)threadIdx.x + 64 * TRAIN_WAVES * k, NP - 2)];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = threadIdx.x + 64 * TRAIN_WAVES * k;
            if (i < NP)
                sh.w.par[L::at(i)] = w[k];
        }
    }
    __syncthreads();
    const float *W = sh.w.par;
#pragma unroll
    for (int f0 = 0; f0 < 8; f0 += TRAIN_WAVES) {
        const int f = f0 + wave, m = f >> 1, ks = f & 1;
        bf16x8 a, b;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            a[j] = bw(W, L::w2 + kp(ks, g, j) * (H + 1) + 16 * m + n);     // W2[k][16m+n]
            b[j] = bw(W, L::w2 + (16 * m + n) * (H + 1) + kp(ks, g, j));   // W2[16m+n][k]
        }
        sh.w.W2[0][f][l] = __builtin_bit_cast(uint4, a);
        sh.w.W2[1][f][l] = __builtin_bit_cast(uint4, b);
    }
    static_assert(TRAIN_WAVES == 4, "a wavefront per fragment below");
    {
        const int f = wave;
        bf16x4 a, b;
        f32x4 c1, c2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 4 * g + j;
            const __bf16 w1 = bw(W, L::w1 + min(r, C - 1) * (H + 1) + 16 * f + n);
            const __bf16 w3 = bw(W, L::w3 + (16 * f + n) * O + min(r, O - 1));
            a[j] = r < C ? w1 : (__bf16)0.0f;   // W1[r][16f+n]
            b[j] = r < O ? w3 : (__bf16)0.0f;   // W3[16f+n][r]
            c1[j] = W[L::b1 + 16 * f + r];
            c2[j] = W[L::b2 + 16 * f + r];
        }
        sh.w.small[0][f][l] = __builtin_bit_cast(uint2, a);
        sh.w.small[1][f][l] = __builtin_bit_cast(uint2, b);
        if (n == 0) {
            sh.w.bias[0][f][g] = c1;
            sh.w.bias[1][f][g] = c2;
        }
    }
    {
        const int f = wave, ks = f & 1;
        bf16x8 a;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = kp(ks, g, j);
            const __bf16 w = bw(W, f < 2 ? L::w3 + k * O + min(n, O - 1) : L::w1 + min(n, C - 1) * (H + 1) + k);
            a[j] = n < (f < 2 ? O : C) ? w : (__bf16)0.0f;   // W3[k][n], then W1[n][k]
        }
        sh.w.W13[f][l] = __builtin_bit_cast(uint4, a);
    }
    f32x4 b3i;   // (rows from O on are not used)
#pragma unroll
    for (int j = 0; j < 4; ++j)
        b3i[j] = W[L::b3 + min(4 * g + j, O - 1)];
    __syncthreads();
    const auto a1f = [&](int m) { return __builtin_bit_cast(bf16x4, sh.w.small[0][m][l]); };
    const auto ab3 = [&](int m) { return __builtin_bit_cast(bf16x4, sh.w.small[1][m][l]); };
    const auto a3f = [&](int ks) { return as8(sh.w.W13[ks][l]); };
    const auto ab1 = [&](int ks) { return as8(sh.w.W13[2 + ks][l]); };
    const auto w2 = [&](int dir, int m, int ks) { return as8(sh.w.W2[dir][2 * m + ks][l]); };

    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 gw2[4][4], gw1[4], gw3[4];
    float gb1[4][4], gb2[4][4], gb3[4], loss = 0.0f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gw1[a] = zero;
        gw3[a] = zero;
        gb3[a] = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            gw2[a][b] = zero;
            gb1[a][b] = gb2[a][b] = 0.0f;
        }
    }

    const float inv_b = 2.0f / (float)t.batch;
    const int64_t s0 = min(((int64_t)blockIdx.x * TRAIN_WAVES + wave) * chunk, t.batch);
    const int64_t s1 = min(s0 + chunk, t.batch);
    // The pairs of tiles are software-pipelined: the batch indices of pair k+2
    // and the latents, targets and latent Adam moments of pair k+1 are loaded
    // while pair k computes (batch entries own distinct latents, so the
    // Adam step of pair k never writes what pair k+1 has read).
    // Batch index of this lane's column of the tile at sb (an address inside
    // the chunk also past its end).
    auto index_at = [&](int64_t sb) -> int32_t { return t.idx[min(sb + n, s1 - 1)]; };
    struct TileIn {
        bool use;    // the column holds a sample of the chunk inside the lattice
        int32_t p;   // its lattice point (0 for unused columns)
        f32x4 z, mq, vq;
        float tg[O];
    };
    // unused columns read element 0 and contribute nothing
    auto load_tile = [&](int64_t sb, int32_t raw, TileIn &T) {
        T.use = sb + n < s1 && (uint64_t)(int64_t)raw < (uint64_t)t.n_lattice;
        T.p = T.use ? raw : 0;
        T.z = zero;
        T.mq = zero;
        T.vq = zero;
        if (4 * g < C) {
            const int64_t q = (int64_t)T.p * C + 4 * g;
            T.z = *reinterpret_cast<const f32x4 *>(t.latents + q);
            T.mq = *reinterpret_cast<const f32x4 *>(t.m_lat + q);
            T.vq = *reinterpret_cast<const f32x4 *>(t.v_lat + q);
        }
#pragma unroll
        for (int o = 0; o < O; ++o)
            T.tg[o] = g == 0 ? t.targets[(int64_t)T.p * O + o] : 0.0f;
    };
    TileIn cur[2], nxt[2];
    int32_t raw_next[2] = {0, 0};
    if (s0 < s1) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            load_tile(s0 + 16 * u, index_at(s0 + 16 * u), cur[u]);
            raw_next[u] = index_at(s0 + 32 + 16 * u);
        }
    }
    for (int64_t sb = s0; sb < s1; sb += 32) {
        if (sb + 32 < s1) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
                load_tile(sb + 32 + 16 * u, raw_next[u], nxt[u]);   // pair k+1
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            raw_next[u] = index_at(sb + 64 + 16 * u);   // pair k+2
        // finite inputs for unused columns, so that their zero gradients stay zero
        bf16x4 zb[2], dyb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
            zb[u] = to_bf16x4(cur[u].use ? cur[u].z : zero);

        // forward: A1, H1, A2, H2, Y (columns = samples)
        f32x4 a1[2][4], a2[2][4], y[2];
        uint4 h1w[2][2], h2w[2][2], d2w[2][2], d1w[2][2];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                a1[u][m] = mfma16(a1f(m), zb[u], sh.w.bias[0][m][g]);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            h1w[u][0] = pack8<true>(a1[u][0], a1[u][1]);
            h1w[u][1] = pack8<true>(a1[u][2], a1[u][3]);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                a2[u][m] = mfma32(w2(0, m, 1), as8(h1w[u][1]),
                                  mfma32(w2(0, m, 0), as8(h1w[u][0]), sh.w.bias[1][m][g]));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            h2w[u][0] = pack8<true>(a2[u][0], a2[u][1]);
            h2w[u][1] = pack8<true>(a2[u][2], a2[u][3]);
            y[u] = mfma32(a3f(1), as8(h2w[u][1]), mfma32(a3f(0), as8(h2w[u][0]), b3i));
        }

        // dL/dY on rows 4g + j < O (lanes g = 0)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f32x4 dy = zero;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool row = g == 0 && j < O && cur[u].use;
                const float e = y[u][j] - (j < O ? cur[u].tg[j < O ? j : 0] : 0.0f);
                loss = row ? __builtin_fmaf(e, e, loss) : loss;
                dy[j] = row ? e * inv_b : 0.0f;
                gb3[j] += dy[j];
            }
            dyb[u] = to_bf16x4(dy);
        }

        // backward: dA2 = W3 dY (rectified), dA1 = W2 dA2 (rectified), dZ = W1 dA1
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f32x4 da[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const f32x4 d = mfma16(ab3(m), dyb[u], zero);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    da[m][j] = a2[u][m][j] > 0.0f ? d[j] : 0.0f;
                    gb2[m][j] += da[m][j];
                }
            }
            d2w[u][0] = pack8<false>(da[0], da[1]);
            d2w[u][1] = pack8<false>(da[2], da[3]);
        }
        f32x4 d1[2][4];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                d1[u][m] = mfma32(w2(1, m, 1), as8(d2w[u][1]), mfma32(w2(1, m, 0), as8(d2w[u][0]), zero));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d1[u][m][j] = a1[u][m][j] > 0.0f ? d1[u][m][j] : 0.0f;
                    gb1[m][j] += d1[u][m][j];
                }
            d1w[u][0] = pack8<false>(d1[u][0], d1[u][1]);
            d1w[u][1] = pack8<false>(d1[u][2], d1[u][3]);
        }

        // stage the tiles in LDS as [sample][feature]
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            TileLds &T = sh.w.tile[wave][u];
            uint2 *h1 = reinterpret_cast<uint2 *>(T.H1 + n * RS + 4 * g);
            uint2 *h2 = reinterpret_cast<uint2 *>(T.H2 + n * RS + 4 * g);
            uint2 *e2 = reinterpret_cast<uint2 *>(T.A2 + n * RS + 4 * g);
            uint2 *e1 = reinterpret_cast<uint2 *>(T.A1 + n * RS + 4 * g);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                h1[(32 * ks) / 4] = make_uint2(h1w[u][ks].x, h1w[u][ks].y);        // rows 32ks..
                h1[(32 * ks + 16) / 4] = make_uint2(h1w[u][ks].z, h1w[u][ks].w);   // rows 32ks+16..
                h2[(32 * ks) / 4] = make_uint2(h2w[u][ks].x, h2w[u][ks].y);
                h2[(32 * ks + 16) / 4] = make_uint2(h2w[u][ks].z, h2w[u][ks].w);
                e2[(32 * ks) / 4] = make_uint2(d2w[u][ks].x, d2w[u][ks].y);
                e2[(32 * ks + 16) / 4] = make_uint2(d2w[u][ks].z, d2w[u][ks].w);
                e1[(32 * ks) / 4] = make_uint2(d1w[u][ks].x, d1w[u][ks].y);
                e1[(32 * ks + 16) / 4] = make_uint2(d1w[u][ks].z, d1w[u][ks].w);
            }
            *reinterpret_cast<uint2 *>(T.Z + n * RS16 + 4 * g) = __builtin_bit_cast(uint2, zb[u]);
            *reinterpret_cast<uint2 *>(T.Y + n * RS16 + 4 * g) = __builtin_bit_cast(uint2, dyb[u]);
        }

        // the latents' gradients (channels 4g..4g+3 of sample n) and their Adam step
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const f32x4 dz = mfma32(ab1(1), as8(d1w[u][1]), mfma32(ab1(0), as8(d1w[u][0]), zero));
            if (cur[u].use && 4 * g < C) {
                if (t.grad_latents)
                    *reinterpret_cast<f32x4 *>(t.grad_latents + (sb + 16 * u + n) * C + 4 * g) = dz;
                const int64_t q = (int64_t)cur[u].p * C + 4 * g;
                const f32x4 z = cur[u].z, mq = cur[u].mq, vq = cur[u].vq;
                f32x4 mo, vo, zo;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    mo[j] = 0.9f * mq[j] + 0.1f * dz[j];
                    vo[j] = 0.999f * vq[j] + 0.001f * dz[j] * dz[j];
                    // bias corrections by the reciprocals, the step by the hardware
                    // square root and reciprocal (1 ulp each)
                    const float den = __builtin_amdgcn_sqrtf(vo[j] * t.inv_bc2) + 1e-8f;
                    zo[j] = z[j] - t.lr_latent * (mo[j] * t.inv_bc1) * __builtin_amdgcn_rcpf(den);
                }
                *reinterpret_cast<f32x4 *>(t.m_lat + q) = mo;
                *reinterpret_cast<f32x4 *>(t.v_lat + q) = vo;
                *reinterpret_cast<f32x4 *>(t.latents + q) = zo;
            }
        }
        wave_lds_fence();
        // weight gradients, K = the pair's 32 samples
        const auto both = [&](const uint16_t *s, const uint16_t *s2, auto stride, int f0) {
            constexpr int S = decltype(stride)::value;
            const bf16x4 a = col4<S>(s, g, n, f0), b = col4<S>(s2, g, n, f0);
            const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
            return as8(make_uint4(x.x, x.y, y.x, y.y));
        };
        const TileLds &A = sh.w.tile[wave][0], &B = sh.w.tile[wave][1];
        const std::integral_constant<int, RS> wide;
        const std::integral_constant<int, RS16> narrow;
        bf16x8 ca[4], cb[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            ca[m] = both(A.H1, B.H1, wide, 16 * m);   // H1[16m+n][s]
            cb[m] = both(A.A2, B.A2, wide, 16 * m);   // dA2[16m+n][s]
        }
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int mo = 0; mo < 4; ++mo)
                gw2[mi][mo] = mfma32(ca[mi], cb[mo], gw2[mi][mo]);
        const bf16x8 zc = both(A.Z, B.Z, narrow, 0);      // Z[n][s]
#pragma unroll
        for (int m = 0; m < 4; ++m)
            gw1[m] = mfma32(zc, both(A.A1, B.A1, wide, 16 * m), gw1[m]);
        const bf16x8 yc = both(A.Y, B.Y, narrow, 0);      // dY[n][s]
#pragma unroll
        for (int m = 0; m < 4; ++m)
            gw3[m] = mfma32(both(A.H2, B.H2, wide, 16 * m), yc, gw3[m]);
        wave_lds_fence();
#pragma unroll
        for (int u = 0; u < 2; ++u)
            cur[u] = nxt[u];
    }

    // the wavefronts' gradients in the packed layout, then the loss, added in
    // wavefront order in LDS and written as one row
    float s1v[4][4], s2v[4][4], s3v[4], lsum = loss;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // bias sums over the lanes of one row group (same g, all columns n)
            s1v[m][j] = sum16(gb1[m][j]);
            s2v[m][j] = sum16(gb2[m][j]);
        }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        s3v[j] = sum16(gb3[j]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        lsum += __shfl_xor(lsum, m);
    __syncthreads();
    {
        float *sum = sh.sum[wave];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int mo = 0; mo < 4; ++mo)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    sum[L::w2 + (16 * mi + 4 * g + j) * (H + 1) + 16 * mo + n] = gw2[mi][mo][j];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (4 * g + j < C)
                    sum[L::w1 + (4 * g + j) * (H + 1) + 16 * m + n] = gw1[m][j];
                if (n < O)
                    sum[L::w3 + (16 * m + 4 * g + j) * O + n] = gw3[m][j];
                if (n == 0) {
                    sum[L::b1 + 16 * m + 4 * g + j] = s1v[m][j];
                    sum[L::b2 + 16 * m + 4 * g + j] = s2v[m][j];
                }
            }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (l == 0 && j < O)
                sum[L::b3 + j] = s3v[j];
        if (l == 0)
            sum[L::loss] = lsum;
    }
    __syncthreads();
    float *out = partials + (int64_t)blockIdx.x * NP;
#pragma unroll 7
    for (int k = 0; k < NR; ++k) {
        const int j = threadIdx.x + 64 * TRAIN_WAVES * k, i = L::at(min(j, NP - 1));
        float v = sh.sum[0][i];
#pragma unroll
        for (int w = 1; w < TRAIN_WAVES; ++w)
            v += sh.sum[w][i];
        if (j < NP)
            out[j] = v;
    }
}

hipError_t launch_train_mfma(const TrainCall &t, float *partials, int nrows, int64_t chunk, hipStream_t s)
{
    if (t.C == 8 && t.O == 4)
        k_train_mfma<8, 4><<<dim3(nrows), dim3(64 * TRAIN_WAVES), 0, s>>>(t, chunk, partials);
    else
        k_train_mfma<16, 1><<<dim3(nrows), dim3(64 * TRAIN_WAVES), 0, s>>>(t, chunk, partials);
    return hipGetLastError();
}

}  // namespace sfk
