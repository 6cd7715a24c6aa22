// Backward pass of the surrogate: one kernel per layer, each reading the
// gradient dz of its layer's pre-activation and the pre-activation z of the
// layer below once, and one reduction of the weight-gradient partials.
//
// Only z is kept by the forward pass; a = bf16(GELU(z)) is formed again from z
// (the same bits) next to GELU'(z), which shares its exponential.  The weight
// gradients are products over positions, dW[tap][co][ci] = sum_y
// dz[y - (tap-2) d, co] a[y, ci]: both operands are rows of 64 channels in LDS,
// and ds_read_b64_tr_b16 hands a lane four consecutive positions of one channel
// (16 lanes with the addresses of four rows of 16 channels get one column each),
// so no transposed copy is staged.  A workgroup keeps its partial sums in
// registers over its run of tiles; k_reduce sums the workgroups' partials in a
// fixed order, so the gradient is deterministic.
//
// [256, 1024] on MI355X: the backward pass 457 -> 124 us (a kernel per data and
// per weight gradient before: layer-1 weights 109, layer-4 weights 78, transposing
// weight gradients 54 + 53, data gradients 36 + 36 + 30, six reductions 31); now
// k_bwd_out 29, k_bwd_hidden 41 and 50, k_reduce 10.
#include "srg_common.h"

namespace srg {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int TB = 128;  // positions per tile

// Eight consecutive rows (positions) of one channel: rows r .. r + 7 of the
// column that the lane's place in its 16 lanes selects.  p: row r + j / 4,
// column c0 + 4 (j % 4) for lane j of the 16, rows of RS elements.
__device__ __forceinline__ bf16x8 column8(const __bf16 *p) {
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * RS));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// A float32 operand as three bfloat16 terms (24 bits of significand): products
// with a bfloat16 factor, summed in float32, carry the float32 product.  finite()
// sets the later terms of an infinity (inf - inf: a NaN) to zero.
struct Split3 {
    bf16x8 t[3];
    __device__ __forceinline__ void set(const float (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const __bf16 h = to_bf(v[j]);
            const float r = v[j] - to_f(h);
            const __bf16 m = to_bf(r);
            t[0][j] = h;
            t[1][j] = m;
            t[2][j] = to_bf(r - to_f(m));
        }
    }
    __device__ __forceinline__ void finite(const float (&v)[8]) {
        float top = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) top = __builtin_fmaxf(top, __builtin_fabsf(v[j]));
        if (__builtin_amdgcn_ballot_w64(top == __builtin_inff()) == 0) return;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (__builtin_fabsf(v[j]) == __builtin_inff()) t[1][j] = t[2][j] = to_bf(0.0f);
    }
};

// GELU(z) and GELU'(z) = Phi(z) + z phi(z), phi(z) = exp(-z^2 / 2) / sqrt(2 pi), of one
// value, sharing the error function's exponential
__device__ __forceinline__ void gelu_both(float z, float &g, float &dg) {
    const ErfExp q = erf_exp(z * 0.70710678118654752f);
    g = 0.5f * z * (1.0f + q.erf);
    dg = __builtin_fmaf(z * 0.39894228040143268f, q.e, 0.5f * (1.0f + q.erf));
}

// ---------------------------------------------------------------------------
// Layer 4 (64 -> 2, dilation 27) and the GELU of layer 3:
//   dz3[x, ci] = bf16(GELU'(z3) sum_{tap, c} dy[c, x - (tap-2) 27] W4[tap][c][ci]),
//   dW4[tap][c][ci] = sum_y dy[c, y - (tap-2) 27] a3[y, ci],  db4[c] = sum dy,
// with dy = 0.25 dout (the residual's scale).  A thread takes rows' 8-channel
// pieces of one channel group (its 80 weights in registers); the weight
// gradient is 16 (tap, c: 10 used) x 64 channels over the tile's 128 positions,
// 32 per wavefront, v_mfma_f32_16x16x32_bf16 with dy in three bfloat16 terms.
// Partials part[g][642].
// ---------------------------------------------------------------------------
constexpr int H4 = 2 * 27;
constexpr int NW4P = KT * 2 * CH + 2;

__global__ void __launch_bounds__(256) k_bwd_out(const float *__restrict__ dout, const __bf16 *__restrict__ W4,
                                                 const __bf16 *__restrict__ z3, __bf16 *__restrict__ dz3,
                                                 float *__restrict__ part, int ntiles, int L) {
    __shared__ __attribute__((aligned(16))) __bf16 at[TB * RS];  // a3 of the tile
    __shared__ float dyl[2][TB + 2 * H4];
    __shared__ float red[4][16 * CH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, v = threadIdx.x & 7;
    const int g = lane >> 4, m = lane & 15;
    float w[2 * KT][8];  // this thread's channels 8 v ..
#pragma unroll
    for (int k = 0; k < 2 * KT; ++k) {
        const bf16x8 wv = *(const bf16x8 *)(W4 + k * CH + 8 * v);
#pragma unroll
        for (int j = 0; j < 8; ++j) w[k][j] = to_f(wv[j]);
    }
    floatx4 acc[4] = {};
    float bacc[2] = {0.0f, 0.0f};
    const int tps = L / TB;
    const int t0 = (int)((int64_t)blockIdx.x * ntiles / gridDim.x), t1 = (int)((int64_t)(blockIdx.x + 1) * ntiles / gridDim.x);
    // the tap and component of the lane's row of the weight gradient (rows from 10 on are zero)
    const int mt = m < 2 * KT ? m >> 1 : 0, mc = m & 1;
    bf16x8 zn[4];
    auto fetch = [&](int t) {
        const int64_t base = (int64_t)t * TB * CH;  // tiles follow each other in memory
#pragma unroll
        for (int k = 0; k < 4; ++k) zn[k] = *(const bf16x8 *)(z3 + base + (int64_t)(threadIdx.x + 256 * k) * 8);
    };
    if (t0 < t1) fetch(t0);
    for (int t = t0; t < t1; ++t) {
        const int b = t / tps, x0 = (t % tps) * TB;
        for (int i = threadIdx.x; i < 2 * (TB + 2 * H4); i += 256) {
            const int c = i >= TB + 2 * H4, k = i - c * (TB + 2 * H4), x = x0 - H4 + k;
            dyl[c][k] = (x >= 0 && x < L) ? FS * dout[(int64_t)b * 2 * L + (int64_t)c * L + x] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int p = (threadIdx.x + 256 * k) >> 3;
            float dyv[2 * KT];
#pragma unroll
            for (int q = 0; q < 2 * KT; ++q) dyv[q] = dyl[q & 1][H4 + p - ((q >> 1) - 2) * 27];
            bf16x8 av, dv;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float s = 0.0f;
#pragma unroll
                for (int q = 0; q < 2 * KT; ++q) s = __builtin_fmaf(dyv[q], w[q][j], s);
                float ga, dg;
                gelu_both(to_f(zn[k][j]), ga, dg);
                av[j] = to_bf(ga);
                dv[j] = to_bf(s * dg);
            }
            *(bf16x8 *)(at + p * RS + 8 * v) = av;
            *(bf16x8 *)(dz3 + (int64_t)t * TB * CH + (int64_t)(threadIdx.x + 256 * k) * 8) = dv;
        }
        if (threadIdx.x < TB) {
            bacc[0] += dyl[0][H4 + threadIdx.x];
            bacc[1] += dyl[1][H4 + threadIdx.x];
        }
        if (t + 1 < t1) fetch(t + 1);
        __syncthreads();
        float f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = m < 2 * KT ? dyl[mc][H4 + 32 * wave + 8 * g + j - (mt - 2) * 27] : 0.0f;
        Split3 d;
        d.set(f);
        d.finite(f);  // dy of an overflowed loss
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const bf16x8 bv = column8(at + (32 * wave + 8 * g + (m >> 2)) * RS + 16 * cb + 4 * (m & 3));
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d.t[q], bv, acc[cb], 0, 0, 0);
        }
        __syncthreads();  // the tile and dy are rewritten next
    }
    // result: row 4 g + r, channel 16 cb + m
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][(4 * g + r) * CH + 16 * cb + m] = acc[cb][r];
    float *bs = reinterpret_cast<float *>(at);  // the bias sums of the threads
    bs[threadIdx.x] = bacc[0];
    bs[256 + threadIdx.x] = bacc[1];
    __syncthreads();
    float *pg = part + (int64_t)blockIdx.x * NW4P;
    for (int o = threadIdx.x; o < KT * 2 * CH; o += 256) pg[o] = ((red[0][o] + red[1][o]) + red[2][o]) + red[3][o];
    if (threadIdx.x < 2) {
        float s = 0.0f;
        for (int k = 0; k < TB; ++k) s += bs[256 * threadIdx.x + k];
        pg[KT * 2 * CH + threadIdx.x] = s;
    }
}

// ---------------------------------------------------------------------------
// A 64 -> 64 layer of dilation D and the GELU of the layer below:
//   dzp[y, ci] = bf16(GELU'(zp) sum_{tap, co} dz[y - (tap-2) D, co] W[tap][co][ci]),
//   dW[tap][co][ci] = sum_y dz[y - (tap-2) D, co] a[y, ci],  db[co] = sum dz.
// Eight wavefronts per workgroup, one workgroup per compute unit: wavefronts 0-3
// form the data gradient (two 32 x 32 blocks of channels x positions each, the
// transposed weights of their 32 channels in registers), wavefronts 4-7 the
// weight gradient (32 x 32 channels each, five taps), both from the same staged
// rows; 160 v_mfma_f32_32x32x16_bf16 each per tile.  The next tile's rows are
// fetched into registers meanwhile.
// FIRST: the layer below is layer 1, whose dz is needed only for its weights:
// dzp stays in LDS and dW1[tap][co][c] = sum_y dzp[y, co] f[c, y + tap - 2],
// db1 = sum dzp follow there, the 15 features of a position (in three bfloat16
// terms) and a one for the bias as the 16 columns of v_mfma_f32_16x16x32_bf16.  That
// variant takes all 256 registers and spills 9 more.
// ---------------------------------------------------------------------------
template <int D>
struct BwdTile {
    static constexpr int ROWS = TB + 4 * D;       // staged rows of dz
    static constexpr int GS = CH + 4;             // row stride of GELU'(z) (floats)
    static constexpr size_t lds = (size_t)(ROWS + 2 * TB) * RS * sizeof(__bf16) + (size_t)TB * GS * sizeof(float);
};
constexpr int NWH = KT * CH * CH + CH;   // partials of a 64 -> 64 layer: weights, biases
constexpr int NW1P = KT * CH * 3 + CH;   // of layer 1

template <int D, bool FIRST>
__global__ void __launch_bounds__(512) k_bwd_hidden(const __bf16 *__restrict__ dz, const __bf16 *__restrict__ zp,
                                                    const __bf16 *__restrict__ Wt, __bf16 *__restrict__ dzp,
                                                    float *__restrict__ part, const float *__restrict__ nu,
                                                    const float *__restrict__ tau, float *__restrict__ part1,
                                                    int ntiles, int L) {
    constexpr int ROWS = BwdTile<D>::ROWS, GS = BwdTile<D>::GS;
    extern __shared__ unsigned char smem[];
    __bf16 *dt = reinterpret_cast<__bf16 *>(smem);             // [ROWS][RS]: dz of x0 - 2 D ..
    __bf16 *at = dt + ROWS * RS;                               // [TB][RS]: a of the layer below
    __bf16 *ot = at + TB * RS;                                 // [TB][RS]: dzp
    float *gp = reinterpret_cast<float *>(ot + TB * RS);       // [TB][GS]: GELU'(zp)
    __shared__ float fs[2][3][FIRST ? TB + 4 : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool weights = wave >= 4;  // this wavefront's half of the work
    const int lr = lane & 31, lh = lane >> 5, g = lane >> 4, j16 = lane & 15;
    const bf16x8 zero8 = {};
    const int tps = L / TB;
    const int t0 = (int)((int64_t)blockIdx.x * ntiles / gridDim.x), t1 = (int)((int64_t)(blockIdx.x + 1) * ntiles / gridDim.x);

    constexpr int PD = (ROWS * 8 + 511) / 512;
    bf16x8 dn[PD], zn[2];
    float fn[1];
    auto fetch = [&](int t) {
        const int b = t / tps, x0 = (t % tps) * TB;
#pragma unroll
        for (int k = 0; k < PD; ++k) {
            const int i = threadIdx.x + 512 * k, r = i >> 3, pos = x0 - 2 * D + r;
            dn[k] = (r < ROWS && pos >= 0 && pos < L) ? *(const bf16x8 *)(dz + ((int64_t)b * L + pos) * CH + 8 * (i & 7))
                                                     : zero8;
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            zn[k] = *(const bf16x8 *)(zp + (int64_t)t * TB * CH + (int64_t)(threadIdx.x + 512 * k) * 8);
        if (FIRST && threadIdx.x < 3 * (TB + 4))
            fn[0] = feature(nu, tau, b, L, threadIdx.x / (TB + 4), x0 - 2 + threadIdx.x % (TB + 4));
    };

    // wavefronts 0-3: the weights of output channels 32 nb ..; wavefronts 4-7: sums
    const int nb = wave & 1, ph = (wave >> 1) & 1;
    bf16x8 wb[KT][4];
    floatx16 acc[KT];
    if (!weights) {
#pragma unroll
        for (int tap = 0; tap < KT; ++tap)
#pragma unroll
            for (int kc = 0; kc < 4; ++kc)
                wb[tap][kc] = *(const bf16x8 *)(Wt + (int64_t)(tap * CH + nb * 32 + lr) * CH + 16 * kc + 8 * lh);
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) acc[t] = floatx16{};
    floatx4 acc1[2] = {};
    float bsum[8] = {};
    if (t0 < t1) fetch(t0);
    for (int t = t0; t < t1; ++t) {
        // stage: rows of dz, a and GELU' of the tile
#pragma unroll
        for (int k = 0; k < PD; ++k) {
            const int i = threadIdx.x + 512 * k, r = i >> 3;
            if (r < ROWS) *(bf16x8 *)(dt + r * RS + 8 * (i & 7)) = dn[k];
            if (r >= 2 * D && r < 2 * D + TB) {
#pragma unroll
                for (int j = 0; j < 8; ++j) bsum[j] += to_f(dn[k][j]);
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = threadIdx.x + 512 * k, p = i >> 3, c = 8 * (i & 7);
            bf16x8 av;
            float dg[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float ga;
                gelu_both(to_f(zn[k][j]), ga, dg[j]);
                av[j] = to_bf(ga);
            }
            *(bf16x8 *)(at + p * RS + c) = av;
            *(floatx4 *)(gp + p * GS + c) = floatx4{dg[0], dg[1], dg[2], dg[3]};
            *(floatx4 *)(gp + p * GS + c + 4) = floatx4{dg[4], dg[5], dg[6], dg[7]};
        }
        if (FIRST && threadIdx.x < 3 * (TB + 4)) fs[t & 1][threadIdx.x / (TB + 4)][threadIdx.x % (TB + 4)] = fn[0];
        __syncthreads();
        if (t + 1 < t1) fetch(t + 1);
        if (!weights) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = 64 * ph + 32 * h + lr;  // this lane's position of the tile
                floatx16 s = {};
#pragma unroll
                for (int tap = 0; tap < KT; ++tap) {
                    const __bf16 *row = dt + (p + (KT - 1 - tap) * D) * RS + 8 * lh;
#pragma unroll
                    for (int kc = 0; kc < 4; ++kc)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[tap][kc], *(const bf16x8 *)(row + 16 * kc), s, 0, 0, 0);
                }
                // element r: channel 32 nb + 8 (r / 4) + 4 lh + r % 4 of position p
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = 32 * nb + 8 * q + 4 * lh;
                    const floatx4 dg = *(const floatx4 *)(gp + p * GS + c);
                    *reinterpret_cast<uint2 *>(ot + p * RS + c) = make_uint2(pack_bf2(s[4 * q] * dg[0], s[4 * q + 1] * dg[1]),
                                                                            pack_bf2(s[4 * q + 2] * dg[2], s[4 * q + 3] * dg[3]));
                }
            }
        } else {
            // channels co 32 nb .., ci 32 ph ..; rows 16 ks + 8 lh .. of 16 lanes' columns
            const __bf16 *ab = at + (8 * lh + (j16 >> 2)) * RS + 32 * ph + 16 * (g & 1) + 4 * (j16 & 3);
            const __bf16 *db = dt + (8 * lh + (j16 >> 2)) * RS + 32 * nb + 16 * (g & 1) + 4 * (j16 & 3);
#pragma unroll 2
            for (int ks = 0; ks < TB; ks += 16) {
                const bf16x8 bv = column8(ab + ks * RS);
#pragma unroll
                for (int tap = 0; tap < KT; ++tap) {
                    const bf16x8 av = column8(db + (ks + (KT - 1 - tap) * D) * RS);
                    acc[tap] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[tap], 0, 0, 0);
                }
            }
        }
        __syncthreads();  // dzp is whole; dt, at and gp are free
        if (!FIRST) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = threadIdx.x + 512 * k;
                *(bf16x8 *)(dzp + (int64_t)t * TB * CH + (int64_t)i * 8) = *(const bf16x8 *)(ot + (i >> 3) * RS + 8 * (i & 7));
            }
        } else {
            // positions 32 (wave % 4) .., channels 32 (wave / 4) ..; column j16: feature (tap, c) = (j16 / 3, j16 % 3)
            const int x = 32 * (wave & 3) + 8 * g;
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = j16 < 15 ? fs[t & 1][j16 % 3][x + j + j16 / 3] : 1.0f;
            Split3 d;
            d.set(f);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const bf16x8 av = column8(ot + (x + (j16 >> 2)) * RS + 32 * (wave >> 2) + 16 * cb + 4 * (j16 & 3));
#pragma unroll
                for (int q = 0; q < 3; ++q) acc1[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, d.t[q], acc1[cb], 0, 0, 0);
            }
        }
    }
    float *pg = part + (int64_t)blockIdx.x * NWH;
    if (weights) {
#pragma unroll
        for (int tap = 0; tap < KT; ++tap)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int co = 32 * nb + 8 * (r >> 2) + 4 * lh + (r & 3);
                pg[(tap * CH + co) * CH + 32 * ph + lr] = acc[tap][r];
            }
    }
    // biases: thread (row group, channel group) sums, then over the 64 row groups in order
    float *bs = gp;  // [64][CH]; the last barrier of the loop freed it
#pragma unroll
    for (int j = 0; j < 8; ++j) bs[(threadIdx.x >> 3) * CH + 8 * (threadIdx.x & 7) + j] = bsum[j];
    float *f1 = bs + 64 * CH;  // [4][CH][16]: the first layer's sums of the four position groups
    __syncthreads();
    if (threadIdx.x < CH) {
        float s = 0.0f;
        for (int k = 0; k < 64; ++k) s += bs[k * CH + threadIdx.x];
        pg[KT * CH * CH + threadIdx.x] = s;
    }
    if (FIRST) {
        // row 4 g + r of block cb: channel 32 (wave / 4) + 16 cb + 4 g + r, column j16
        float *o = f1 + (wave & 3) * CH * 16;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[(32 * (wave >> 2) + 16 * cb + 4 * g + r) * 16 + j16] = acc1[cb][r];
        __syncthreads();
        float *p1 = part1 + (int64_t)blockIdx.x * NW1P;
        for (int i = threadIdx.x; i < CH * 16; i += 512) {
            const int co = i >> 4, k = i & 15;
            const float s = ((f1[i] + f1[CH * 16 + i]) + f1[2 * CH * 16 + i]) + f1[3 * CH * 16 + i];
            p1[k < 15 ? ((k / 3) * CH + co) * 3 + k % 3 : KT * CH * 3 + co] = s;
        }
    }
}

// The gradient from all partials: dst[i] = sum over g of part[g][i] in a fixed
// order (four interleaved sums, g = j mod 4, then ((s0 + s1) + s2) + s3), the four
// layers' outputs one after the other.  64 outputs of one layer per workgroup.
struct Segments {
    const float *part[4];
    int groups[4], n[4], first[4];  // partials, outputs, first workgroup
    int dst[4];                     // first output in the gradient
};
__global__ void __launch_bounds__(256) k_reduce(Segments s, float *__restrict__ grad) {
    __shared__ float sums[4][64];
    int l = 0;
#pragma unroll
    for (int k = 1; k < 4; ++k)
        if ((int)blockIdx.x >= s.first[k]) l = k;
    const int t = threadIdx.x & 63, j = threadIdx.x >> 6;
    const int i = (blockIdx.x - s.first[l]) * 64 + t, n = s.n[l], G = s.groups[l];
    const float *part = s.part[l];
    float a = 0.0f;
    if (i < n) {
#pragma unroll 16
        for (int g = j; g < G; g += 4) a += part[(int64_t)g * n + i];
    }
    sums[j][t] = a;
    __syncthreads();
    if (j == 0 && i < n) grad[s.dst[l] + i] = ((sums[0][t] + sums[1][t]) + sums[2][t]) + sums[3][t];
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t bwd_out(const float *dout, const __bf16 *W4, const __bf16 *z3, __bf16 *dz3, float *part, int G, int B,
                   int L, hipStream_t s) {
    if (L % TB || G < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bwd_out, dim3(G), dim3(256), 0, s, dout, W4, z3, dz3, part, B * (L / TB), L);
    return hipGetLastError();
}

hipError_t bwd_hidden(int d, const __bf16 *dz, const __bf16 *zp, const __bf16 *Wt, __bf16 *dzp, float *part,
                      const float *nu, const float *tau, float *part1, int G, int B, int L, hipStream_t s) {
    if (L % TB || G < 1) return hipErrorInvalidValue;
    const int nt = B * (L / TB);
    static LdsLimit limit9, limit3;
    if (d == 9) {
        const hipError_t e = limit9.raise((const void *)k_bwd_hidden<9, false>, (int)BwdTile<9>::lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_bwd_hidden<9, false>), dim3(G), dim3(512), BwdTile<9>::lds, s, dz, zp, Wt, dzp, part, nu, tau,
                           part1, nt, L);
    } else if (d == 3) {
        const hipError_t e = limit3.raise((const void *)k_bwd_hidden<3, true>, (int)BwdTile<3>::lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_bwd_hidden<3, true>), dim3(G), dim3(512), BwdTile<3>::lds, s, dz, zp, Wt, dzp, part, nu, tau,
                           part1, nt, L);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// parts and groups of layers 1-4, outputs n[l] at dst[l] of the gradient
hipError_t reduce(const float *const (&part)[4], const int (&groups)[4], const int (&n)[4], const int (&dst)[4],
                  float *grad, hipStream_t s) {
    Segments sg;
    int blocks = 0;
    for (int l = 0; l < 4; ++l) {
        sg.part[l] = part[l];
        sg.groups[l] = groups[l];
        sg.n[l] = n[l];
        sg.dst[l] = dst[l];
        sg.first[l] = blocks;
        blocks += (n[l] + 63) / 64;
    }
    hipLaunchKernelGGL(k_reduce, dim3(blocks), dim3(256), 0, s, sg, grad);
    return hipGetLastError();
}

}  // namespace srg
