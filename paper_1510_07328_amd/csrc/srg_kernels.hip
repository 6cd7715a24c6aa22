// Kernels of the 1D convolutional surrogate: forward, backward and Adam.
//
// Network: features (n-1)/0.25, u/0.25, (tau-0.75)/0.25 -> conv 3->64 (dilation 1)
// -> GELU -> conv 64->64 (d 3) -> GELU -> conv 64->64 (d 9) -> GELU -> conv 64->2
// (d 27) = y;  n' = n + 0.25 y0, u' = u + 0.25 y1.  Kernel 5, zero padding.
// conv(a)[x, co] = b[co] + sum_{tap, ci} W[tap][co][ci] a[x + (tap-2) d, ci].
//
// Storage: activations bfloat16, channels last ([B][L][64]); weights bfloat16
// (from float32 master copies), accumulation float32.  The two 64->64 layers
// (97% of the flops) run on the bf16 matrix cores: a workgroup computes a 64
// (positions) x 64 (channels) tile as four 32x32 blocks, one per wavefront, with
// v_mfma_f32_32x32x16_bf16 over K = 5 taps x 64 channels.  The backward pass is in
// srg_backward.hip.
#include "srg_common.h"

namespace srg {

// ---------------------------------------------------------------------------
// layer 1: 3 -> 64, dilation 1, on the matrix cores.  A 16 x 16 block (16
// channels x 16 positions) is one v_mfma_f32_16x16x32_bf16 over 32 slots
// k = 8 g + j (g = lane / 16).  The features F of slot j are
//   g = 0, 1: n(t), t = 0..4, then u(0), u(1), u(2);
//   g = 2, 3: u(3), u(4), the bias slot, tau(t), t = 0..4,
// where n(t), u(t), tau(t) are the scaled n, u, tau at position x + t - 2 (zero
// outside the sample).  Even g hold bf16(F), odd g bf16(F - bf16(F)); both
// multiply the same bfloat16 weight, so each product sees about 16 bits of the
// float32 feature (the weights are bfloat16 already).  The bias slot is split
// the other way: its feature is 1 in both and its weights are the float32 bias
// as bf16(b) (g = 2) and bf16(b - bf16(b)) (g = 3).  The sum starts from zero.
// A lane's results are the 4 consecutive channels 4 g + r of position lane % 16.
// The fused inference builds the same operands, so its layer 1 equals this
// kernel's bit for bit.
// ---------------------------------------------------------------------------
constexpr int P1F = 256;
// feature slots of a lane group: (feature channel, tap) with channel 3 = the bias slot
__device__ __forceinline__ int l1_slot_ch(int s, int j) { return s == 0 ? (j < 5 ? 0 : 1) : (j < 2 ? 1 : (j == 2 ? 3 : 2)); }
__device__ __forceinline__ int l1_slot_tap(int s, int j) { return s == 0 ? (j < 5 ? j : j - 5) : (j < 2 ? 3 + j : (j == 2 ? 0 : j - 3)); }

// bf16(a), bf16(b) packed (lo = false) or the bfloat16 roundings of their
// remainders a - bf16(a), b - bf16(b) (lo = true)
__device__ __forceinline__ unsigned hl_pair(float a, float b, bool lo) {
    const unsigned hi = pack_bf2(a, b);
    const float ha = __builtin_bit_cast(float, hi << 16), hb = __builtin_bit_cast(float, hi & 0xffff0000u);
    const unsigned rem = pack_bf2(a - ha, b - hb);
    return lo ? rem : hi;
}
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
// The weight operand of channel ch for lane group g.
__device__ __forceinline__ bf16x8 l1_weights(const __bf16 *__restrict__ W1, const float *__restrict__ b1, int ch,
                                             int g) {
    auto w = [&](int t, int f) { return W1[(t * CH + ch) * 3 + f]; };
    const float bias = b1[ch];
    const __bf16 bh = to_bf(bias), bl = to_bf(bias - to_f(bh));
    if (g < 2) return bf16x8{w(0, 0), w(1, 0), w(2, 0), w(3, 0), w(4, 0), w(0, 1), w(1, 1), w(2, 1)};
    return bf16x8{w(3, 1), w(4, 1), g == 2 ? bh : bl, w(0, 2), w(1, 2), w(2, 2), w(3, 2), w(4, 2)};
}
// The features operand of a lane of group g from its 8 slot features (the bias
// slot's value is ignored).
__device__ __forceinline__ bf16x8 l1_features(const float (&F)[8], int g) {
    const bool lo = g & 1;
    u32x4_t v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = hl_pair(F[2 * i], F[2 * i + 1], lo);
    if (g >= 2) v[1] = (v[1] & 0xffff0000u) | 0x3f80u;  // the bias slot: 1.0
    return __builtin_bit_cast(bf16x8, v);
}

// A workgroup (4 wavefronts) takes 256 positions of one sample, a wavefront 64
// (four 16-position groups, each for the 64 channels as four 16 x 16 blocks);
// the scaled n, u, tau of the workgroup's positions (with a 2-position halo) are
// staged in LDS.  A wavefront's results go through an LDS tile of its 64 rows and
// leave as 16-byte row stores: z1 (only when not null: a forward that is
// followed by a backward), then a1 = bf16(GELU(z)) by the table.
__global__ void __launch_bounds__(256) k_l1_fwd(const float *__restrict__ nu, const float *__restrict__ tau,
                                                const __bf16 *__restrict__ W1, const float *__restrict__ b1,
                                                __bf16 *__restrict__ z1, __bf16 *__restrict__ a1, int L) {
    __shared__ float fs[3][P1F + 4];
    __shared__ __attribute__((aligned(16))) __bf16 tile[4][64 * RS];  // per wavefront: 64 rows of 64 channels
    __shared__ unsigned short gt[GeluT16::N];
    const int b = blockIdx.y, x0 = blockIdx.x * P1F;
    for (int i = threadIdx.x; i < 3 * (P1F + 4); i += blockDim.x) {
        const int c = i / (P1F + 4), k = i % (P1F + 4);
        fs[c][k] = feature(nu, tau, b, L, c, x0 - 2 + k);
    }
    GeluT16::fill(gt);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lc = lane & 15, g = lane >> 4, s = g >> 1;
    bf16x8 wa[4];
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) wa[cg] = l1_weights(W1, b1, 16 * cg + lc, g);
    __syncthreads();
    __bf16 *tw = tile[wave];
    const int xw = x0 + 64 * wave;  // L is a multiple of 128: a wavefront's 64 positions are all inside or all past the end
    if (xw >= L) return;
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
        const int xl = 64 * wave + 16 * pg;
        float F[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int c = l1_slot_ch(s, j);
            const float v = fs[c == 3 ? 0 : c][xl + lc + l1_slot_tap(s, j)];
            F[j] = c == 3 ? 1.0f : v;
        }
        const bf16x8 f = l1_features(F, g);
        __bf16 *trow = tw + (16 * pg + lc) * RS + 4 * g;
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
            const floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[cg], f, floatx4{}, 0, 0, 0);
            *reinterpret_cast<uint2 *>(trow + 16 * cg) =
                make_uint2(pack_bf2(acc[0], acc[1]), pack_bf2(acc[2], acc[3]));
        }
    }
    // the wavefront's z tile, rows of 128 bytes: 8 lanes per row, 8 rows per pass
    const int rr = lane >> 3, cv = 8 * (lane & 7);
    const int64_t obase = ((int64_t)b * L + xw) * CH;
    // the tile is the wavefront's own: order its writes before the reads below
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int pass = 0; pass < 8; ++pass) {
        const int r = 8 * pass + rr;
        const bf16x8 zv = *reinterpret_cast<const bf16x8 *>(tw + r * RS + cv);
        if (z1) *reinterpret_cast<bf16x8 *>(z1 + obase + (int64_t)r * CH + cv) = zv;
        const u32x4_t zq = __builtin_bit_cast(u32x4_t, zv);
        unsigned zz[4] = {zq[0], zq[1], zq[2], zq[3]}, av[4];
        gelu_bf2_n<GeluT16>(zz, av, gt);
        *reinterpret_cast<u32x4_t *>(a1 + obase + (int64_t)r * CH + cv) = u32x4_t{av[0], av[1], av[2], av[3]};
    }
}

// ---------------------------------------------------------------------------
// 64 -> 64 layers on the matrix cores (profiles longer than the one-kernel
// forward takes): out[x, n] = bias[n] + sum_{tap,k} in[x + (tap-2)d, k] Wop[tap][n][k];
// stores a = bf16(GELU(z)) with z = bf16(out), and z itself when out_z is not null.
// A workgroup keeps the layer's weights in LDS and walks tiles of TM = 128
// positions (b, x0) with stride gridDim.x; each of its 4 wavefronts computes 32
// positions x 64 channels as two 32 x 32 blocks (v_mfma_f32_32x32x16_bf16, K =
// 5 taps x 64 channels).  LDS rows are padded to 72 elements so that the 16-byte
// operand reads of 8 consecutive rows fall in distinct banks.  Results go back
// through LDS and leave as 16-byte row stores.
// ---------------------------------------------------------------------------
constexpr int TM = 128;

__global__ void __launch_bounds__(256) k_hidden(const __bf16 *__restrict__ in, const __bf16 *__restrict__ Wop,
                                                const float *__restrict__ bias,
                                                __bf16 *__restrict__ out_z, __bf16 *__restrict__ out_a, int B, int L,
                                                int d) {
    extern __shared__ unsigned char smem[];
    __bf16 *wl = reinterpret_cast<__bf16 *>(smem);  // [5 * 64][RS]
    __bf16 *tile = wl + KT * CH * RS;  // [TM + 4d][RS] input rows, then the results [TM][RS]
    for (int i = threadIdx.x; i < KT * CH * (CH / 8); i += blockDim.x)
        *(bf16x8 *)(wl + (i >> 3) * RS + 8 * (i & 7)) = ((const bf16x8 *)Wop)[i];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = 32 * wave, lr = lane & 31, lk = 8 * (lane >> 5);
    const int tiles_per_sample = L / TM, ntiles = B * tiles_per_sample;
    const int rows = TM + 4 * d;
    const bf16x8 zero8 = {};
    // The input rows of a tile (at most (TM + 36) x 8 vectors of 16 bytes, i.e. 6
    // per thread) are fetched into registers one tile ahead, so that their
    // latency overlaps the previous tile's matrix and epilogue work.
    constexpr int PF = ((TM + 4 * 9) * (CH / 8) + 255) / 256;
    bf16x8 pf[PF];
    auto fetch = [&](int t) {
        const int b = t / tiles_per_sample, x0 = (t % tiles_per_sample) * TM;
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = threadIdx.x + 256 * k;
            const int r = i >> 3, v = i & 7;
            const int pos = x0 - 2 * d + r;
            pf[k] = (r < rows && pos >= 0 && pos < L) ? *(const bf16x8 *)(in + ((int64_t)b * L + pos) * CH + 8 * v)
                                                     : zero8;
        }
    };
    if ((int)blockIdx.x < ntiles) fetch(blockIdx.x);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int b = t / tiles_per_sample, x0 = (t % tiles_per_sample) * TM;
        __syncthreads();  // weights loaded / previous tile's results written out
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = threadIdx.x + 256 * k;
            if ((i >> 3) < rows) *(bf16x8 *)(tile + (i >> 3) * RS + 8 * (i & 7)) = pf[k];
        }
        __syncthreads();
        if (t + (int)gridDim.x < ntiles) fetch(t + gridDim.x);
        floatx16 acc0 = {}, acc1 = {};
#pragma unroll
        for (int r = 0; r < 16; ++r) {  // the sums start from the bias
            acc0[r] = bias[lr];
            acc1[r] = bias[32 + lr];
        }
#pragma unroll
        for (int tap = 0; tap < KT; ++tap) {
            const int off = tap * d;
            const __bf16 *arow = tile + (m0 + lr + off) * RS + lk;
            const __bf16 *b0row = wl + (tap * CH + lr) * RS + lk;
            const __bf16 *b1row = b0row + 32 * RS;
#pragma unroll
            for (int kc = 0; kc < CH; kc += 16) {
                const bf16x8 av = *(const bf16x8 *)(arow + kc);
                const bf16x8 bv0 = *(const bf16x8 *)(b0row + kc);
                const bf16x8 bv1 = *(const bf16x8 *)(b1row + kc);
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv0, acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv1, acc1, 0, 0, 0);
            }
        }
        __syncthreads();  // every wavefront is done reading the input tile
        // D[i][j]: i = 8 (r / 4) + 4 (lane / 32) + r % 4 (position), j = lane % 32 (channel)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int pl = m0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            tile[pl * RS + lr] = to_bf(acc0[r]);
            tile[pl * RS + 32 + lr] = to_bf(acc1[r]);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < TM * (CH / 8); i += blockDim.x) {
            const int p = i >> 3, v = i & 7;
            const int64_t row = ((int64_t)b * L + x0 + p) * CH + 8 * v;
            const bf16x8 zv = *(const bf16x8 *)(tile + p * RS + 8 * v);
            if (out_z) *(bf16x8 *)(out_z + row) = zv;
            bf16x8 av;
#pragma unroll
            for (int j = 0; j < 8; ++j) av[j] = to_bf(gelu(to_f(zv[j])));
            *(bf16x8 *)(out_a + row) = av;
        }
    }
}

// ---------------------------------------------------------------------------
// layer 4: 64 -> 2, dilation 27, on the matrix cores.  A workgroup stages the a3
// rows of its 256 positions and their +-54 halo in LDS once; then, for 16 positions at a time
// a wavefront forms y[x, c] = sum_{tap, ci} a3[x + (tap-2) 27, ci] W4[tap][c][ci] as a
// [16 x 320] x [320 x 16] product, 10 steps of v_mfma_f32_16x16x32_bf16 (K = one
// tap x 32 channels per step), the two output columns padded to 16 with zero
// weights.  A operand: lane l holds position l % 16 and channels 8 (l / 16) ..
// + 7 of the step's 32 (one 16-byte load of the a3 row); B operand: lane l holds
// column l % 16, the same 8 channels; D: lane l holds column l % 16 of
// positions 4 (l / 16) .. + 3.  Forward writes n' = n + 0.25 (b4[0] + y0) and
// u' = u + 0.25 (b4[1] + y1) ([B][2][L]).
// ---------------------------------------------------------------------------
constexpr int P4F = 256;     // positions per workgroup (4 wavefronts x 4 passes of 16)
constexpr int RS4 = CH + 8;  // LDS row stride (elements) of the staged a3 rows

__global__ void __launch_bounds__(256) k_l4_fwd(const __bf16 *__restrict__ a3, const __bf16 *__restrict__ W4,
                                                const float *__restrict__ b4, const float *__restrict__ nu,
                                                float *__restrict__ out, int L) {
    // a3 rows x0 - 54 .. x0 + 256 + 53 (zero outside [0, L)), rows padded to 72 elements
    __shared__ __bf16 rows[(P4F + 4 * 27) * RS4];
    const int b = blockIdx.y, x0 = blockIdx.x * P4F;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, kq = lane >> 4;
    const bf16x8 zero8 = {};
    for (int i = threadIdx.x; i < (P4F + 4 * 27) * (CH / 8); i += blockDim.x) {
        const int r = i >> 3, v = i & 7;
        const int pos = x0 - 2 * 27 + r;
        *(bf16x8 *)(rows + r * RS4 + 8 * v) =
            (pos >= 0 && pos < L) ? *(const bf16x8 *)(a3 + ((int64_t)b * L + pos) * CH + 8 * v) : zero8;
    }
    bf16x8 bw[2 * KT];
#pragma unroll
    for (int kb = 0; kb < 2 * KT; ++kb) {
        const int tap = kb >> 1, ci = 32 * (kb & 1) + 8 * kq;
        bw[kb] = col < 2 ? *(const bf16x8 *)(W4 + (tap * 2 + col) * CH + ci) : zero8;
    }
    const float bias = col < 2 ? b4[col] : 0.0f;
    __syncthreads();
    for (int p = 16 * wave; p < P4F; p += 64) {
        if (x0 + p >= L) break;  // uniform per wavefront (L is a multiple of 128)
        floatx4 acc = {};
#pragma unroll
        for (int kb = 0; kb < 2 * KT; ++kb) {
            const int r = p + col + (kb >> 1) * 27;  // row of position x0 + p + col + (tap - 2) 27
            const bf16x8 av = *(const bf16x8 *)(rows + r * RS4 + 32 * (kb & 1) + 8 * kq);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bw[kb], acc, 0, 0, 0);
        }
        if (col < 2) {
            const int64_t o = (int64_t)b * 2 * L + (int64_t)col * L;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xi = x0 + p + 4 * kq + r;
                out[o + xi] = nu[o + xi] + FS * (bias + acc[r]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Inference forward, all four layers in one kernel: the activations never leave
// LDS.  One workgroup (8 wavefronts) streams NS samples (one or two) from left to
// right in chunks of FC = 64 positions: sample k occupies the stream positions
// [k (L + FC), k (L + FC) + L), and the chunk between two samples is padding
// (wider than the 54-position reach of the widest layer, so no tap sees the
// other sample).  Each of a1, a2, a3 lives in a ring of FR = 256 rows (stream
// position X in row X mod 256, rows of 72 elements as above).  In iteration c,
// layer k produces the chunk of positions [64 c - D_k, 64 c - D_k + 64) with
// D = 0, 96, 192, 320: each layer lags the one below by at least a chunk plus
// its receptive half-width (2 d), so that everything it reads was written in an
// earlier iteration, and the rows a layer writes in an iteration are never read
// in that iteration (ring spans 166, 178 and 246 rows < 256).  One barrier per
// iteration.  Rows at positions outside the samples hold zeros (the zero
// padding); chunks and blocks outside skip their arithmetic (L is a multiple of
// 64, so every chunk and 32- or 16-row block lies wholly inside a sample or
// wholly outside).
// Work split: every wave takes two 16 x 16 blocks of layer 1 (operands as in
// k_l1_fwd); waves 0-3 the four 32 x 32 blocks of layer 2 and, 16 positions
// each, layer 4; waves 4-7 the blocks of layer 3.  A 32 x 32 block is channels x
// positions, with the weights as the first operand, so that a lane's results
// are 4 x 4 consecutive channels of one position (four 8-byte stores); each
// wave keeps its slices of its layers' weights in registers.  The raw n, u of the
// samples are staged in LDS before the loop (8 L bytes per sample, so
// NS L <= FMAXL), which leaves no global load inside it: a load there would make
// the wait for it also wait for the output stores in flight.  The features of
// the next chunk are written to a double buffer during each iteration.  The GELU
// is the 16 KB table (GeluT32), its reads issued together and the results
// stored; the rare wavefront with a value outside the table then replaces those
// words (a test before the reads, with the branch between them and the stores,
// cost about 4 %).  Every output element takes
// the same operations in the same order as in k_l1_fwd, k_hidden and k_l4_fwd,
// so the result equals theirs bit for bit.
// ---------------------------------------------------------------------------
constexpr int FC = 64, FR = 256, FMAXL = 4096;
constexpr int FFP = FC + 8;  // feature buffer row: positions 64 c - 2 .. 64 c + 65
// a segment of a sample starts its stream FLEAD positions early and ends it FLEAD
// late: the reach of the four layers' taps, rounded up to a 32-row block
constexpr int FLEAD = 96;
static_assert(FLEAD >= 2 * (1 + 3 + 9 + 27) && FLEAD % 32 == 0, "the lead covers the taps");
// lag of layer k >= lag of layer k - 1 + one chunk + the half-width 2 d_k of its
// taps, rounded up to a multiple of 32 so that no 32-row block wraps its ring
constexpr int FD2 = 96, FD3 = 192, FD4 = 320;
static_assert(FD2 >= FC + 2 * 3 && FD3 >= FD2 + FC + 2 * 9 && FD4 >= FD3 + FC + 2 * 27, "lags cover the taps");
static_assert(FD2 % 32 == 0 && FD3 % 32 == 0 && FD4 % 32 == 0, "blocks aligned to 32 rows");
// ring span: from the lowest row read to the highest row written in one iteration
static_assert(FD2 + 2 * 3 + FC <= FR && FD3 + 2 * 9 - FD2 + FC <= FR && FD4 + 2 * 27 - FD3 + FC <= FR,
              "ring spans");
static_assert(FC >= 2 * 27, "the padding chunk between two samples covers the widest reach");
constexpr int FMAXS = 2;  // samples per workgroup (the sample of a stream position is one comparison)
constexpr size_t FUSED_RINGS = (size_t)3 * FR * RS * sizeof(__bf16);  // then NS x 2 x (L + 4) floats of n, u

template <bool KEEP, bool SEG>
__global__ void __launch_bounds__(512) k_fwd_fused(const float *__restrict__ nu, const float *__restrict__ tau,
                                                   const __bf16 *__restrict__ W1, const float *__restrict__ b1,
                                                   const __bf16 *__restrict__ W2, const float *__restrict__ b2,
                                                   const __bf16 *__restrict__ W3, const float *__restrict__ b3,
                                                   const __bf16 *__restrict__ W4, const float *__restrict__ b4,
                                                   float *__restrict__ out, __bf16 *__restrict__ z1,
                                                   __bf16 *__restrict__ z2, __bf16 *__restrict__ z3, int B, int L,
                                                   int spw, int segs, int seglen) {
    extern __shared__ unsigned char smem[];
    __bf16 *r1 = reinterpret_cast<__bf16 *>(smem);  // a1 ring [FR][RS]
    __bf16 *r2 = r1 + FR * RS;                      // a2 ring
    __bf16 *r3 = r2 + FR * RS;                      // a3 ring
    // the samples of this workgroup, or its segment: positions [x0, x0 + len) of one
    // sample, the stream starting `lead` positions before
    const int s0 = SEG ? (int)blockIdx.x / segs : (int)blockIdx.x * spw;
    const int ns = SEG ? 1 : (B - s0 < spw ? B - s0 : spw);
    const int x0 = SEG ? ((int)blockIdx.x % segs) * seglen : 0;
    const int len = SEG && L - x0 >= seglen ? seglen : L - x0;
    const int lead = x0 < FLEAD ? x0 : FLEAD, base = x0 - lead;
    const int W = SEG ? (L - x0 - len < FLEAD ? L : x0 + len + FLEAD) - base : L;  // stream positions of a sample
    // per sample raw n then u, each with two cells of padding per side (n = 1, u = 0: features 0)
    float *nus = reinterpret_cast<float *>(smem + FUSED_RINGS);
    const int LP = W + 4;
    __shared__ unsigned short gt[GeluT32::N];       // GELU table
    __shared__ float feat[2 * 3 * FFP];             // features of the current and the next chunk
    const int SL = W + FC;                          // stream stride of a sample
    const int LT = ns * SL - FC;                    // stream length
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bf16x8 zero8 = {};
    for (int i = threadIdx.x; i < 3 * FR * RS / 8; i += blockDim.x) reinterpret_cast<bf16x8 *>(smem)[i] = zero8;
    GeluT32::fill(gt);
    for (int i = threadIdx.x; i < ns * 2 * LP; i += blockDim.x) {
        const int k = i / (2 * LP), r = i - k * 2 * LP;
        const int ch = r >= LP, x = base + r - ch * LP - 2;
        nus[i] = (x >= 0 && x < L) ? nu[(int64_t)(s0 + k) * 2 * L + (int64_t)ch * L + x] : (ch ? 0.0f : 1.0f);
    }
    // stream position X < 2 SL: sample k = (X >= SL), position base + X - k SL of it
    auto inside = [&](int X) { return X >= 0 && X < LT && X - (X >= SL ? SL : 0) < W; };
    // of the positions this workgroup writes
    auto own = [&](int X) { return SEG ? X >= lead && X < lead + len : inside(X); };
    // row of a stream position inside a sample in the kept activations
    auto row_of = [&](int X) { return (int64_t)(s0 + (X >= SL)) * L + (base + X - (X >= SL ? SL : 0)); };
    // layers 1-3: this wave's block (positions 32 mb .., channels 32 nb ..)
    const bool upper = wave >= 4;  // layer 3 and layer 1
    const int mb = wave & 1, nb = (wave >> 1) & 1;
    const int lr = lane & 31, lk = 8 * (lane >> 5);
    // layer 1: 16 positions 16 (wave % 4) .. of each chunk, channels 32 (wave / 4) ..
    // as two 16 x 16 blocks; lane = (position lc, slot group g1)
    const int lc = lane & 15, g1 = lane >> 4, s1 = g1 >> 1, pg1 = wave & 3, h1 = wave >> 2;
    bf16x8 wa1[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) wa1[q] = l1_weights(W1, b1, 32 * h1 + 16 * q + lc, g1);
    const __bf16 *Wl = upper ? W3 : W2;
    bf16x8 wb[KT][4];
#pragma unroll
    for (int tap = 0; tap < KT; ++tap)
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
            wb[tap][kc] = *(const bf16x8 *)(Wl + (int64_t)(tap * CH + nb * 32 + lr) * CH + 16 * kc + lk);
    // layer 4 (waves 0-3): lane = (position col within 16, channel quarter kq)
    const int col = lane & 15, kq = lane >> 4;
    bf16x8 bw[2 * KT];
#pragma unroll
    for (int kb = 0; kb < 2 * KT; ++kb) {
        const int tap = kb >> 1, ci = 32 * (kb & 1) + 8 * kq;
        bw[kb] = col < 2 ? *(const bf16x8 *)(W4 + (tap * 2 + col) * CH + ci) : zero8;
    }
    const float bias4 = col < 2 ? b4[col] : 0.0f;
    // layers 2 / 3: the biases of this lane's 16 result channels
    // nb 32 + 8 (r / 4) + 4 (lane / 32) + r % 4
    floatx16 bz;
#pragma unroll
    for (int r = 0; r < 16; ++r) bz[r] = (upper ? b3 : b2)[nb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)];
    // per sample: the tau feature
    float ftau[FMAXS];
#pragma unroll
    for (int k = 0; k < FMAXS; ++k) ftau[k] = k < ns ? (tau[s0 + k] - TAU_C) / FS : 0.0f;
    const int d = upper ? 9 : 3, D = upper ? FD3 : FD2;
    const __bf16 *rin = upper ? r2 : r1;
    __bf16 *rout = upper ? r3 : r2;
    const int niter = ((SEG ? lead + len : LT) + FD4 - 1) / FC + 1;
    // Let the weight loads land before the loop: otherwise the compiler's wait
    // counts inside the loop stay conservative and every iteration's last matrix
    // operation waits for all vector-memory traffic in flight (the previous
    // chunk's stores).  vmcnt(0), the other counters free.
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();

    // layer 1: two 16 x 16 blocks (operands as in k_l1_fwd)
    auto layer1 = [&](int c) {
        const int X = c * FC + 16 * pg1 + lc;  // this lane's position
        __bf16 *orow = r1 + (X & (FR - 1)) * RS + 32 * h1 + 4 * g1;
        if (!inside(c * FC + (SEG ? 16 * pg1 : 0))) {
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<uint2 *>(orow + 16 * q) = make_uint2(0u, 0u);
        } else {
            const float *fb = feat + (c & 1) * 3 * FFP + 16 * pg1 + lc;
            float F[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int ch = l1_slot_ch(s1, j);
                const float v = fb[(ch == 3 ? 0 : ch) * FFP + l1_slot_tap(s1, j)];
                F[j] = ch == 3 ? 1.0f : v;
            }
            const bf16x8 f = l1_features(F, g1);
            unsigned zq[4], g[4];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa1[q], f, floatx4{}, 0, 0, 0);
                zq[2 * q] = pack_bf2(acc[0], acc[1]);
                zq[2 * q + 1] = pack_bf2(acc[2], acc[3]);
            }
            gelu_bf2_table<GeluT32>(zq, g, gt);
            if (KEEP && (!SEG || own(c * FC + 16 * pg1))) {
                __bf16 *zr = z1 + row_of(X) * CH + 32 * h1 + 4 * g1;
#pragma unroll
                for (int q = 0; q < 2; ++q) *reinterpret_cast<uint2 *>(zr + 16 * q) = make_uint2(zq[2 * q], zq[2 * q + 1]);
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<uint2 *>(orow + 16 * q) = make_uint2(g[2 * q], g[2 * q + 1]);
            if (__builtin_amdgcn_ballot_w64(gelu_bf2_outside<GeluT32>(zq) != 0u) != 0) {  // rare
#pragma unroll
                for (int i = 0; i < 4; ++i) g[i] = gelu_bf2_word<GeluT32>(zq[i], gt);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    *reinterpret_cast<uint2 *>(orow + 16 * q) = make_uint2(g[2 * q], g[2 * q + 1]);
            }
        }
    };
    // layer 2 (waves 0-3) or 3 (waves 4-7): one 32 x 32 block, channels x positions
    auto block = [&](int c) {
        const int p0 = c * FC - D + 32 * mb;  // a multiple of 32: the block's rows do not wrap
        // result element r of this lane: position p0 + lr, channel nb 32 + 8 (r / 4) + 4 (lane / 32) + r % 4
        __bf16 *orow = rout + ((p0 + lr) & (FR - 1)) * RS + nb * 32 + 4 * (lane >> 5);
        if (!inside(p0)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2 *>(orow + 8 * q) = make_uint2(0u, 0u);
        } else {
            floatx16 acc = bz;  // the sums start from the bias
            // the operands of tap t + 1 are read while tap t's products run (the
            // scheduling barriers keep the compiler from moving the reads back
            // next to their products, where each pair waited for its own reads)
            bf16x8 av[2][4];
            auto fetch = [&](int tap, bf16x8 (&v)[4]) {
                const __bf16 *arow = rin + ((p0 + lr + (tap - 2) * d) & (FR - 1)) * RS + lk;
#pragma unroll
                for (int kc = 0; kc < 4; ++kc) v[kc] = *(const bf16x8 *)(arow + 16 * kc);
            };
            fetch(0, av[0]);
#pragma unroll
            for (int tap = 0; tap < KT; ++tap) {
                if (tap + 1 < KT) fetch(tap + 1, av[(tap + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kc = 0; kc < 4; ++kc)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[tap][kc], av[tap & 1][kc], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            unsigned zq[8], g[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) zq[i] = pack_bf2(acc[2 * i], acc[2 * i + 1]);
            gelu_bf2_table<GeluT32>(zq, g, gt);
            if (KEEP && (!SEG || own(p0))) {
                __bf16 *zr = (upper ? z3 : z2) + row_of(p0 + lr) * CH + nb * 32 + 4 * (lane >> 5);
#pragma unroll
                for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2 *>(zr + 8 * q) = make_uint2(zq[2 * q], zq[2 * q + 1]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2 *>(orow + 8 * q) = make_uint2(g[2 * q], g[2 * q + 1]);
            if (__builtin_amdgcn_ballot_w64(gelu_bf2_outside<GeluT32>(zq) != 0u) != 0) {  // rare
#pragma unroll
                for (int i = 0; i < 8; ++i) g[i] = gelu_bf2_word<GeluT32>(zq[i], gt);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<uint2 *>(orow + 8 * q) = make_uint2(g[2 * q], g[2 * q + 1]);
            }
        }
    };
    // layer 4 (waves 0-3): 16 positions each, n' = n + 0.25 (b4 + y)
    auto layer4 = [&](int c) {
        const int p = c * FC - FD4 + 16 * wave;
        if (own(p)) {
            floatx4 acc = {};
            bf16x8 av[2 * KT];  // all ten operands read before the first product
#pragma unroll
            for (int kb = 0; kb < 2 * KT; ++kb) {
                const int pos = p + col + ((kb >> 1) - 2) * 27;
                av[kb] = *(const bf16x8 *)(r3 + (pos & (FR - 1)) * RS + 32 * (kb & 1) + 8 * kq);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < 2 * KT; ++kb)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[kb], bw[kb], acc, 0, 0, 0);
            if (col < 2) {
                const int k = p >= SL, xl = p - k * SL;
                const int64_t o = (int64_t)(s0 + k) * 2 * L + (int64_t)col * L + base;
                const float *nk = nus + k * 2 * LP + col * LP + 2;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int xi = xl + 4 * kq + r;
                    out[o + xi] = nk[xi] + FS * (bias4 + acc[r]);
                }
            }
        }
    };
    // the features n, u, tau of stream positions 64 (c + 1) - 2 .. 64 (c + 1) + 65
    // into the feature buffer of chunk c + 1 (zero outside the samples), by the
    // first 204 threads
    auto features = [&](int c) {
        const int i = threadIdx.x;
        if (i < 3 * (FC + 4)) {
            const int ch = i / (FC + 4), q = i % (FC + 4);
            const int X = (c + 1) * FC - 2 + q;
            float v = 0.0f;
            if (inside(X)) {
                const int k = X >= SL, xl = X - k * SL;
                if (ch == 2) {
                    v = k ? ftau[1] : ftau[0];
                } else {
                    const float raw = nus[k * 2 * LP + ch * LP + xl + 2];
                    v = ch == 0 ? (raw - 1.0f) / FS : raw / FS;
                }
            }
            feat[((c + 1) & 1) * 3 * FFP + ch * FFP + q] = v;
        }
    };
    features(-1);
    __syncthreads();
    // The sections of an iteration read only what earlier iterations wrote, so
    // their order within an iteration is free.
    for (int c = 0; c < niter; ++c) {
        layer1(c);
        block(c);
        if (!upper) layer4(c);
        features(c);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// loss: e = (out - target) / 0.25 over both fields; L = mean(e^2) + lambda mean_b (mean_x e0)^2
// (the second term asks for conserved mass without enforcing it).
// dout = dL/d out; per-sample sums of e^2 and e0 written to stats[b][2].
// One workgroup per sample.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_loss(const float *__restrict__ out, const float *__restrict__ target,
                                              float *__restrict__ dout, float *__restrict__ stats, int B, int L,
                                              float lambda_mass) {
    const int b = blockIdx.x;
    const int64_t o = (int64_t)b * 2 * L;
    float se = 0.0f, s0 = 0.0f;
    for (int i = threadIdx.x; i < 2 * L; i += blockDim.x) {
        const float e = (out[o + i] - target[o + i]) / FS;
        se += e * e;
        if (i < L) s0 += e;
    }
    __shared__ float r1[256], r2[256];
    r1[threadIdx.x] = se;
    r2[threadIdx.x] = s0;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            r1[threadIdx.x] += r1[threadIdx.x + s];
            r2[threadIdx.x] += r2[threadIdx.x + s];
        }
        __syncthreads();
    }
    const float mean_e0 = r2[0] / L;
    const float N = float(B) * 2.0f * L;
    for (int i = threadIdx.x; i < 2 * L; i += blockDim.x) {
        const float e = (out[o + i] - target[o + i]) / FS;
        float g = 2.0f * e / N;
        if (i < L) g += lambda_mass * 2.0f * mean_e0 / (float(B) * L);
        dout[o + i] = g / FS;
    }
    if (threadIdx.x == 0) {
        stats[2 * b] = r1[0];
        stats[2 * b + 1] = mean_e0;
    }
}

// per-sample relative mass residual |sum n' - sum n| / sum n of a prediction
__global__ void __launch_bounds__(256) k_mass_residual(const float *__restrict__ in, const float *__restrict__ out,
                                                       float *__restrict__ resid, int L) {
    const int b = blockIdx.x;
    const int64_t o = (int64_t)b * 2 * L;
    double s_in = 0.0, s_out = 0.0;
    for (int i = threadIdx.x; i < L; i += blockDim.x) {
        s_in += in[o + i];
        s_out += out[o + i];
    }
    __shared__ double r1[256], r2[256];
    r1[threadIdx.x] = s_in;
    r2[threadIdx.x] = s_out;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            r1[threadIdx.x] += r1[threadIdx.x + s];
            r2[threadIdx.x] += r2[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) resid[b] = float(fabs(r2[0] - r1[0]) / r1[0]);
}

// Acceptance indicator of a prediction for the hybrid advance: the relative
// mass residual as above, or +inf when any predicted value is not finite or
// any predicted density is not positive (a state the lattice step cannot take).
__global__ void __launch_bounds__(256) k_indicator(const float *__restrict__ in, const float *__restrict__ out,
                                                   float *__restrict__ resid, int L) {
    const int b = blockIdx.x;
    const int64_t o = (int64_t)b * 2 * L;
    double s_in = 0.0, s_out = 0.0;
    int bad = 0;
    for (int i = threadIdx.x; i < L; i += blockDim.x) {
        const float n1 = out[o + i], u1 = out[o + L + i];
        bad |= (int)!(n1 > 0.0f) | (int)!isfinite(n1) | (int)!isfinite(u1);
        s_in += in[o + i];
        s_out += n1;
    }
    __shared__ double r1[256], r2[256];
    __shared__ int rb[256];
    r1[threadIdx.x] = s_in;
    r2[threadIdx.x] = s_out;
    rb[threadIdx.x] = bad;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            r1[threadIdx.x] += r1[threadIdx.x + s];
            r2[threadIdx.x] += r2[threadIdx.x + s];
            rb[threadIdx.x] |= rb[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) resid[b] = rb[0] ? __builtin_inff() : float(fabs(r2[0] - r1[0]) / r1[0]);
}


// ---------------------------------------------------------------------------
// Adam on the float32 master vector (bias-corrected), then the bfloat16 copies.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                              const float *__restrict__ g, int n, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// bf16 copies: plain copy for [tap][co][ci] and the transposed [tap][ci][co] of a 64x64 layer
__global__ void __launch_bounds__(256) k_to_bf16(const float *__restrict__ src, __bf16 *__restrict__ dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = to_bf(src[i]);
}

__global__ void __launch_bounds__(256) k_transpose_bf16(const float *__restrict__ src, __bf16 *__restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KT * CH * CH) return;
    const int tap = i / (CH * CH), co = (i / CH) % CH, ci = i % CH;
    dst[(tap * CH + ci) * CH + co] = to_bf(src[i]);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t l1_fwd(const float *nu, const float *tau, const __bf16 *W1, const float *b1, __bf16 *z1, __bf16 *a1, int B,
                  int L, hipStream_t s) {
    hipLaunchKernelGGL(k_l1_fwd, dim3((L + P1F - 1) / P1F, B), dim3(256), 0, s, nu, tau, W1, b1, z1, a1, L);
    return hipGetLastError();
}

size_t hidden_lds(int d) { return (size_t)(KT * CH + TM + 4 * d) * RS * sizeof(__bf16); }

hipError_t hidden(const __bf16 *in, const __bf16 *Wop, const float *bias, __bf16 *out_z, __bf16 *out_a, int B, int L,
                  int d, hipStream_t s) {
    if (L % TM || (d != 3 && d != 9)) return hipErrorInvalidValue;
    static LdsLimit limit;
    const hipError_t attr = limit.raise((const void *)k_hidden, (int)hidden_lds(9));
    if (attr != hipSuccess) return attr;
    const int ntiles = B * (L / TM);
    const int grid = ntiles < 512 ? ntiles : 512;  // two workgroups per CU (about 70 KB of LDS each)
    hipLaunchKernelGGL(k_hidden, dim3(grid), dim3(256), hidden_lds(d), s, in, Wop, bias, out_z, out_a, B, L, d);
    return hipGetLastError();
}

int fused_max_length() { return FMAXL; }

hipError_t fwd_fused(const float *nu, const float *tau, const __bf16 *W1, const float *b1, const __bf16 *W2,
                     const float *b2, const __bf16 *W3, const float *b3, const __bf16 *W4, const float *b4, float *out,
                     __bf16 *z1, __bf16 *z2, __bf16 *z3, int B, int L, hipStream_t s) {
    if (B < 1 || L < FC || L % FC || L > FMAXL) return hipErrorInvalidValue;
    constexpr size_t kMaxStage = (size_t)2 * (FMAXL + 4) > (size_t)FMAXS * 2 * (FMAXL / FMAXS + 4)
                                     ? (size_t)2 * (FMAXL + 4)
                                     : (size_t)FMAXS * 2 * (FMAXL / FMAXS + 4);
    // with the static LDS (the GELU table and the feature buffers), within the 160 KiB of a workgroup
    static_assert(FUSED_RINGS + kMaxStage * sizeof(float) + GeluT32::N * sizeof(unsigned short) +
                          2 * 3 * FFP * sizeof(float) <= 160 * 1024,
                  "LDS of the largest staging");
    // two samples per workgroup once there are more samples than compute units
    // (one workgroup fits a CU): the padding chunk between them replaces the
    // pipeline's fill and drain, and no second wave of workgroups is needed
    const int cus = device_cus();
    const int spw = (cus > 0 && B > cus && L * FMAXS <= FMAXL) ? FMAXS : 1;
    // With fewer samples than compute units a sample is cut into segments of whole
    // chunks, one workgroup each: a workgroup takes len / 64 + 5 iterations for len
    // positions and 1.5 more for a segment's lead, which the cut has to repay.
    // Whole samples against segments, us per call: 1 x 384 23.6 -> 19.3, 1 x 1024
    // 41.2 -> 19.7, 1 x 4096 126 -> 20.0, 64 x 1024 42.8 -> 27.4, 40 x 4096 128 -> 40.5
    // (layer by layer with the activations kept: 26.6, 27.8, 29.2, 47.2, 69.0).
    // Not in place (out == nu): a segment stages its neighbours' ends of n, u while
    // they write theirs; a whole sample is staged by the workgroup that writes it.
    int segs = 1, seglen = L;
    if (cus > 0 && B < cus && out != nu) {
        const int want = cus / B < L / FC ? cus / B : L / FC;
        const int sl = (L / FC + want - 1) / want * FC;
        if (sl + FLEAD < L) {
            seglen = sl;
            segs = (L + sl - 1) / sl;
        }
    }
    const int grid = segs > 1 ? B * segs : (B + spw - 1) / spw;
    const int window = segs > 1 && seglen + 2 * FLEAD < L ? seglen + 2 * FLEAD : L;
    const size_t lds = FUSED_RINGS + (size_t)spw * 2 * (window + 4) * sizeof(float);
    using Kernel = decltype(&k_fwd_fused<false, false>);
    static constexpr Kernel kernels[4] = {k_fwd_fused<false, false>, k_fwd_fused<true, false>, k_fwd_fused<false, true>,
                                          k_fwd_fused<true, true>};
    static LdsLimit limits[4];
    const int v = (z1 ? 1 : 0) + (segs > 1 ? 2 : 0);
    const hipError_t attr = limits[v].raise((const void *)kernels[v], (int)(FUSED_RINGS + kMaxStage * sizeof(float)));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kernels[v], dim3(grid), dim3(512), lds, s, nu, tau, W1, b1, W2, b2, W3, b3, W4, b4, out, z1, z2, z3,
                       B, L, spw, segs, seglen);
    return hipGetLastError();
}

hipError_t l4_fwd(const __bf16 *a3, const __bf16 *W4, const float *b4, const float *nu, float *out, int B, int L,
                  hipStream_t s) {
    hipLaunchKernelGGL(k_l4_fwd, dim3((L + P4F - 1) / P4F, B), dim3(256), 0, s, a3, W4, b4, nu, out, L);
    return hipGetLastError();
}

hipError_t loss(const float *out, const float *target, float *dout, float *stats, int B, int L, float lambda,
                hipStream_t s) {
    hipLaunchKernelGGL(k_loss, dim3(B), dim3(256), 0, s, out, target, dout, stats, B, L, lambda);
    return hipGetLastError();
}

hipError_t mass_residual(const float *in, const float *out, float *resid, int B, int L, hipStream_t s) {
    hipLaunchKernelGGL(k_mass_residual, dim3(B), dim3(256), 0, s, in, out, resid, L);
    return hipGetLastError();
}

hipError_t indicator(const float *in, const float *out, float *resid, int B, int L, hipStream_t s) {
    hipLaunchKernelGGL(k_indicator, dim3(B), dim3(256), 0, s, in, out, resid, L);
    return hipGetLastError();
}

hipError_t adam(float *p, float *m, float *v, const float *g, int n, float lr, float b1, float b2, float eps, float c1,
                float c2, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, p, m, v, g, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t to_bf16(const float *src, __bf16 *dst, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3((n + 255) / 256), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

hipError_t transpose_bf16(const float *src, __bf16 *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_transpose_bf16, dim3((KT * CH * CH + 255) / 256), dim3(256), 0, s, src, dst);
    return hipGetLastError();
}

}  // namespace srg
