// Kernels of the reconstruction network (learned decimation): a BF16 GEMM
// on gfx950 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation),
// im2col for 3x3 convolutions, and the elementwise pieces of training
// (bias + ReLU epilogue, ReLU backward, 2x2 average pool and nearest
// upsample with their adjoints, channel concat/split, loss, Adam, tone
// map).  Activations are NHWC; every image dimension and channel count the
// network uses is a multiple of 8 and 32.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "nn_internal.h"

namespace splotch {
namespace nn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ bf16_t f2bf(float f) {
    // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return (bf16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// ------------------------------------------------------------------ GEMM
// C[z][M][N] (FP32) = sum over k in split z of A[m][k] * B[k][n].
// A is [M][K] (lda) or, with TRANS_A, stored as [K][M] (lda).  B is [K][N].
// Workgroup tile BM x BN x 32 with 4 waves; each wave owns (BM/WM) x
// (BN/WN) outputs as 16x16 MFMA tiles.
constexpr int BK = 32;
constexpr int PAD = 8;  // LDS row pad (bf16) keeps 16-byte fragment reads aligned

template <int BM, int BN, bool TRANS_A>
__global__ __launch_bounds__(256) void k_gemm(const bf16_t *A, const bf16_t *B, float *C, int M,
                                              int N, int K, int lda, int ldb, int k_per_split) {
    constexpr int WN = BN / 32 >= 2 ? 2 : 1;  // waves along N
    constexpr int WM = 4 / WN;                // waves along M
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16;  // MFMA tiles per wave
    __shared__ __attribute__((aligned(16))) bf16_t sA[BM][BK + PAD];
    __shared__ __attribute__((aligned(16))) bf16_t sB[BN][BK + PAD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
    const int kbeg = blockIdx.z * k_per_split;
    const int kend = min(K, kbeg + k_per_split);
    f32x4 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = kbeg; k0 < kend; k0 += BK) {
        // stage A tile as sA[m][k]
        for (int e = tid; e < BM * BK / 8; e += 256) {
            if (!TRANS_A) {
                const int r = e / (BK / 8), c8 = (e % (BK / 8)) * 8;
                const int m = m0 + r, k = k0 + c8;
                const bf16_t *src = A + (size_t)m * lda + k;
                if (m < M && k + 8 <= kend && ((reinterpret_cast<uintptr_t>(src) & 15u) == 0)) {
                    *reinterpret_cast<uint4 *>(&sA[r][c8]) = *reinterpret_cast<const uint4 *>(src);
                } else {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        sA[r][c8 + q] = (m < M && k + q < kend) ? src[q] : (bf16_t)0;
                }
            } else {
                const int kr = e / (BM / 8), m8 = (e % (BM / 8)) * 8;
                const int k = k0 + kr;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int m = m0 + m8 + q;
                    sA[m8 + q][kr] = (m < M && k < kend) ? A[(size_t)k * lda + m] : (bf16_t)0;
                }
            }
        }
        // stage B tile transposed as sB[n][k]
        for (int e = tid; e < BN * BK / 8; e += 256) {
            const int kr = e / (BN / 8), n8 = (e % (BN / 8)) * 8;
            const int k = k0 + kr;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int n = n0 + n8 + q;
                sB[n8 + q][kr] = (n < N && k < kend) ? B[(size_t)k * ldb + n] : (bf16_t)0;
            }
        }
        __syncthreads();
        const int kq = (lane >> 4) * 8;
        bf16x8 af[TM], bfr[TN];
#pragma unroll
        for (int a = 0; a < TM; ++a)
            af[a] = *reinterpret_cast<const bf16x8 *>(&sA[(wm * TM + a) * 16 + (lane & 15)][kq]);
#pragma unroll
        for (int b = 0; b < TN; ++b)
            bfr[b] = *reinterpret_cast<const bf16x8 *>(&sB[(wn * TN + b) * 16 + (lane & 15)][kq]);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
        __syncthreads();
    }
    float *Cz = C + (size_t)blockIdx.z * M * N;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int n = n0 + (wn * TN + b) * 16 + (lane & 15);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = m0 + (wm * TM + a) * 16 + (lane >> 4) * 4 + q;
                if (m < M && n < N) Cz[(size_t)m * N + n] = acc[a][b][q];
            }
        }
}

// Tone-map scale: the host value, or the device sum times inv_count (the
// image mean); a non-positive or non-finite scale becomes 1.
__device__ __forceinline__ float tone_scale(const float *sum, float inv_count, float s) {
    if (sum) s = sum[0] * inv_count;
    return (s > 0.f && s < 3.0e38f) ? s : 1.f;
}

// ------------------------------------------------------- fused 3x3 convolution
// Forward weights [cout][9 cin] from the GEMM operand [9 cin][cout]: row n
// holds output channel n's taps (tap-major, then input channel), so a
// lane's 8 consecutive reduction terms are one 16-byte read.
__global__ void k_conv_wf(const bf16_t *w, bf16_t *wf, int cin, int cout) {
    const size_t k9 = (size_t)9 * cin, total = k9 * cout;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const size_t n = e / k9, k = e % k9;
        wf[e] = w[k * cout + n];
    }
}

// out = epilogue(conv3x3(x, W) + bias) for NHWC BF16 x, without an im2col
// buffer: the implicit GEMM (pixels x cout, reduction over 9 taps x cin)
// runs on the matrix cores from LDS.  A workgroup owns an 8 x 16 pixel
// tile and CO output channels; per 32-channel slice of the input it stages
// the tile with its one-pixel halo (zeros outside the image) and the
// slice's weights for all 9 taps, then each wave accumulates 2 rows of 16
// pixels x CO channels, one MFMA per (row, 16 channels) per tap.  Small
// tiles: for the deep levels, whose pixels would not fill the GPU otherwise,
// and for inputs of more than 128 channels (k_conv3x3_wide does the others).
// 64 output channels a workgroup stage the input half as often and are slower
// (60 KB of LDS, two workgroups a CU instead of four): 192 to 64 channels on
// eight 1024 x 1024 images 4.44 ms instead of 3.56, 256 to 128 on four
// 256 x 256 337 us instead of 264.
constexpr int kCTH = 8, kCTW = 16;           // output tile rows, columns
constexpr int kCHW = kCTW + 2;               // halo tile width
constexpr int kCHP = (kCTH + 2) * kCHW;      // halo tile pixels
constexpr int kCK = 32;                      // input channels per stage
constexpr int kCRow = kCK + PAD;             // LDS row (bf16); 80 B spreads the banks

__global__ __launch_bounds__(256) void k_conv3x3(const bf16_t *x, const bf16_t *wf,
                                                 const float *bias, int relu,
                                                 const float *residual, bf16_t *out_bf,
                                                 float *out_f, int h, int w, int cin, int cout) {
    constexpr int CO = 32, NT = CO / 16;
    __shared__ __attribute__((aligned(16))) bf16_t sX[kCHP][kCRow];
    __shared__ __attribute__((aligned(16))) bf16_t sW[9 * CO][kCRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (w + kCTW - 1) / kCTW, tiles_y = (h + kCTH - 1) / kCTH;
    const int tile = (int)(blockIdx.x % (unsigned)(tiles_x * tiles_y));
    const int img = (int)(blockIdx.x / (unsigned)(tiles_x * tiles_y));
    const int y0 = (tile / tiles_x) * kCTH, x0 = (tile % tiles_x) * kCTW;
    const int n0 = (int)blockIdx.y * CO;
    const size_t k9 = (size_t)9 * cin;
    const size_t plane = (size_t)img * h;
    f32x4 acc[2][NT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kq = (lane >> 4) * 8;
    for (int c0 = 0; c0 < cin; c0 += kCK) {
        __syncthreads();  // the previous slice's fragments are read
        for (int e = tid; e < kCHP * 4; e += 256) {
            const int p = e >> 2, q = (e & 3) * 8;
            const int yy = y0 - 1 + p / kCHW, xx = x0 - 1 + p % kCHW;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (yy >= 0 && yy < h && xx >= 0 && xx < w)
                v = *reinterpret_cast<const uint4 *>(x + ((plane + yy) * w + xx) * cin + c0 + q);
            *reinterpret_cast<uint4 *>(&sX[p][q]) = v;
        }
        for (int e = tid; e < 9 * CO * 4; e += 256) {
            const int r = e >> 2, q = (e & 3) * 8;
            const int tap = r / CO, nl = r % CO;
            *reinterpret_cast<uint4 *>(&sW[r][q]) = *reinterpret_cast<const uint4 *>(
                wf + (size_t)(n0 + nl) * k9 + (size_t)tap * cin + c0 + q);
        }
        __syncthreads();
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3, dx = tap % 3;
            bf16x8 af[2], bfr[NT];
#pragma unroll
            for (int a = 0; a < 2; ++a)
                af[a] = *reinterpret_cast<const bf16x8 *>(
                    &sX[(2 * wave + a + dy) * kCHW + (lane & 15) + dx][kq]);
#pragma unroll
            for (int b = 0; b < NT; ++b)
                bfr[b] = *reinterpret_cast<const bf16x8 *>(&sW[tap * CO + b * 16 + (lane & 15)][kq]);
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b],
                                                                        0, 0, 0);
        }
    }
    // output (pixel, channel) of acc[a][b][q]: row 2 wave + a, column
    // 4 (lane / 16) + q of the tile; channel n0 + 16 b + lane % 16
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int yy = y0 + 2 * wave + a;
        if (yy >= h) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int xx = x0 + (lane >> 4) * 4 + q;
            if (xx >= w) continue;
            const size_t pix = (plane + yy) * w + xx;
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int n = n0 + b * 16 + (lane & 15);
                const size_t e = pix * cout + n;
                float v = acc[a][b][q];
                if (bias) v += bias[n];
                if (relu) v = v > 0.f ? v : 0.f;
                if (residual) v += residual[e];
                if (out_bf) out_bf[e] = f2bf(v);
                if (out_f) out_f[e] = v;
            }
        }
    }
}

// The same convolution, with the same sums bit for bit, for images with
// enough pixels: a workgroup owns a 16 x 32 pixel tile and 32 output
// channels, each of its four waves 8 rows of 16 pixels.  The weights of a
// 32-channel slice sit in registers (9 taps x 32 channels, 72 registers), read
// once where the input has one slice and the workgroups go through the tiles
// in turns; an input row's three fragments serve three output rows, so a
// wave issues 144 MFMAs for 30 fragment reads of LDS.  The weights are the
// MFMA's first operand: a lane then holds four consecutive channels of a
// pixel, and stores, bias and residual are 8- and 16-byte accesses.
// The next tile's pixels are fetched into registers while a tile is
// multiplied.  1024 x 1024 pixels of 32 channels take 39 us (76 us with FP32
// residual and output), where the kernel above, whose workgroups stage 23 KB
// of weights for 128 pixels and store two bytes a lane, takes 71 us (173 us)
// and reading and writing the images 27 us (64 us) at a copy's rate.
//
// Inputs of SL = 2 to 4 slices keep all their weights in LDS (23 KB a slice)
// and read a slice's into the registers at each step; their tiles have four
// rows a wave, so that two workgroups still fit a CU at SL = 2.
constexpr int kWTW = 32, kWHW = kWTW + 2;
template <int SL>
struct Wide {
    static constexpr int R = SL == 1 ? 8 : 4;  // rows a wave
    static constexpr int TH = 2 * R;           // rows a tile
    static constexpr int HP = (TH + 2) * kWHW; // pixels with the halo
};

// HEAD is the last layer of one image's reconstruction.  The residual is the
// tone map of the decimated image in the first three channels and zero in the
// others, so it comes from that image itself, and the first three channels are
// mapped back into the planar image where they are computed: beside the
// layer's FP32 output neither an FP32 input of 32 channels (134 MB for
// 1024 x 1024 pixels) nor a pass that maps back touches memory: a
// reconstruction of that size takes 715 us, 764 in separate steps.
struct Head {
    const float *dec;  // planar [3][h][w]
    const float *sum;  // its sum and 1 / (3 h w): the tone-map scale
    float inv_count;
    float *img;        // planar [3][h][w], may be dec
};
template <int SL, bool HEAD = false>
__global__ __launch_bounds__(256, SL <= 2 ? 2 : 1) void k_conv3x3_wide(const bf16_t *x, const bf16_t *wf,
                                                         const float *bias, int relu,
                                                         const float *residual, bf16_t *out_bf,
                                                         float *out_f, int n, int h, int w,
                                                         int cin, int cout, Head head) {
    constexpr int NB = 2;  // 16-channel blocks
    constexpr int R = Wide<SL>::R, TH = Wide<SL>::TH, HP = Wide<SL>::HP;
    __shared__ __attribute__((aligned(16))) bf16_t sX[HP][kCRow];
    __shared__ __attribute__((aligned(16))) bf16_t sWt[SL > 1 ? SL * 9 * 32 : 1][kCRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int px = lane & 15, kq = (lane >> 4) * 8;
    const int tiles_x = (w + kWTW - 1) / kWTW, tiles_y = (h + TH - 1) / TH;
    const uint32_t per_img = (uint32_t)(tiles_x * tiles_y), tiles = per_img * (uint32_t)n;
    const int n0 = (int)blockIdx.y * 32;
    const size_t k9 = (size_t)9 * cin;
    const int col = (wave & 1) * 16 + px, row = (wave >> 1) * R;
    bf16x8 wr[9][NB];
    if (SL > 1) {
        // [slice][tap][output channel] rows
        for (int e = tid; e < SL * 9 * 32 * 4; e += 256) {
            const int r = e >> 2, q = (e & 3) * 8, sl = r / 288, tap = r % 288 / 32;
            if (sl * kCK >= cin) break;
            *reinterpret_cast<uint4 *>(&sWt[r][q]) = *reinterpret_cast<const uint4 *>(
                wf + (size_t)(n0 + (r & 31)) * k9 + (size_t)tap * cin + sl * kCK + q);
        }
    }
    auto load_w = [&](int c0) {
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                wr[tap][b] =
                    SL > 1 ? *reinterpret_cast<const bf16x8 *>(
                                 &sWt[(c0 / kCK * 9 + tap) * 32 + b * 16 + px][kq])
                           : *reinterpret_cast<const bf16x8 *>(
                                 wf + (size_t)(n0 + b * 16 + px) * k9 + (size_t)tap * cin + kq);
    };
    float4 bv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const float *q = bias + n0 + b * 16 + (lane >> 4) * 4;
        bv[b] = bias ? make_float4(q[0], q[1], q[2], q[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // A step is a 32-channel slice of a tile.  The next step's pixels are in
    // flight, in registers, while this one's are multiplied.
    constexpr int kLoads = (HP * 4 + 255) / 256;
    uint4 next[kLoads];
    auto fetch = [&](uint32_t t, int c0) {
        const int img = (int)(t / per_img), tt = (int)(t % per_img);
        const int y0 = (tt / tiles_x) * TH, x0 = (tt % tiles_x) * kWTW;
        const bf16_t *src = x + (size_t)img * h * w * cin + c0;
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int e = tid + 256 * k, p = e >> 2, q = (e & 3) * 8;
            const int yy = y0 - 1 + p / kWHW, xx = x0 - 1 + p % kWHW;
            next[k] = make_uint4(0u, 0u, 0u, 0u);
            if (p < HP && yy >= 0 && yy < h && xx >= 0 && xx < w)
                next[k] = *reinterpret_cast<const uint4 *>(src + ((size_t)yy * w + xx) * cin + q);
        }
    };
    if (blockIdx.x < tiles) fetch(blockIdx.x, 0);
    if (SL == 1) load_w(0);
    for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int img = (int)(t / per_img), tt = (int)(t % per_img);
        const int y0 = (tt / tiles_x) * TH, x0 = (tt % tiles_x) * kWTW;
        const size_t plane = (size_t)img * h;
        f32x4 acc[R][NB];
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < (SL == 1 ? kCK : cin); c0 += kCK) {
            __syncthreads();  // the previous step's fragments are read
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                const int e = tid + 256 * k;
                if (e < HP * 4) *reinterpret_cast<uint4 *>(&sX[e >> 2][(e & 3) * 8]) = next[k];
            }
            __syncthreads();
            if (SL > 1 && c0 + kCK < cin)
                fetch(t, c0 + kCK);
            else if (t + gridDim.x < tiles)
                fetch(t + gridDim.x, 0);
            if (SL > 1) load_w(c0);
            // the next row's fragments are read before a row's MFMAs; the
            // barriers keep the compiler from reading all rows at once (it
            // would spill)
            bf16x8 xf[2][3];
            auto read_row = [&](int ir) {
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    xf[ir & 1][dx] =
                        *reinterpret_cast<const bf16x8 *>(&sX[(row + ir) * kWHW + col + dx][kq]);
            };
            read_row(0);
#pragma unroll
            for (int ir = 0; ir < R + 2; ++ir) {
                if (ir + 1 < R + 2) read_row(ir + 1);
#pragma unroll
                for (int a = ir - 2; a <= ir; ++a) {
                    if (a < 0 || a >= R) continue;
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                wr[(ir - a) * 3 + dx][b], xf[ir & 1][dx], acc[a][b], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // output (pixel, channel) of acc[a][b][q]: row `row` + a, column
        // `col`; channel n0 + 16 b + 4 (lane / 16) + q
        // HEAD: the image's three channels of all rows sit in lanes 0 to 15;
        // each quarter of the wave takes the logarithms (and, below, the
        // exponentials) of R / 4 of the rows.
        constexpr int Q = R / 4;
        const bool image = HEAD && n0 == 0;
        const int quarter = lane >> 4;
        const size_t plane3 = (size_t)h * w;
        float tone[HEAD ? Q : 1][3], sc = 1.f;
        if (image) {
            sc = tone_scale(head.sum, head.inv_count, 1.0f);
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const int yy = y0 + row + quarter * Q + j;
                const bool in = yy < h && x0 + col < w;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float d = in ? head.dec[c * plane3 + (size_t)yy * w + x0 + col] : 0.f;
                    tone[j][c] = log1pf(fmaxf(d, 0.f) / sc);
                    // rounded before it is added, as from memory
                    asm volatile("" : "+v"(tone[j][c]));
                }
            }
        }
#pragma unroll
        for (int a = 0; a < R; ++a) {
            const int yy = y0 + row + a;
            float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f);
            if (image) {
                const int from = a / Q * 16 + px;
                const float t0 = __shfl(tone[a % Q][0], from, 64);
                const float t1 = __shfl(tone[a % Q][1], from, 64);
                const float t2 = __shfl(tone[a % Q][2], from, 64);
                if (lane < 16) r0 = make_float4(t0, t1, t2, 0.f);
            }
            if (yy >= h || x0 + col >= w) continue;
            const size_t pix = (plane + yy) * w + x0 + col;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const size_t e = pix * cout + n0 + b * 16 + (lane >> 4) * 4;
                float4 v = make_float4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]);
                if (bias) {
                    v.x += bv[b].x;
                    v.y += bv[b].y;
                    v.z += bv[b].z;
                    v.w += bv[b].w;
                }
                if (relu) {
                    v.x = v.x > 0.f ? v.x : 0.f;
                    v.y = v.y > 0.f ? v.y : 0.f;
                    v.z = v.z > 0.f ? v.z : 0.f;
                    v.w = v.w > 0.f ? v.w : 0.f;
                }
                if (HEAD || residual) {
                    float4 r = b == 0 ? r0 : make_float4(0.f, 0.f, 0.f, 0.f);
                    if (!HEAD) r = *reinterpret_cast<const float4 *>(residual + e);
                    v.x += r.x;
                    v.y += r.y;
                    v.z += r.z;
                    v.w += r.w;
                }
                if (out_bf)
                    *reinterpret_cast<ushort4 *>(out_bf + e) =
                        make_ushort4(f2bf(v.x), f2bf(v.y), f2bf(v.z), f2bf(v.w));
                if (out_f) *reinterpret_cast<float4 *>(out_f + e) = v;
            }
        }
        if (image) {
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const int yy = y0 + row + quarter * Q + j;
                float v[3];
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const float t = __shfl(acc[k * Q + j][0][c], px, 64);
                        if (k == 0 || quarter == k) v[c] = t;
                    }
                if (yy >= h || x0 + col >= w) continue;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    head.img[c * plane3 + (size_t)yy * w + x0 + col] =
                        sc * expm1f(v[c] + bias[c] + tone[j][c]);
            }
        }
    }
}

// Adjoint weights: wf[ci][9 cout], the forward operand w[9 cin][cout] with
// its taps mirrored and channels swapped, so that backward-data is the same
// convolution of dZ (cout channels in, cin out).
__global__ void k_conv_wf_adjoint(const bf16_t *w, bf16_t *wf, int cin, int cout) {
    const int k9 = 9 * cout, total = k9 * cin;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int ci = e / k9, k = e % k9, tap = k / cout, co = k % cout;
        wf[e] = w[((size_t)(8 - tap) * cin + ci) * cout + co];
    }
}

// The convolution with its reduction in tap-major order (tap, then input
// channels) for inputs of several 32-channel slices: the order in which
// backward-data sums.  All slices of the halo tile are staged at once and
// the weights a tap at a time.  SL: slices the tile holds (cin <= 32 SL).
template <int SL>
__global__ __launch_bounds__(256) void k_conv3x3_taps(const bf16_t *x, const bf16_t *wf,
                                                      float *out, int h, int w, int cin,
                                                      int cout) {
    constexpr int NT = 2;  // 32 output channels
    constexpr int ROW = SL * kCK + PAD;
    __shared__ __attribute__((aligned(16))) bf16_t sX[kCHP][ROW];
    __shared__ __attribute__((aligned(16))) bf16_t sW[2][32][ROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (w + kCTW - 1) / kCTW, tiles_y = (h + kCTH - 1) / kCTH;
    const int tile = (int)(blockIdx.x % (unsigned)(tiles_x * tiles_y));
    const int img = (int)(blockIdx.x / (unsigned)(tiles_x * tiles_y));
    const int y0 = (tile / tiles_x) * kCTH, x0 = (tile % tiles_x) * kCTW;
    const int n0 = (int)blockIdx.y * 32;
    const size_t k9 = (size_t)9 * cin, plane = (size_t)img * h;
    const int c8 = cin / 8;
    for (int e = tid; e < kCHP * c8; e += 256) {
        const int p = e / c8, q = (e % c8) * 8;
        const int yy = y0 - 1 + p / kCHW, xx = x0 - 1 + p % kCHW;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (yy >= 0 && yy < h && xx >= 0 && xx < w)
            v = *reinterpret_cast<const uint4 *>(x + ((plane + yy) * w + xx) * cin + q);
        *reinterpret_cast<uint4 *>(&sX[p][q]) = v;
    }
    auto stage_w = [&](int tap) {
        for (int e = tid; e < 32 * c8; e += 256) {
            const int r = e / c8, q = (e % c8) * 8;
            *reinterpret_cast<uint4 *>(&sW[tap & 1][r][q]) = *reinterpret_cast<const uint4 *>(
                wf + (size_t)(n0 + r) * k9 + (size_t)tap * cin + q);
        }
    };
    f32x4 acc[2][NT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kq = (lane >> 4) * 8;
    stage_w(0);
    __syncthreads();
    for (int tap = 0; tap < 9; ++tap) {
        // the next tap's weights into the half that the tap before used
        if (tap + 1 < 9) stage_w(tap + 1);
        const int dy = tap / 3, dx = tap % 3;
        for (int c0 = 0; c0 < cin; c0 += kCK) {
            bf16x8 af[2], bfr[NT];
#pragma unroll
            for (int a = 0; a < 2; ++a)
                af[a] = *reinterpret_cast<const bf16x8 *>(
                    &sX[(2 * wave + a + dy) * kCHW + (lane & 15) + dx][c0 + kq]);
#pragma unroll
            for (int b = 0; b < NT; ++b)
                bfr[b] = *reinterpret_cast<const bf16x8 *>(
                    &sW[tap & 1][b * 16 + (lane & 15)][c0 + kq]);
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b],
                                                                        0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int yy = y0 + 2 * wave + a;
        if (yy >= h) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int xx = x0 + (lane >> 4) * 4 + q;
            if (xx >= w) continue;
#pragma unroll
            for (int b = 0; b < NT; ++b)
                out[((plane + yy) * w + xx) * cout + n0 + b * 16 + (lane & 15)] = acc[a][b][q];
        }
    }
}

// ------------------------------------------------------- weight gradient
// part[s][tap][ci][co] = sum over the pixels p of split s of
// x[p shifted by tap][ci] dz[p][co], without an im2col buffer: the
// reduction runs over pixels, so both MFMA operands are wanted
// channel-major.  A workgroup stages 8 x 32 pixel tiles of 32 channels of dz
// and, with the one-pixel halo, of x in LDS as they lie in memory, and
// ds_read_b64_tr_b16 transposes on the way to the registers (16 lanes read
// four pixels x 16 channels; lane l gets channel l of the four), so a tap's
// shift is a row offset.  Each of the four waves owns 16 x 16 channels and
// all nine taps (36 accumulator registers); an input row's three fragments
// serve three output rows.  The halves of a row are swapped for pixels with
// bit 3 set: the 32 lanes of a transposed read then meet distinct LDS banks.
// Bound by reading x and dz once per 32 x 32 channel block (0.54 GB, 0.11 ms
// at a copy's rate, on four 1024 x 1024 images of 32 channels): 0.24 ms
// there and 0.48 ms for 64 to 32 channels, where im2col and a split-K GEMM
// with transposing element loads took 2.73 and 7.4 ms.
constexpr int kDTH = 8, kDTW = 32, kDHW = kDTW + 2;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int dw_at(int p, int c) { return p * 32 + (c ^ ((p & 8) << 1)); }

// Eight consecutive pixels (from p) of channel c0 + lane % 16, p including
// this lane's 8 (lane / 16).
__device__ __forceinline__ bf16x8 read_tr8(const bf16_t *s, int p, int c0, int lane) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const int r = (lane & 15) >> 2, c = c0 + (lane & 3) * 4;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(s + dw_at(p + r, c)));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(s + dw_at(p + 4 + r, c)));
    const s16x8 v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

__global__ __launch_bounds__(256) void k_conv3x3_dw(const bf16_t *x, const bf16_t *dz, float *part,
                                                    int n, int h, int w, int cin, int cout) {
    __shared__ __attribute__((aligned(16))) bf16_t sX[(kDTH + 2) * kDHW * 32];
    __shared__ __attribute__((aligned(16))) bf16_t sZ[kDTH * kDTW * 32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cb = cin / 32, ci0 = (int)(blockIdx.y % (unsigned)cb) * 32,
              co0 = (int)(blockIdx.y / (unsigned)cb) * 32;
    const int mi = (wave & 1) * 16, ni = (wave >> 1) * 16;
    const int tiles_x = (w + kDTW - 1) / kDTW, tiles_y = (h + kDTH - 1) / kDTH;
    const long long tiles = (long long)tiles_x * tiles_y * n;
    const long long per = (tiles + gridDim.x - 1) / gridDim.x;
    const long long t0 = per * blockIdx.x, t1 = t0 + per < tiles ? t0 + per : tiles;
    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int g8 = (lane >> 4) * 8;
    for (long long t = t0; t < t1; ++t) {
        const int img = (int)(t / (tiles_x * tiles_y)), tt = (int)(t % (tiles_x * tiles_y));
        const int y0 = (tt / tiles_x) * kDTH, x0 = (tt % tiles_x) * kDTW;
        const size_t plane = (size_t)img * h;
        __syncthreads();  // the previous tile's fragments are read
        for (int e = tid; e < (kDTH + 2) * kDHW * 4; e += 256) {
            const int p = e >> 2, q = (e & 3) * 8;
            const int yy = y0 - 1 + p / kDHW, xx = x0 - 1 + p % kDHW;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (yy >= 0 && yy < h && xx >= 0 && xx < w)
                v = *reinterpret_cast<const uint4 *>(x + ((plane + yy) * w + xx) * cin + ci0 + q);
            *reinterpret_cast<uint4 *>(&sX[dw_at(p, q)]) = v;
        }
        for (int e = tid; e < kDTH * kDTW * 4; e += 256) {
            const int p = e >> 2, q = (e & 3) * 8;
            const int yy = y0 + p / kDTW, xx = x0 + p % kDTW;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (yy < h && xx < w)
                v = *reinterpret_cast<const uint4 *>(dz + ((plane + yy) * w + xx) * cout + co0 + q);
            *reinterpret_cast<uint4 *>(&sZ[dw_at(p, q)]) = v;
        }
        __syncthreads();
        bf16x8 af[3][3];  // input row (mod 3), tap column
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) af[r][dx] = read_tr8(sX, r * kDHW + dx + g8, mi, lane);
#pragma unroll
        for (int r = 0; r < kDTH; ++r) {
            const bf16x8 bf = read_tr8(sZ, r * kDTW + g8, ni, lane);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
                af[(r + 2) % 3][dx] = read_tr8(sX, (r + 2) * kDHW + dx + g8, mi, lane);
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
                acc[tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[(r + tap / 3) % 3][tap % 3],
                                                                   bf, acc[tap], 0, 0, 0);
        }
    }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ci = ci0 + mi + (lane >> 4) * 4 + q, co = co0 + ni + (lane & 15);
            part[(((size_t)blockIdx.x * 9 + tap) * cin + ci) * cout + co] = acc[tap][q];
        }
}

// out[e] = sum of part[s][e] over the splits: 64 values a workgroup, each
// summed by 16 threads (a thread per value took 62 us for 256 splits).
__global__ __launch_bounds__(1024) void k_sum_splits(const float *part, int splits, size_t mn,
                                                     float *out) {
    __shared__ float sh[16][64];
    const size_t e = (size_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int g = threadIdx.x >> 6;
    float v = 0.f;
    if (e < mn)
        for (int z = g; z < splits; z += 16) v += part[(size_t)z * mn + e];
    sh[g][threadIdx.x & 63] = v;
    __syncthreads();
    if (g == 0 && e < mn) {
        for (int k = 1; k < 16; ++k) v += sh[k][threadIdx.x];
        out[e] = v;
    }
}

// ------------------------------------------------------------------ im2col
// out[p][tap*C + c] = in[p shifted by tap][c] (zero outside the image),
// taps in (ky, kx) row-major order, p = (img, y, x).
__global__ void k_im2col3x3(const bf16_t *in, bf16_t *out, int n, int h, int w, int c) {
    const size_t total = (size_t)n * h * w * 9 * (c / 8);
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int c8 = (int)(e % (c / 8)) * 8;
        size_t r = e / (c / 8);
        const int tap = (int)(r % 9);
        const size_t p = r / 9;
        const int x = (int)(p % w), y = (int)((p / w) % h), img = (int)(p / ((size_t)w * h));
        const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (yy >= 0 && yy < h && xx >= 0 && xx < w)
            v = *reinterpret_cast<const uint4 *>(in + (((size_t)img * h + yy) * w + xx) * c + c8);
        *reinterpret_cast<uint4 *>(out + (p * 9 + tap) * c + c8) = v;
    }
}

// Weights of the adjoint (backward-data) convolution.  Forward weights are
// stored as the GEMM operand w[tap][ci][co]; the adjoint operand is
// wt[tap'][co][ci] = w[8 - tap'][ci][co] (taps mirrored, channels swapped).
__global__ void k_flip_weights(const bf16_t *w, bf16_t *wt, int cout, int cin) {
    const int total = 9 * cin * cout;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int co = e % cout, ci = (e / cout) % cin, tap = e / (cout * cin);
        wt[((size_t)(8 - tap) * cout + co) * cin + ci] = w[e];
    }
}

// Sum split-K partials, add bias, apply ReLU; write BF16 and/or FP32,
// optionally adding a residual (FP32) after the activation.
__global__ void k_epilogue(const float *Cp, int splits, size_t mn, int n, const float *bias,
                           int relu, const float *residual, bf16_t *out_bf, float *out_f) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < mn; e += stride) {
        float v = 0.f;
        for (int z = 0; z < splits; ++z) v += Cp[(size_t)z * mn + e];
        if (bias) v += bias[e % n];
        if (relu) v = v > 0.f ? v : 0.f;
        if (residual) v += residual[e];
        if (out_bf) out_bf[e] = f2bf(v);
        if (out_f) out_f[e] = v;
    }
}

// dZ = dY * [Y > 0] (ReLU adjoint), written as BF16 for the GEMMs (and as
// FP32 where asked for).
__global__ void k_relu_bwd(const float *dy, const bf16_t *y, int relu, bf16_t *dz_bf,
                           float *dz_f, size_t total) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        float g = dy[e];
        if (relu && !(bf2f(y[e]) > 0.f)) g = 0.f;
        dz_bf[e] = f2bf(g);
        if (dz_f) dz_f[e] = g;
    }
}

// The same for [rows][cols] with the bias gradient's per-block column sums
// of the FP32 dZ (part, as k_colsum_part's) taken on the way, four channels
// a thread: dZ in FP32 need not be written and read again.  cols is a
// multiple of 4, at most 256; y may be null (no ReLU).
__global__ __launch_bounds__(256) void k_relu_bwd_bias(const float *dy, const bf16_t *y,
                                                       size_t rows, int cols,
                                                       size_t rows_per_block, bf16_t *dz_bf,
                                                       float *part) {
    __shared__ float4 sh[256];
    const int c4 = cols / 4, per_row = 256 / c4;
    const int t = threadIdx.x, c = t % c4, r0 = t / c4;
    const size_t beg = (size_t)blockIdx.x * rows_per_block;
    const size_t end = beg + rows_per_block < rows ? beg + rows_per_block : rows;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r0 < per_row)
        for (size_t r = beg + r0; r < end; r += per_row) {
            const size_t e = r * cols + 4 * c;
            float4 g = *reinterpret_cast<const float4 *>(dy + e);
            if (y) {
                const ushort4 v = *reinterpret_cast<const ushort4 *>(y + e);
                if (!(bf2f(v.x) > 0.f)) g.x = 0.f;
                if (!(bf2f(v.y) > 0.f)) g.y = 0.f;
                if (!(bf2f(v.z) > 0.f)) g.z = 0.f;
                if (!(bf2f(v.w) > 0.f)) g.w = 0.f;
            }
            *reinterpret_cast<ushort4 *>(dz_bf + e) =
                make_ushort4(f2bf(g.x), f2bf(g.y), f2bf(g.z), f2bf(g.w));
            s.x += g.x;
            s.y += g.y;
            s.z += g.z;
            s.w += g.w;
        }
    sh[t] = s;
    __syncthreads();
    if (t < c4) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k = 0; k < per_row; ++k) {
            const float4 v = sh[k * c4 + t];
            a.x += v.x;
            a.y += v.y;
            a.z += v.z;
            a.w += v.w;
        }
        *reinterpret_cast<float4 *>(part + (size_t)blockIdx.x * cols + 4 * t) = a;
    }
}

// Column sums of in[rows][cols] (cols <= 256) in two passes: each block
// sums a contiguous chunk of rows for every column (lanes spread over
// columns, coalesced), then one pass adds the per-block partials in order.
__global__ void k_colsum_part(const float *in, size_t rows, int cols, size_t rows_per_block,
                              float *part) {
    __shared__ float sh[256];
    const int per_row = 256 / cols;  // rows covered by one sweep of the block
    const int t = threadIdx.x, c = t % cols, r0 = t / cols;
    const size_t beg = (size_t)blockIdx.x * rows_per_block;
    const size_t end = beg + rows_per_block < rows ? beg + rows_per_block : rows;
    float s = 0.f;
    if (r0 < per_row)
        for (size_t r = beg + r0; r < end; r += per_row) s += in[r * cols + c];
    sh[t] = s;
    __syncthreads();
    if (t < cols) {
        float tot = 0.f;
        for (int k = 0; k < per_row; ++k) tot += sh[k * cols + t];
        part[(size_t)blockIdx.x * cols + t] = tot;
    }
}

// Adds a column's partials (at most kColsumBlocks) in block order: the whole
// workgroup fetches them into LDS and one thread adds.  The order matters to
// the tone map's mean, whose last bit decides bfloat16 roundings all through
// the network.  (One thread that fetched and added took 64 us for 1024.)
__global__ __launch_bounds__(256) void k_colsum_final(const float *part, int nblocks, int cols,
                                                      float *out) {
    __shared__ __attribute__((aligned(16))) float sh[kColsumBlocks];
    const int c = blockIdx.x;
    for (int b = threadIdx.x; b < kColsumBlocks; b += 256)
        sh[b] = b < nblocks ? part[(size_t)b * cols + c] : 0.f;
    __syncthreads();
    if (threadIdx.x != 0) return;
    float s = 0.f;
    int b = 0;
    for (; b + 16 <= nblocks; b += 16) {
#pragma unroll
        for (int q = 0; q < 16; q += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(&sh[b + q]);
            s += v.x;
            s += v.y;
            s += v.z;
            s += v.w;
        }
    }
    for (; b < nblocks; ++b) s += sh[b];
    out[c] = s;
}

// 2x2 average pool (NHWC, BF16 in/out) and its adjoint (FP32 in/out).
// Eight channels per thread (one 16-byte load per input pixel).
__global__ void k_pool2(const bf16_t *in, bf16_t *out, int n, int h, int w, int c) {
    const int ho = h / 2, wo = w / 2, c8 = c / 8;
    const size_t total = (size_t)n * ho * wo * c8;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c8) * 8;
        size_t p = e / c8;
        const int x = (int)(p % wo), y = (int)((p / wo) % ho), img = (int)(p / ((size_t)wo * ho));
        const size_t b = (((size_t)img * h + 2 * y) * w + 2 * x) * c + ch;
        const size_t row = (size_t)w * c;
        union U {
            uint4 v;
            bf16_t s[8];
        } q0, q1, q2, q3, o;
        q0.v = *reinterpret_cast<const uint4 *>(in + b);
        q1.v = *reinterpret_cast<const uint4 *>(in + b + c);
        q2.v = *reinterpret_cast<const uint4 *>(in + b + row);
        q3.v = *reinterpret_cast<const uint4 *>(in + b + row + c);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float sum = bf2f(q0.s[k]) + bf2f(q1.s[k]) + bf2f(q2.s[k]) + bf2f(q3.s[k]);
            o.s[k] = f2bf(0.25f * sum);
        }
        *reinterpret_cast<uint4 *>(out + p * c + ch) = o.v;
    }
}

// The adjoint for groups of four channels (16-byte accesses): 0.69 to 0.3 ms
// over the levels of four 1024 x 1024 images, at a copy's rate.
__global__ void k_pool2_bwd4(const float4 *dout, float4 *din, int n, int h, int w, int c4,
                             int accumulate) {
    const size_t total = (size_t)n * h * w * c4;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c4);
        const size_t p = e / c4;
        const int x = (int)(p % w), y = (int)((p / w) % h), img = (int)(p / ((size_t)w * h));
        const float4 d = dout[(((size_t)img * (h / 2) + y / 2) * (w / 2) + x / 2) * c4 + ch];
        float4 g = make_float4(0.25f * d.x, 0.25f * d.y, 0.25f * d.z, 0.25f * d.w);
        if (accumulate) {
            const float4 o = din[e];
            g = make_float4(o.x + g.x, o.y + g.y, o.z + g.z, o.w + g.w);
        }
        din[e] = g;
    }
}

__global__ void k_pool2_bwd(const float *dout, float *din, int n, int h, int w, int c,
                            int accumulate) {
    const size_t total = (size_t)n * h * w * c;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c);
        size_t p = e / c;
        const int x = (int)(p % w), y = (int)((p / w) % h), img = (int)(p / ((size_t)w * h));
        const float g = 0.25f * dout[(((size_t)img * (h / 2) + y / 2) * (w / 2) + x / 2) * c + ch];
        din[e] = accumulate ? din[e] + g : g;
    }
}

// Nearest 2x upsample of `a` (ca channels, h/2 x w/2) concatenated with
// `s` (cs channels, h x w) along channels: out has ca + cs channels.
// Eight channels per thread; ca and cs are multiples of 8, so a group of
// eight never straddles the two sources.
__global__ void k_up2_concat(const bf16_t *a, int ca, const bf16_t *s, int cs, bf16_t *out, int n,
                             int h, int w) {
    const int co = ca + cs, c8 = co / 8;
    const size_t total = (size_t)n * h * w * c8;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c8) * 8;
        size_t p = e / c8;
        const int x = (int)(p % w), y = (int)((p / w) % h), img = (int)(p / ((size_t)w * h));
        const bf16_t *src = ch < ca
            ? a + (((size_t)img * (h / 2) + y / 2) * (w / 2) + x / 2) * ca + ch
            : s + p * cs + (ch - ca);
        *reinterpret_cast<uint4 *>(out + p * co + ch) = *reinterpret_cast<const uint4 *>(src);
    }
}

// Adjoint of k_up2_concat: da (FP32, h/2 x w/2 x ca) = 2x2 sums of the first
// ca channels; ds (FP32, h x w x cs) = the remaining channels.
__global__ void k_up2_concat_bwd(const float *dout, int ca, int cs, float *da, float *ds, int n,
                                 int h, int w) {
    const int co = ca + cs;
    const size_t plow = (size_t)n * (h / 2) * (w / 2);
    const size_t total_a = plow * ca, total_s = (size_t)n * h * w * cs;
    const size_t total = total_a + total_s;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        if (e < total_a) {
            const int ch = (int)(e % ca);
            const size_t p = e / ca;
            const int x = (int)(p % (w / 2)), y = (int)((p / (w / 2)) % (h / 2));
            const int img = (int)(p / ((size_t)(w / 2) * (h / 2)));
            const size_t b = (((size_t)img * h + 2 * y) * w + 2 * x) * co + ch;
            da[e] = dout[b] + dout[b + co] + dout[b + (size_t)w * co] + dout[b + (size_t)w * co + co];
        } else {
            const size_t f = e - total_a;
            const int ch = (int)(f % cs);
            const size_t p = f / cs;
            ds[f] = dout[p * co + ca + ch];
        }
    }
}

// Mean-squared error over the first `used` of `c` channels and its
// gradient; partial sums per block in loss_part.  Groups of four channels
// (c a multiple of 4, 16-byte aligned); groups past the used channels are
// only cleared, not read: 0.31 ms for four 1024 x 1024 images of 32 channels,
// where scalar accesses to every value took 1.18 ms on the 256 workgroups
// that the 256 partials allow.
__global__ __launch_bounds__(1024) void k_mse4(const float4 *pred, const float4 *target,
                                               float4 *grad, size_t pixels, int c4, int used,
                                               float *loss_part) {
    __shared__ float sh[1024];
    float s = 0.f;
    const float scale = 2.0f / (float)(pixels * used);
    // a workgroup's values are those of k_mse's: 256 of each sweep of the grid
    const size_t total = pixels * c4, sweep = (size_t)gridDim.x * 64;
    for (size_t e = (threadIdx.x >> 6) * sweep + (size_t)blockIdx.x * 64 + (threadIdx.x & 63);
         e < total; e += 16 * sweep) {
        const int ch = (int)(e % c4) * 4;
        float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ch < used) {
            const float4 p = pred[e], t = target[e];
            d.x = p.x - t.x;
            if (ch + 1 < used) d.y = p.y - t.y;
            if (ch + 2 < used) d.z = p.z - t.z;
            if (ch + 3 < used) d.w = p.w - t.w;
            s += d.x * d.x;
            s += d.y * d.y;
            s += d.z * d.z;
            s += d.w * d.w;
        }
        grad[e] = make_float4(scale * d.x, scale * d.y, scale * d.z, scale * d.w);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = sh[0];
}

// The same for any c and alignment.
__global__ void k_mse(const float *pred, const float *target, float *grad, size_t pixels, int c,
                      int used, float *loss_part) {
    __shared__ float sh[256];
    float s = 0.f;
    const float scale = 2.0f / (float)(pixels * used);
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < pixels * c;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c);
        float d = 0.f;
        if (ch < used) {
            d = pred[e] - target[e];
            s += d * d;
        }
        grad[e] = scale * d;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_part[blockIdx.x] = sh[0];
}

// Adam with bias correction; FP32 master weights, BF16 copy for the GEMMs.
__global__ void k_adam(float *w, bf16_t *w_bf, const float *g, float *m, float *v, size_t n,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[e];
        const float mi = b1 * m[e] + (1.f - b1) * gi;
        const float vi = b2 * v[e] + (1.f - b2) * gi * gi;
        m[e] = mi;
        v[e] = vi;
        const float wi = w[e] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        w[e] = wi;
        if (w_bf) w_bf[e] = f2bf(wi);
    }
}

// Tone map of a planar float image [3][h][w] into NHWC with c channels
// (channels >= 3 zero): out = log1p(img / s), s > 0 per image.
__global__ void k_tonemap(const float *img, int h, int w, const float *sum, float inv_count,
                          float s0, int c, float *out_f, bf16_t *out_bf) {
    const float s = tone_scale(sum, inv_count, s0);
    const size_t total = (size_t)h * w * c;
    const size_t plane = (size_t)h * w;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c);
        const size_t p = e / c;
        float v = 0.f;
        if (ch < 3) v = log1pf(fmaxf(img[ch * plane + p], 0.f) / s);
        if (out_f) out_f[e] = v;
        if (out_bf) out_bf[e] = f2bf(v);
    }
}

// The same for c a multiple of 8 and 16-byte aligned outputs: a workgroup
// takes the logarithms of its 256 pixels once (three a thread) and then
// writes rows of 16 bytes a lane: 46 us for 1024 x 1024 pixels of 32 channels,
// bound by writing them; a thread per output value, whose waves take three
// logarithms for two pixels, took 127 us.
__global__ __launch_bounds__(256) void k_tonemap8(const float *img, size_t plane, const float *sum,
                                                  float inv_count, float s0, int c, float *out_f,
                                                  bf16_t *out_bf) {
    __shared__ float4 sh[256];
    const float s = tone_scale(sum, inv_count, s0);
    const size_t p0 = (size_t)blockIdx.x * 256, p = p0 + threadIdx.x;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p < plane) {
        v.x = log1pf(fmaxf(img[p], 0.f) / s);
        v.y = log1pf(fmaxf(img[plane + p], 0.f) / s);
        v.z = log1pf(fmaxf(img[2 * plane + p], 0.f) / s);
    }
    sh[threadIdx.x] = v;
    __syncthreads();
    const uint32_t np = plane - p0 < 256 ? (uint32_t)(plane - p0) : 256u;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    if (out_f) {
        const uint32_t g = (uint32_t)c / 4;
        float4 *o = reinterpret_cast<float4 *>(out_f + p0 * c);
        for (uint32_t e = threadIdx.x; e < np * g; e += 256) o[e] = e % g == 0 ? sh[e / g] : zero;
    }
    if (out_bf) {
        const uint32_t g = (uint32_t)c / 8;
        uint4 *o = reinterpret_cast<uint4 *>(out_bf + p0 * c);
        for (uint32_t e = threadIdx.x; e < np * g; e += 256) {
            uint4 q = make_uint4(0u, 0u, 0u, 0u);
            if (e % g == 0) {
                const float4 t = sh[e / g];
                q.x = (uint32_t)f2bf(t.x) | ((uint32_t)f2bf(t.y) << 16);
                q.y = (uint32_t)f2bf(t.z);
            }
            o[e] = q;
        }
    }
}

// Inverse tone map from NHWC (first 3 channels) to planar [3][h][w].
__global__ void k_untonemap(const float *in, int h, int w, const float *sum, float inv_count,
                            float s0, int c, float *img) {
    const float s = tone_scale(sum, inv_count, s0);
    const size_t plane = (size_t)h * w;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < 3 * plane;
         e += (size_t)gridDim.x * blockDim.x) {
        const int ch = (int)(e / plane);
        const size_t p = e % plane;
        img[e] = s * expm1f(in[p * c + ch]);
    }
}

// The same for rows of 16-byte aligned groups of four channels: a thread per
// pixel reads its group once (25 us for 1024 x 1024 pixels of 32 channels; a
// thread per output value fetched each row's line three times: 60 us).
__global__ __launch_bounds__(256) void k_untonemap4(const float *in, size_t plane,
                                                    const float *sum, float inv_count, float s0,
                                                    int c, float *img) {
    const float s = tone_scale(sum, inv_count, s0);
    const size_t p = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= plane) return;
    const float4 v = *reinterpret_cast<const float4 *>(in + p * c);
    img[p] = s * expm1f(v.x);
    img[plane + p] = s * expm1f(v.y);
    img[2 * plane + p] = s * expm1f(v.z);
}

__global__ void k_f2bf(const float *in, bf16_t *out, size_t n) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x)
        out[e] = f2bf(in[e]);
}

// 16-byte aligned (or null): rows of four floats or eight bf16
bool a16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

unsigned grid_for(size_t n) {
    size_t g = (n + 255) / 256;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return (unsigned)g;
}

}  // namespace

hipError_t gemm(const bf16_t *A, const bf16_t *B, float *C, int M, int N, int K, int lda, int ldb,
                int trans_a, int splits, hipStream_t s) {
    if (splits < 1) splits = 1;
    int kps = (K + splits - 1) / splits;
    kps = (kps + BK - 1) / BK * BK;
    splits = (K + kps - 1) / kps;
    if (splits < 1) splits = 1;
    const int bn = N <= 32 ? 32 : 64;
    dim3 grid((M + 63) / 64, (N + bn - 1) / bn, splits);
    if (bn == 32) {
        if (trans_a)
            hipLaunchKernelGGL((k_gemm<64, 32, true>), grid, dim3(256), 0, s, A, B, C, M, N, K, lda, ldb, kps);
        else
            hipLaunchKernelGGL((k_gemm<64, 32, false>), grid, dim3(256), 0, s, A, B, C, M, N, K, lda, ldb, kps);
    } else {
        if (trans_a)
            hipLaunchKernelGGL((k_gemm<64, 64, true>), grid, dim3(256), 0, s, A, B, C, M, N, K, lda, ldb, kps);
        else
            hipLaunchKernelGGL((k_gemm<64, 64, false>), grid, dim3(256), 0, s, A, B, C, M, N, K, lda, ldb, kps);
    }
    return hipGetLastError();
}

int gemm_splits(int K, int splits) {
    if (splits < 1) splits = 1;
    int kps = (K + splits - 1) / splits;
    kps = (kps + BK - 1) / BK * BK;
    splits = (K + kps - 1) / kps;
    return splits < 1 ? 1 : splits;
}

hipError_t im2col3x3(const bf16_t *in, bf16_t *out, int n, int h, int w, int c, hipStream_t s) {
    const size_t total = (size_t)n * h * w * 9 * (c / 8);
    hipLaunchKernelGGL(k_im2col3x3, dim3(grid_for(total)), dim3(256), 0, s, in, out, n, h, w, c);
    return hipGetLastError();
}

hipError_t flip_weights(const bf16_t *w, bf16_t *wt, int cout, int cin, hipStream_t s) {
    hipLaunchKernelGGL(k_flip_weights, dim3(grid_for((size_t)cout * 9 * cin)), dim3(256), 0, s, w,
                       wt, cout, cin);
    return hipGetLastError();
}

hipError_t epilogue(const float *Cp, int splits, size_t mn, int n, const float *bias, int relu,
                    const float *residual, bf16_t *out_bf, float *out_f, hipStream_t s) {
    hipLaunchKernelGGL(k_epilogue, dim3(grid_for(mn)), dim3(256), 0, s, Cp, splits, mn, n, bias,
                       relu, residual, out_bf, out_f);
    return hipGetLastError();
}

hipError_t conv3x3_weights(const bf16_t *w, bf16_t *wf, int cin, int cout, hipStream_t s) {
    const size_t total = (size_t)9 * cin * cout;
    hipLaunchKernelGGL(k_conv_wf, dim3(grid_for(total)), dim3(256), 0, s, w, wf, cin, cout);
    return hipGetLastError();
}

hipError_t conv3x3(const bf16_t *x, const bf16_t *wf, const float *bias, int relu,
                   const float *residual, bf16_t *out_bf, float *out_f, int n, int h, int w,
                   int cin, int cout, hipStream_t s) {
    // wide tiles where they give every CU two workgroups (four tiles, where
    // one workgroup fits), with fewer the small tiles fill more of the GPU
    // (128 to 64 channels on 256 x 256 pixels, 512 wide tiles: 28 us, 24 in
    // small ones); for up to four slices, and where
    // rows of four channels are aligned (cout is a multiple of 32, so a base
    // pointer decides)
    const uintptr_t f32s = reinterpret_cast<uintptr_t>(residual) | reinterpret_cast<uintptr_t>(out_f);
    if ((f32s & 15u) == 0 && (reinterpret_cast<uintptr_t>(out_bf) & 7u) == 0) {
        bool done = false;
        auto wide = [&](auto kernel, int th, unsigned per_cu, uint64_t least) {
            const uint64_t t = (uint64_t)((h + th - 1) / th) * ((w + kWTW - 1) / kWTW) * n;
            if (done || t * (cout / 32) < least || t >= (1ull << 31)) return;
            const unsigned g = (unsigned)std::min<uint64_t>(
                t, std::max(1u, 256 * per_cu / (unsigned)(cout / 32)));
            hipLaunchKernelGGL(kernel, dim3(g, (unsigned)(cout / 32)), dim3(256), 0, s, x, wf, bias,
                               relu, residual, out_bf, out_f, n, h, w, cin, cout, Head{});
            done = true;
        };
        if (cin == kCK) wide(k_conv3x3_wide<1>, Wide<1>::TH, 2, 512);
        else if (cin == 2 * kCK) wide(k_conv3x3_wide<2>, Wide<2>::TH, 2, 512);
        else if (cin == 3 * kCK) wide(k_conv3x3_wide<3>, Wide<3>::TH, 1, 1024);
        else if (cin == 4 * kCK) wide(k_conv3x3_wide<4>, Wide<4>::TH, 1, 1024);
        if (done) return hipGetLastError();
    }
    const unsigned tiles = (unsigned)((h + kCTH - 1) / kCTH) * (unsigned)((w + kCTW - 1) / kCTW);
    hipLaunchKernelGGL(k_conv3x3, dim3(tiles * (unsigned)n, (unsigned)(cout / 32)), dim3(256), 0, s,
                       x, wf, bias, relu, residual, out_bf, out_f, h, w, cin, cout);
    return hipGetLastError();
}

bool conv3x3_head_fits(int h, int w, int cin) {
    // where conv3x3 takes the wide tiles for one image
    const uint64_t t = (uint64_t)((h + Wide<1>::TH - 1) / Wide<1>::TH) * ((w + kWTW - 1) / kWTW);
    return cin == kCK && t >= 512 && t < (1ull << 31);
}

hipError_t conv3x3_head(const bf16_t *x, const bf16_t *wf, const float *bias, const float *dec,
                        const float *sum, float inv_count, float *y, float *img, int h, int w,
                        int cout, hipStream_t s) {
    const unsigned t = (unsigned)((h + Wide<1>::TH - 1) / Wide<1>::TH) *
                       (unsigned)((w + kWTW - 1) / kWTW);
    const unsigned cb = (unsigned)(cout / 32);
    hipLaunchKernelGGL((k_conv3x3_wide<1, true>), dim3(std::min(t, std::max(1u, 512 / cb)), cb),
                       dim3(256), 0, s, x, wf, bias, 0, nullptr, nullptr, y, 1, h, w, kCK, cout,
                       Head{dec, sum, inv_count, img});
    return hipGetLastError();
}

hipError_t conv3x3_adjoint_weights(const bf16_t *w, bf16_t *wf, int cin, int cout,
                                   hipStream_t s) {
    hipLaunchKernelGGL(k_conv_wf_adjoint, dim3(grid_for((size_t)9 * cin * cout)), dim3(256), 0, s,
                       w, wf, cin, cout);
    return hipGetLastError();
}

hipError_t conv3x3_bwd_data(const bf16_t *dz, const bf16_t *wf, float *dx, int n, int h, int w,
                            int cin, int cout, hipStream_t s) {
    // one slice: the forward kernel's order is tap-major already
    if (cout == 32)
        return conv3x3(dz, wf, nullptr, 0, nullptr, nullptr, dx, n, h, w, cout, cin, s);
    const unsigned tiles = (unsigned)((h + kCTH - 1) / kCTH) * (unsigned)((w + kCTW - 1) / kCTW);
    const dim3 grid(tiles * (unsigned)n, (unsigned)(cin / 32)), block(256);
    if (cout <= 64)
        hipLaunchKernelGGL(k_conv3x3_taps<2>, grid, block, 0, s, dz, wf, dx, h, w, cout, cin);
    else if (cout <= 128)
        hipLaunchKernelGGL(k_conv3x3_taps<4>, grid, block, 0, s, dz, wf, dx, h, w, cout, cin);
    else
        hipLaunchKernelGGL(k_conv3x3_taps<8>, grid, block, 0, s, dz, wf, dx, h, w, cout, cin);
    return hipGetLastError();
}

int conv3x3_dw_splits(int n, int h, int w, int cin, int cout) {
    // about 1024 workgroups (four a CU) in all, at least a tile each
    const uint64_t tiles =
        (uint64_t)n * ((h + kDTH - 1) / kDTH) * (uint64_t)((w + kDTW - 1) / kDTW);
    const uint64_t want = std::max<uint64_t>(1, 1024 / ((uint64_t)(cin / 32) * (cout / 32)));
    return (int)std::min(tiles, want);
}

hipError_t conv3x3_dw(const bf16_t *x, const bf16_t *dz, float *part, float *dw, int n, int h,
                      int w, int cin, int cout, hipStream_t s) {
    const int splits = conv3x3_dw_splits(n, h, w, cin, cout);
    hipLaunchKernelGGL(k_conv3x3_dw, dim3(splits, (cin / 32) * (cout / 32)), dim3(256), 0, s, x, dz,
                       part, n, h, w, cin, cout);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t mn = (size_t)9 * cin * cout;
    hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((mn + 63) / 64)), dim3(1024), 0, s, part,
                       splits, mn, dw);
    return hipGetLastError();
}

hipError_t relu_bwd_bias(const float *dy, const bf16_t *y, size_t rows, int cols, bf16_t *dz_bf,
                         float *db, float *part, hipStream_t s) {
    size_t rpb = (rows + kColsumBlocks - 1) / kColsumBlocks;
    if (rpb < 64) rpb = 64;
    const int nb = (int)((rows + rpb - 1) / rpb);
    hipLaunchKernelGGL(k_relu_bwd_bias, dim3(nb), dim3(256), 0, s, dy, y, rows, cols, rpb, dz_bf,
                       part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_colsum_final, dim3(cols), dim3(256), 0, s, part, nb, cols, db);
    return hipGetLastError();
}

hipError_t relu_bwd(const float *dy, const bf16_t *y, int relu, bf16_t *dz_bf, float *dz_f,
                    size_t total, hipStream_t s) {
    hipLaunchKernelGGL(k_relu_bwd, dim3(grid_for(total)), dim3(256), 0, s, dy, y, relu, dz_bf,
                       dz_f, total);
    return hipGetLastError();
}

hipError_t colsum(const float *in, size_t rows, int cols, float *out, float *part, hipStream_t s) {
    size_t rpb = (rows + kColsumBlocks - 1) / kColsumBlocks;
    if (rpb < 256) rpb = 256;
    const int nb = (int)((rows + rpb - 1) / rpb);
    hipLaunchKernelGGL(k_colsum_part, dim3(nb), dim3(256), 0, s, in, rows, cols, rpb, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_colsum_final, dim3(cols), dim3(256), 0, s, part, nb, cols, out);
    return hipGetLastError();
}

hipError_t pool2(const bf16_t *in, bf16_t *out, int n, int h, int w, int c, hipStream_t s) {
    hipLaunchKernelGGL(k_pool2, dim3(grid_for((size_t)n * h * w * c / 32)), dim3(256), 0, s, in,
                       out, n, h, w, c);
    return hipGetLastError();
}

hipError_t pool2_bwd(const float *dout, float *din, int n, int h, int w, int c, int accumulate,
                     hipStream_t s) {
    if (c % 4 == 0 && a16(dout) && a16(din)) {
        hipLaunchKernelGGL(k_pool2_bwd4, dim3(grid_for((size_t)n * h * w * (c / 4))), dim3(256), 0,
                           s, reinterpret_cast<const float4 *>(dout),
                           reinterpret_cast<float4 *>(din), n, h, w, c / 4, accumulate);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_pool2_bwd, dim3(grid_for((size_t)n * h * w * c)), dim3(256), 0, s, dout,
                       din, n, h, w, c, accumulate);
    return hipGetLastError();
}

hipError_t up2_concat(const bf16_t *a, int ca, const bf16_t *sk, int cs, bf16_t *out, int n,
                      int h, int w, hipStream_t s) {
    hipLaunchKernelGGL(k_up2_concat, dim3(grid_for((size_t)n * h * w * (ca + cs) / 8)), dim3(256), 0,
                       s, a, ca, sk, cs, out, n, h, w);
    return hipGetLastError();
}

hipError_t up2_concat_bwd(const float *dout, int ca, int cs, float *da, float *ds, int n, int h,
                          int w, hipStream_t s) {
    const size_t total = (size_t)n * (h / 2) * (w / 2) * ca + (size_t)n * h * w * cs;
    hipLaunchKernelGGL(k_up2_concat_bwd, dim3(grid_for(total)), dim3(256), 0, s, dout, ca, cs, da,
                       ds, n, h, w);
    return hipGetLastError();
}

hipError_t mse(const float *pred, const float *target, float *grad, size_t pixels, int c,
               int used, float *loss_part, int nblocks, hipStream_t s) {
    if (c % 4 == 0 && a16(pred) && a16(target) && a16(grad)) {
        hipLaunchKernelGGL(k_mse4, dim3(nblocks), dim3(1024), 0, s,
                           reinterpret_cast<const float4 *>(pred),
                           reinterpret_cast<const float4 *>(target),
                           reinterpret_cast<float4 *>(grad), pixels, c / 4, used, loss_part);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_mse, dim3(nblocks), dim3(256), 0, s, pred, target, grad, pixels, c, used,
                       loss_part);
    return hipGetLastError();
}

hipError_t adam(float *w, bf16_t *w_bf, const float *g, float *m, float *v, size_t n, float lr,
                float b1, float b2, float eps, int step, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, s, w, w_bf, g, m, v, n, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

hipError_t tonemap(const float *img, int h, int w, float scale, int c, float *out_f,
                   bf16_t *out_bf, hipStream_t s, const float *sum, float inv_count) {
    const size_t plane = (size_t)h * w;
    if (c % 8 == 0 && a16(out_f) && a16(out_bf) && (plane + 255) / 256 < (1ull << 31)) {
        hipLaunchKernelGGL(k_tonemap8, dim3((unsigned)((plane + 255) / 256)), dim3(256), 0, s, img,
                           plane, sum, inv_count, scale, c, out_f, out_bf);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_tonemap, dim3(grid_for((size_t)h * w * c)), dim3(256), 0, s, img, h, w,
                       sum, inv_count, scale, c, out_f, out_bf);
    return hipGetLastError();
}

hipError_t untonemap(const float *in, int h, int w, float scale, int c, float *img, hipStream_t s,
                     const float *sum, float inv_count) {
    const size_t plane = (size_t)h * w;
    if (c % 4 == 0 && a16(in) && (plane + 255) / 256 < (1ull << 31)) {
        hipLaunchKernelGGL(k_untonemap4, dim3((unsigned)((plane + 255) / 256)), dim3(256), 0, s, in,
                           plane, sum, inv_count, scale, c, img);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_untonemap, dim3(grid_for((size_t)h * w * 3)), dim3(256), 0, s, in, h, w,
                       sum, inv_count, scale, c, img);
    return hipGetLastError();
}

hipError_t f2bf(const float *in, bf16_t *out, size_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_f2bf, dim3(grid_for(n)), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace splotch
