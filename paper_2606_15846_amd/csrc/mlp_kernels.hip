// Kernels of the small bfloat16 perceptrons (the learned reset proposal's
// network): a tiled GEMM on the gfx950 matrix cores with a fused
// bias/activation epilogue, the activation backward, column sums, the squared
// error loss and AdamW.  Accumulation is always float.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "mlp_internal.hpp"
#include "philox.hpp"

namespace navsim {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBM = 64, kBN = 64, kBK = 32;
constexpr int kLdsK = kBK + 8;  // padded row (80 bytes) of a staged tile
constexpr int kGemmThreads = 256;
constexpr int kColChunk = 32;  // rows per partial column sum
constexpr int kColWidth = 32;  // columns per workgroup of a column sum

__device__ __forceinline__ uint16_t to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);                    // round to nearest even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float from_bf16_bits(uint16_t b) {
    return __uint_as_float((uint32_t)b << 16);
}

// Stage rows [r0, r0 + 64) x k [k0, k0 + 32) of a matrix whose element (r, k)
// is X[r ld + k] (kmajor) or X[k ld + r], as T[r][k] in LDS; zeros outside
// [0, R) x [0, K).
template <bool KMAJOR>
__device__ __forceinline__ void stage_tile(uint16_t (*T)[kLdsK], const uint16_t *X, int64_t ld,
                                           int R, int K, int r0, int k0, bool vec_ok, int tid) {
    if (KMAJOR) {
        const int r = tid >> 2, kk = (tid & 3) * 8;
        const int gr = r0 + r, gk = k0 + kk;
        uint16_t v[8];
        if (vec_ok && gr < R && gk + 8 <= K) {
            const uint4 q = *reinterpret_cast<const uint4 *>(X + (int64_t)gr * ld + gk);
            *reinterpret_cast<uint4 *>(&T[r][kk]) = q;
            return;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = (gr < R && gk + j < K) ? X[(int64_t)gr * ld + gk + j] : (uint16_t)0;
#pragma unroll
        for (int j = 0; j < 8; ++j) T[r][kk + j] = v[j];
    } else {
        const int kr = tid >> 3, rr = (tid & 7) * 8;
        const int gk = k0 + kr, gr = r0 + rr;
        uint16_t v[8];
        if (vec_ok && gk < K && gr + 8 <= R) {
            const uint4 q = *reinterpret_cast<const uint4 *>(X + (int64_t)gk * ld + gr);
            const uint16_t *w = reinterpret_cast<const uint16_t *>(&q);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = w[j];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] = (gk < K && gr + j < R) ? X[(int64_t)gk * ld + gr + j] : (uint16_t)0;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) T[rr + j][kr] = v[j];
    }
}

// Bias, activation (or the derivative of one), stores of element (m, n).
__device__ __forceinline__ void gemm_store(const GemmArgs &g, int m, int n, float v) {
    if (g.bias) v += g.bias[n];
    if (g.bias_rows) v += g.bias_rows[(int64_t)g.row_idx[m] * g.ldbr + n];
    if (g.act == 1 && !(v > 0.0f)) v *= g.slope;
    if (g.act == 2) v = tanhf(v);
    if (g.act == 3 && !(from_bf16_bits(g.H[(int64_t)m * g.ldh + n]) > 0.0f)) v *= g.slope;
    if (g.Cf) g.Cf[(int64_t)m * g.ldcf + n] = v;
    if (g.Cb) g.Cb[(int64_t)m * g.ldcb + n] = to_bf16_bits(v);
}

// One workgroup computes a 64 x 64 block of C; each of its four wavefronts a
// 32 x 32 quarter as 2 x 2 tiles of the 16 x 16 x 32 bfloat16 MFMA.
// Fragment layout of v_mfma_f32_16x16x32_bf16: lane l supplies row l % 16 of
// A and column l % 16 of B, k = 8 (l / 16) .. 8 (l / 16) + 7; it receives
// C[4 (l / 16) + r][l % 16], r = 0..3.
template <bool BK>
__global__ __launch_bounds__(kGemmThreads) void gemm_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) uint16_t As[kBM][kLdsK];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[kBN][kLdsK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * kBM, n0 = blockIdx.x * kBN;
    int M = g.M;
    if (g.m_dev) {
        // rows known only on the device: the grid covers g.M, the rest exits
        const int64_t md = (int64_t)*g.m_dev * g.m_mul;
        M = md < (int64_t)M ? (int)(md > 0 ? md : 0) : M;
        if (m0 >= M) return;
    }
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const bool a_vec = (g.lda % 8 == 0) && (((uintptr_t)g.A & 15) == 0);
    const bool b_vec = (g.ldb % 8 == 0) && (((uintptr_t)g.B & 15) == 0);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    for (int k0 = 0; k0 < g.K; k0 += kBK) {
        stage_tile<true>(As, g.A, g.lda, M, g.K, m0, k0, a_vec, tid);
        stage_tile<BK>(Bs, g.B, g.ldb, g.N, g.K, n0, k0, b_vec, tid);
        __syncthreads();
        bf16x8 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = *reinterpret_cast<const bf16x8 *>(&As[wm + 16 * i + fr][fk]);
            b[i] = *reinterpret_cast<const bf16x8 *>(&Bs[wn + 16 * i + fr][fk]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn + 16 * j + fr;
            if (n >= g.N) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + (lane >> 4) * 4 + r;
                if (m >= M) continue;
                gemm_store(g, m, n, acc[i][j][r]);
            }
        }
}

// The same product where the 64 x 64 blocks leave most of the chip idle (a
// training batch: 16 to 68 of them, each a chain of ceil(K / 32) trips to memory
// and back, about a microsecond a trip): a 32 x 32 block per workgroup, one
// 16 x 16 tile per wavefront, and 128 k's a trip, the loads of the next trips in
// flight.  A transposed operand is turned in
// registers, 4 k's by 8 rows per thread, on its way to LDS.  Same tiles and k
// order, so bitwise the same sums.  A batch of 1,024 on the 1048-256-256-256-5
// network, us a product: first layer 38 -> 13, hidden layers 9 -> 5.6, weight
// gradients 32 -> 13, the table of 512 (map, bin) rows 38 -> 13.  Bound by the
// trips to memory that are left and by the launches (about 5 us each).
constexpr int kSB = 32, kSK = 128;
constexpr int kSAhead = 2;  // trips in flight (even: they alternate between two LDS buffers)
constexpr int kSLds = kSK + 8;

// A thread's share of a 32 x 128 tile (element (r, k) as in stage_tile), t < 128:
// four 16-byte pieces, 8 k's of rows t / 16 + 8 p or 8 rows of k's 4 (t / 4) + p.
template <bool KMAJOR>
__device__ __forceinline__ void small_load(uint4 q[4], const uint16_t *X, int64_t ld, int R, int K,
                                           int r0, int k0, bool whole, int t) {
    // No load stands behind a branch (the compiler waits for each of those where
    // the paths join): addresses outside are clamped, and what they give is cleared
    // in small_store, where it is needed first.  `whole`: 16-byte pieces are
    // aligned and lie inside or outside as a whole; otherwise element by element.
    if (whole) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = r0 + (KMAJOR ? (t >> 4) + 8 * p : (t & 3) * 8);
            const int k = k0 + (KMAJOR ? (t & 15) * 8 : (t >> 2) * 4 + p);
            q[p] = *reinterpret_cast<const uint4 *>(
                X + (r < R && k < K ? (KMAJOR ? (int64_t)r * ld + k : (int64_t)k * ld + r) : 0));
        }
        return;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = r0 + (KMAJOR ? (t >> 4) + 8 * p : (t & 3) * 8);
        const int k = k0 + (KMAJOR ? (t & 15) * 8 : (t >> 2) * 4 + p);
        uint16_t v[8];
        bool in[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int rj = KMAJOR ? r : r + j, kj = KMAJOR ? k + j : k;
            in[j] = rj < R && kj < K;
            v[j] = X[!in[j] ? 0 : KMAJOR ? (int64_t)rj * ld + kj : (int64_t)kj * ld + rj];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = in[j] ? v[j] : (uint16_t)0;
        __builtin_memcpy(&q[p], v, 16);
    }
}

template <bool KMAJOR>
__device__ __forceinline__ void small_store(uint16_t (*T)[kSLds], uint4 q[4], int R, int K, int r0,
                                            int k0, bool whole, int t) {
    if (whole) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = r0 + (KMAJOR ? (t >> 4) + 8 * p : (t & 3) * 8);
            const int k = k0 + (KMAJOR ? (t & 15) * 8 : (t >> 2) * 4 + p);
            if (!(r < R && k < K)) q[p] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    if (KMAJOR) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
            *reinterpret_cast<uint4 *>(&T[(t >> 4) + 8 * p][(t & 15) * 8]) = q[p];
    } else {
        const uint32_t *w[4] = {&q[0].x, &q[1].x, &q[2].x, &q[3].x};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // element j of the four pieces: the low or high half of dword j / 2
            const uint32_t sel = j & 1 ? 0x07060302u : 0x05040100u;
            *reinterpret_cast<uint2 *>(&T[(t & 3) * 8 + j][(t >> 2) * 4]) =
                make_uint2(__builtin_amdgcn_perm(w[1][j >> 1], w[0][j >> 1], sel),
                           __builtin_amdgcn_perm(w[3][j >> 1], w[2][j >> 1], sel));
        }
    }
}

template <bool AK, bool BK>
__device__ __forceinline__ void gemm_small_block(const GemmArgs &g, int bm, int bn) {
    __shared__ __attribute__((aligned(16))) uint16_t T[2][2][kSB][kSLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = bm * kSB, n0 = bn * kSB;
    int M = g.M;
    if (g.m_dev) {
        const int64_t md = (int64_t)*g.m_dev * g.m_mul;
        M = md < (int64_t)M ? (int)(md > 0 ? md : 0) : M;
        if (m0 >= M) return;
    }
    const bool a_vec = g.lda % 8 == 0 && ((uintptr_t)g.A & 15) == 0 && (AK ? g.K : M) % 8 == 0;
    const bool b_vec = g.ldb % 8 == 0 && ((uintptr_t)g.B & 15) == 0 && (BK ? g.K : g.N) % 8 == 0;
    const bool is_a = wave < 2;  // two wavefronts load A, two load B
    const int t = tid & 127;
    uint4 q[kSAhead][4];
    auto load = [&](uint4(&d)[4], int k0) {
        if (k0 >= g.K) return;
        if (is_a)
            small_load<AK>(d, g.A, g.lda, M, g.K, m0, k0, a_vec, t);
        else
            small_load<BK>(d, g.B, g.ldb, g.N, g.K, n0, k0, b_vec, t);
    };
    const int wm = (wave >> 1) * 16, wn = (wave & 1) * 16;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < kSAhead; ++i) load(q[i], i * kSK);
    for (int kg = 0; kg < g.K; kg += kSAhead * kSK) {
#pragma unroll
        for (int i = 0; i < kSAhead; ++i) {
            const int k0 = kg + i * kSK;
            if (k0 >= g.K) break;
            if (is_a)
                small_store<AK>(T[i & 1][0], q[i], M, g.K, m0, k0, a_vec, t);
            else
                small_store<BK>(T[i & 1][1], q[i], g.N, g.K, n0, k0, b_vec, t);
            __syncthreads();  // the other buffer's readers are past their reads
            load(q[i], k0 + kSAhead * kSK);
#pragma unroll
            for (int kb = 0; kb < kSK / 32; ++kb) {
                if (k0 + 32 * kb >= g.K) break;
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&T[i & 1][0][wm + fr][32 * kb + fk]);
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&T[i & 1][1][wn + fr][32 * kb + fk]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
            }
        }
    }
    const int n = n0 + wn + fr;
    if (n >= g.N) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + (lane >> 4) * 4 + r;
        if (m < M) gemm_store(g, m, n, acc[r]);
    }
}

// At the start of a page, as forward_noise_kernel is (27 KB of code; 16 training
// steps 2,743 us at another offset, 2,727 here).
template <bool BK>
__global__ __launch_bounds__(256) __attribute__((aligned(4096)))
void gemm_small_kernel(GemmArgs g) {
    gemm_small_block<true, BK>(g, (int)blockIdx.y, (int)blockIdx.x);
}

// out[n] = sum over m of X[m, n] for 32 columns: chunks of 32 rows in order, 8
// chunks at a time, then the chunk sums in order.
__device__ __forceinline__ void col_sum_block(const ColSum &c, int block) {
    __shared__ float s_part[256 / kColWidth][kColWidth];
    const int col = threadIdx.x % kColWidth, lane = threadIdx.x / kColWidth;
    const int n = block * kColWidth + col;
    const int chunks = (c.M + kColChunk - 1) / kColChunk;
    float total = 0.0f;
    for (int b = 0; b < chunks; b += 256 / kColWidth) {
        // all of a chunk's loads go out together, rows past M as zeros (which
        // leave a sum that starts at +0 as it is)
        const int m0 = (b + lane) * kColChunk;
        float v[kColChunk];
#pragma unroll
        for (int q = 0; q < kColChunk; ++q)
            v[q] = c.X[(int64_t)min(m0 + q, c.M - 1) * c.N + min(n, c.N - 1)];
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < kColChunk; ++q) s += m0 + q < c.M ? v[q] : 0.0f;
        s_part[lane][col] = s;
        __syncthreads();
        if (lane == 0)
            for (int q = 0; q < 256 / kColWidth && b + q < chunks; ++q) total += s_part[q][col];
        __syncthreads();
    }
    if (lane == 0 && n < c.N) c.out[n] = total;
}

// Every weight and bias gradient of a network in one launch: dW = dz^T Hin tiles
// of each layer, then the column sums.  They only wait for the layers' dz, and
// each alone leaves most of the chip idle: a batch of 1,024 on the 1048-256-256-
// 256-5 network took 4 x 13 us for the products and 4 x 13 us for the sums (two
// launches each), together 20 us.
__global__ __launch_bounds__(256) __attribute__((aligned(4096)))
void gradient_kernel(GradientArgs a) {
    int b = (int)blockIdx.x;
    for (int l = 0; l < a.gemms; ++l) {
        const GemmArgs &g = a.gemm[l];
        const int nbn = (g.N + kSB - 1) / kSB, nb = nbn * ((g.M + kSB - 1) / kSB);
        if (b < nb) {
            gemm_small_block<false, false>(g, b / nbn, b % nbn);
            return;
        }
        b -= nb;
    }
    for (int l = 0; l < a.sums; ++l) {
        const int nb = (a.sum[l].N + kColWidth - 1) / kColWidth;
        if (b < nb) {
            col_sum_block(a.sum[l], b);
            return;
        }
        b -= nb;
    }
}

__global__ void sq_loss_kernel(int M, int D, const float *Y, const float *T, const float *w,
                               float *L, float *dYf, uint16_t *dYb) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    float l = 0.0f;
    for (int d = 0; d < D; ++d) {
        const float e = Y[(int64_t)m * D + d] - T[(int64_t)m * D + d];
        l += w[d] * (e * e);
        const float gd = (2.0f * w[d] * e) / (float)M;
        if (dYf) dYf[(int64_t)m * D + d] = gd;
        if (dYb) dYb[(int64_t)m * D + d] = to_bf16_bits(gd);
    }
    if (L) L[m] = l;
}

// Parameter i (bf16 bits v) into the packed image of the weights that
// forward_noise_kernel reads: fragments of 16 output rows by 32 inputs, the 16
// bytes of each lane of a wavefront's load in lane order, so that a load is one
// contiguous kilobyte.  Read from the row-major weights a fragment's 16 lanes
// per row group lie 512 bytes apart, 64 cache lookups a load instead of 8.
__device__ __forceinline__ void store_packed(const PackedNet &f, int64_t i, uint16_t v) {
    const int H = f.hidden;
    int64_t base = 0;
    for (int l = 0; l < f.layers; ++l) {
        const int ni = l == 0 ? f.d0 : H, no = l + 1 < f.layers ? H : 5;
        const int q = (int)(i - f.w_off[l]);
        const int ks = l == 0 ? 2 : H / 32;  // k blocks (layer 0: the noise columns, up to 64)
        if (i >= f.w_off[l] && q < ni * no) {
            const int n = q / ni, k = q - n * ni - (l == 0 ? f.col0 : 0);
            if (k >= 0)
                f.image[base + (((n >> 4) * ks + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (n & 15)) * 8 +
                        (k & 7)] = v;
            return;
        }
        base += (int64_t)((no + 15) / 16) * ks * 512;
    }
}

__global__ void adamw_kernel(int64_t n, float *p, uint16_t *pb, const float *g, float *m, float *v,
                             const uint8_t *decay_mask, float lr, float b1, float b2, float eps,
                             float wd, float bc1, float bc2, PackedNet f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * (gi * gi);
    m[i] = mi;
    v[i] = vi;
    float pi = p[i];
    if (!decay_mask || decay_mask[i]) pi = pi * (1.0f - lr * wd);
    pi = pi - lr * ((mi / bc1) / (sqrtf(vi / bc2) + eps));
    p[i] = pi;
    if (pb) pb[i] = to_bf16_bits(pi);
    if (f.image) store_packed(f, i, to_bf16_bits(pi));
}

__global__ void to_bf16_kernel(int64_t n, const float *x, uint16_t *y, PackedNet f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    y[i] = to_bf16_bits(x[i]);
    if (f.image) store_packed(f, i, to_bf16_bits(x[i]));
}

// Actor input: x[e][j] = bf16(1 / (obs[e][j] - beta)) for the m pooled
// ranges (the reciprocal transform), bf16(obs[e][j]) for the 4 goal and
// velocity features.
__global__ void actor_input_kernel(int N, int m, const float *obs, const float *beta,
                                   uint16_t *x) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int row = m + 4;
    if (i >= (int64_t)N * row) return;
    const int j = (int)(i % row);
    const float v = obs[i];
    x[i] = to_bf16_bits(j < m ? 1.0f / (v - *beta) : v);
}

// Exploration noise: a = clip(a + std n, -1, 1) with n standard normal from
// Box-Muller on Philox(e, n mod 2^32, n div 2^32, 11) words 0 and 1 at step
// n = *step_ctr + step_off (double precision, rounded to float).
__global__ void actor_noise_kernel(int N, float *act, float std, const uint32_t *step_ctr,
                                   int step_off, uint32_t key0, uint32_t key1) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= N) return;
    const uint64_t n = (((uint64_t)step_ctr[1] << 32) | (uint64_t)step_ctr[0]) + (uint64_t)step_off;
    uint32_t c[4] = {(uint32_t)e, (uint32_t)n, (uint32_t)(n >> 32), 11u};
    philox4x32_10(c, key0, key1);
    const double u1 = ((double)c[0] + 0.5) / 4294967296.0, u2 = ((double)c[1] + 0.5) / 4294967296.0;
    const double r = sqrt(-2.0 * log(u1)), t = 2.0 * 3.14159265358979323846 * u2;
    const float n0 = (float)(r * cos(t)), n1 = (float)(r * sin(t));
    float a0 = act[2 * e] + std * n0, a1 = act[2 * e + 1] + std * n1;
    act[2 * e] = fminf(1.0f, fmaxf(-1.0f, a0));
    act[2 * e + 1] = fminf(1.0f, fmaxf(-1.0f, a1));
}

// Whole actor in one launch: a workgroup of 4 wavefronts takes 16 observation
// rows, builds their bf16 inputs in LDS (reciprocal range transform), then
// runs every layer as 16 x 16 x 32 bf16 MFMA tiles, wavefront w taking the
// layer's 16-column blocks w, w + 4, ..., with the weights staged in LDS by
// the workgroup from a padded bf16 image (k-contiguous rows, K padded to 32,
// N to 16, zeros outside), and writes bias + activation to the next layer's
// input rows.  The last layer applies tanh; then one lane per row draws the
// row's exploration noise pair (one Box-Muller transform), adds, clips and
// stores both action components.  Same tiles, k order and rounding points as
// the layer-by-layer GEMM path.
// Threads of the one-launch actor: 8 wavefronts, one 16-column block of a
// layer (<= 128 wide) each, so that a wavefront's serial chain per layer is
// one block's products and epilogue.
constexpr int kActorThreads = 512;
constexpr int kActorWaves = kActorThreads / 64;
constexpr int kActorBlocks = 8 / kActorWaves;  // column blocks per wavefront
constexpr int kActorPasses = 2048 / kActorThreads;  // 16 rows x 128 columns per pass set

__global__ __launch_bounds__(kActorThreads) void actor_fused_kernel(ActorArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint16_t act_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = blockIdx.x * 16;
    const int ld = a.kmax + 8;  // LDS row pitch (bf16): 16 B past a bank cycle
    uint16_t *cur_in = act_lds;        // this layer's input rows [16][ld]
    uint16_t *nxt_in = act_lds + 16 * ld;  // the next layer's
    uint16_t *wl = act_lds + 32 * ld;  // this layer's weights
    float *s_act = reinterpret_cast<float *>(wl + a.wmax);  // [16][2] actions before noise
    const int row = a.m + 4;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    // A layer's weights and biases go to registers one layer ahead: layer
    // l + 1's loads are in flight while layer l runs on the matrix cores.
    // Weights: np kp / 8 <= 128 * 128 / 8 = 2048 vectors, kActorPasses per
    // thread; rows of kp bf16 stored with pitch kp + 8 (conflict-free fragment
    // reads); thread t copies 16-byte column t % 16 of rows t / 16 + (T / 16) i.
    const int wc = threadIdx.x & 15, wr0 = threadIdx.x >> 4;
    constexpr int kRowStep = kActorThreads / 16;
    uint4 t8[kActorPasses];
    float bias[kActorBlocks];
    auto load_layer = [&](int l) {
        const uint4 *src = reinterpret_cast<const uint4 *>(a.w + a.w_off[l]);
        const int rv = a.kpad[l] / 8, np = a.npad[l];
#pragma unroll
        for (int t = 0; t < kActorPasses; ++t) {
            const int rw = wr0 + kRowStep * t;
            t8[t] = (wc < rv && rw < np) ? src[rw * rv + wc] : make_uint4(0u, 0u, 0u, 0u);
        }
        // this lane's biases, for its wavefront's column blocks (np <= 128)
#pragma unroll
        for (int t = 0; t < kActorBlocks; ++t) {
            const int n0 = 16 * (wave + kActorWaves * t);
            bias[t] = n0 < np ? a.b[a.b_off[l] + n0 + fr] : 0.0f;
        }
    };
    load_layer(0);
    // inputs: 16 rows x kpad[0] (<= 128) columns, kActorPasses per thread, loads first
    {
        const int kp0 = a.kpad[0];
        const float beta = *a.beta;
        float v[kActorPasses];
        // every load in bounds (clamped row and column, N >= 1) and issued
        // back to back; out-of-range entries are then replaced by 0
#pragma unroll
        for (int t = 0; t < kActorPasses; ++t) {
            const int q = threadIdx.x + kActorThreads * t, r = q >> 7, j = q & 127, e = row0 + r;
            v[t] = a.obs[(int64_t)min(e, a.N - 1) * row + min(j, row - 1)];
        }
#pragma unroll
        for (int t = 0; t < kActorPasses; ++t) {
            const int q = threadIdx.x + kActorThreads * t, r = q >> 7, j = q & 127, e = row0 + r;
            if (!(e < a.N && j < row)) v[t] = 0.0f;
        }
#pragma unroll
        for (int t = 0; t < kActorPasses; ++t) {
            const int q = threadIdx.x + kActorThreads * t, r = q >> 7, j = q & 127;
            if (j < kp0)
                cur_in[r * ld + j] =
                    to_bf16_bits(j < a.m && row0 + r < a.N ? 1.0f / (v[t] - beta) : v[t]);
        }
    }
    for (int l = 0; l < a.layers; ++l) {
        const int kp = a.kpad[l], np = a.npad[l];
        {
            uint4 *dst = reinterpret_cast<uint4 *>(wl);
            const int rv = kp / 8;
#pragma unroll
            for (int t = 0; t < kActorPasses; ++t) {
                const int rw = wr0 + kRowStep * t;
                if (wc < rv && rw < np) dst[rw * (rv + 1) + wc] = t8[t];
            }
        }
        float bias_l[kActorBlocks];
#pragma unroll
        for (int t = 0; t < kActorBlocks; ++t) bias_l[t] = bias[t];
        __syncthreads();  // inputs and weights in LDS
        if (l + 1 < a.layers) load_layer(l + 1);
        const uint16_t *W = wl;
        const bool last = l + 1 == a.layers;
        // Every fragment is read before the first product, from positions
        // clamped into this layer's K and N (always in bounds), so the reads
        // share one LDS round trip; products past K are then skipped.
        const int nkb = kp / 32;  // 1..4
        bf16x8 av[4];             // the rows' input fragments, shared by every column block
        bf16x8 bv[kActorBlocks][4];  // this wavefront's column blocks
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
            av[kb] = *reinterpret_cast<const bf16x8 *>(&cur_in[fr * ld + 32 * min(kb, nkb - 1) + fk]);
#pragma unroll
        for (int t = 0; t < kActorBlocks; ++t) {
            const int n0 = min(16 * (wave + kActorWaves * t), np - 16);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                bv[t][kb] = *reinterpret_cast<const bf16x8 *>(W + (n0 + fr) * (kp + 8) +
                                                              32 * min(kb, nkb - 1) + fk);
        }
#pragma unroll
        for (int t = 0; t < kActorBlocks; ++t) {
            const int n0 = 16 * (wave + kActorWaves * t);
            if (n0 >= np) break;
            f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                if (kb < nkb) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[kb], bv[t][kb], acc, 0, 0, 0);
            const int n = n0 + fr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int rr = (lane >> 4) * 4 + r;
                float v = acc[r] + bias_l[t];
                if (!last) {
                    if (!(v > 0.0f)) v *= a.slope;
                    nxt_in[rr * ld + n] = to_bf16_bits(v);
                } else if (n < 2) {
                    s_act[rr * 2 + n] = tanhf(v);
                }
            }
        }
        if (!last) {
            // zero the padding columns [np, kpad[l + 1]) of the next input
            const int kn = a.kpad[l + 1], wpad = kn - np;
            for (int q = threadIdx.x; q < 16 * wpad; q += kActorThreads) {
                const int r = q / wpad;
                nxt_in[r * ld + np + (q - r * wpad)] = 0;
            }
            uint16_t *t = cur_in;
            cur_in = nxt_in;
            nxt_in = t;
        }
        __syncthreads();  // next layer's inputs written, this layer's weights no longer read
    }
    // noise, clip and store: one lane per row
    if (threadIdx.x < 16) {
        const int e = row0 + threadIdx.x;
        if (e < a.N) {
            float v0 = s_act[threadIdx.x * 2], v1 = s_act[threadIdx.x * 2 + 1];
            if (a.std > 0.0f) {
                const uint64_t st =
                    (((uint64_t)a.step_ctr[1] << 32) | (uint64_t)a.step_ctr[0]) + (uint64_t)a.step_off;
                uint32_t c[4] = {(uint32_t)e, (uint32_t)st, (uint32_t)(st >> 32), 11u};
                philox4x32_10(c, a.key0, a.key1);
                const double u1 = ((double)c[0] + 0.5) / 4294967296.0;
                const double u2 = ((double)c[1] + 0.5) / 4294967296.0;
                const double rad = sqrt(-2.0 * log(u1));
                const double t = 2.0 * 3.14159265358979323846 * u2;
                v0 = fminf(1.0f, fmaxf(-1.0f, v0 + a.std * (float)(rad * cos(t))));
                v1 = fminf(1.0f, fmaxf(-1.0f, v1 + a.std * (float)(rad * sin(t))));
            }
            a.act[(int64_t)e * 2] = v0;
            a.act[(int64_t)e * 2 + 1] = v1;
        }
    }
}

// The proposer's network on noise rows, all layers in one launch (hidden width
// H): request i's draw j is row i per + j.  A workgroup of 8 wavefronts takes
// 128 rows: it draws their noise (noise_kernel's words), and runs every layer as
// 16 x 16 x 32 bf16 MFMA tiles with the rows' activations in LDS.  The weights
// are the A operand, so that a lane receives 4 consecutive columns of one row and
// writes them to the next layer's input with one 8-byte store.  Each wavefront
// owns 64 columns and 128 / (8 / (H / 64)) rows; its weights come from their
// packed image in L2 straight into registers, and each k block's registers are
// refilled with the next layer's weights as soon as they are used, so the loads
// run under the products.
// Same tiles, k order and rounding points as the layer-by-layer GEMMs (bitwise
// the same outputs), which serve other widths.
//
// Bound by the matrix cores and, as long again, the epilogue's VALU work (5
// instructions per activation) between barriers.  The GEMMs wrote and re-read
// every activation (512 bytes a row and layer).  131,072 rows of the 16-256-256-
// 256-5 network (36 GFLOP) in 67 us, 262,144 in 126 us (570 TFLOP/s), a step's
// 15,700 in 17 us, against 260, 430 and 62 us with the noise kernel and four
// GEMMs; 64 rows and 4 wavefronts a workgroup: 84, 157 and 20 us; weights from
// the row-major matrix instead of the packed image: 109, 217 and 28 us.  The code
// is 13 KB without a loop and starts at a page, so that its speed does not depend
// on the kernels before it (65.1 us, 66.6 at another offset; gradient_kernel 19.1,
// 19.8).
constexpr int kFwdThreads = 512;
constexpr int kFwdRows = kFwdThreads / 4;
constexpr int kFwdZPitch = 72;  // bf16 per noise row in LDS: up to 64 columns, 16 bytes of padding

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// bias + leaky ReLU on a lane's 4 columns, rounded to bf16 (nearest even)
__device__ __forceinline__ uint2 hidden_bf16(f32x4 v, float4 b, float slope) {
    v[0] += b.x;
    v[1] += b.y;
    v[2] += b.z;
    v[3] += b.w;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = v[r] > 0.0f ? v[r] : v[r] * slope;
    return __builtin_bit_cast(uint2, __builtin_convertvector(v, bf16x4));
}

template <int H>
__global__ __launch_bounds__(kFwdThreads) __attribute__((aligned(4096)))
void forward_noise_kernel(ForwardNoiseArgs a) {
    constexpr int KS = H / 32;          // k blocks of a hidden layer
    constexpr int WN = H / 64;          // wavefronts across the columns
    constexpr int MT = WN;              // 16-row tiles per wavefront: 64 / (4 / WN) / 16
    constexpr int LD = H + 8;           // LDS pitch: fragment reads hit every bank once
    __shared__ __attribute__((aligned(16))) uint16_t s_act[kFwdRows * LD];
    __shared__ __attribute__((aligned(16))) uint16_t s_z[kFwdRows * kFwdZPitch];
    __shared__ int s_row[kFwdRows];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (a.clear && blockIdx.x == 0 && tid == 0) *a.clear = 0;
    const int n = a.n_dev ? min(a.n, *a.n_dev) : a.n;
    const int rows = n * a.per;  // at most 2^24
    const int row0 = (int)blockIdx.x * kFwdRows;
    if (row0 >= rows) return;
    const int fr = lane & 15, fk = (lane >> 4) * 8;  // fragment row and first k
    const int n0 = (wave % WN) * 64, m0 = (wave / WN) * (MT * 16);
    // packed weights: fragment (16-row tile, k block) at ((tile) ks + k) 512
    const uint16_t *W1 = a.packed + (n0 >> 4) * 2 * 512 + lane * 8;
    const uint16_t *Wh = a.packed + WN * 4 * 2 * 512 + (n0 >> 4) * KS * 512 + lane * 8;
    bf16x8 w[4][KS];
    auto load_hidden = [&](const uint16_t *W, int i, int k) {
        w[i][k] = *reinterpret_cast<const bf16x8 *>(W + (i * KS + k) * 512);
    };
    // noise: 4 threads a row, 4 columns per draw
    {
        const int r = tid >> 2;
        const int row = row0 + r;
        const bool in = row < rows;
        const int i = in ? (int)((uint32_t)row / (uint32_t)a.per) : 0;
        const int j = in ? row - i * a.per : 0;
        const uint32_t c0 = a.c0 ? a.c0[i] : (uint32_t)i, c1 = a.c1 ? a.c1[i] : a.c1_const;
        if ((tid & 3) == 0) {
            const int m = a.map[i], b = a.bin[i];
            s_row[r] =
                (m >= 0 && m < a.num_maps && b >= 0 && b < a.nbins) ? m * a.nbins + b : 0;
        }
        // the weight loads go out before the draws, behind the loads that these need
        if (a.layers > 2)
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int t = 0; t < 4; ++t) load_hidden(Wh, t, k);
        const int cols = (a.nz + 31) & ~31;
        for (int q = tid & 3; 4 * q < cols; q += 4) {
            uint32_t c[4] = {c0, c1, ((uint32_t)j << 8) | (uint32_t)q, a.stream};
            philox4x32_10(c, a.key0, a.key1);
            uint16_t v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double u = ((double)c[t] + 0.5) / 4294967296.0;
                v[t] = in && 4 * q + t < a.nz ? to_bf16_bits((float)(2.0 * u - 1.0)) : (uint16_t)0;
            }
            *reinterpret_cast<uint2 *>(&s_z[r * kFwdZPitch + 4 * q]) =
                make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16),
                           (uint32_t)v[2] | ((uint32_t)v[3] << 16));
            if (a.z && in)
                for (int t = 0; t < 4; ++t)
                    if (4 * q + t < a.nz) a.z[(int64_t)row * a.nz + 4 * q + t] = v[t];
        }
    }
    f32x4 acc[4][MT];
    // first layer: the noise columns; the rest of its input is the (map, bin) row
    // of the constant table, added like a bias
    {
        bf16x8 w1[2][4];
#pragma unroll
        for (int kz = 0; kz < 2; ++kz)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w1[kz][i] = *reinterpret_cast<const bf16x8 *>(W1 + (i * 2 + kz) * 512);
        __syncthreads();  // noise and table rows in LDS
        // a tile's table entries are loaded while the tile before it is computed
        float4 cb[2][4];
        auto load_table = [&](int j, float4(&c)[4]) {
            const float *ct =
                a.ct + (int64_t)s_row[m0 + 16 * j + fr] * H + n0 + (lane >> 4) * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = *reinterpret_cast<const float4 *>(ct + 16 * i);
        };
        load_table(0, cb[0]);
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            if (j + 1 < MT) load_table(j + 1, cb[(j + 1) & 1]);
            const int m = m0 + 16 * j + fr;
            const bf16x8 z0 = *reinterpret_cast<const bf16x8 *>(&s_z[m * kFwdZPitch + fk]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    w1[0][i], z0, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            if (a.nz > 32) {
                const bf16x8 z1 = *reinterpret_cast<const bf16x8 *>(&s_z[m * kFwdZPitch + 32 + fk]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[1][i], z1, acc[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint2 *>(&s_act[m * LD + n0 + 16 * i + (lane >> 4) * 4]) =
                    hidden_bf16(acc[i][j], cb[j & 1][i], a.slope);
        }
    }
    __syncthreads();
    auto hidden = [&](int l, auto more) {  // more: another hidden layer follows
        const uint16_t *W = Wh + (int64_t)l * H * H;  // layer l + 1's
        float4 bias[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            bias[i] = *reinterpret_cast<const float4 *>(a.p + a.b_off[l] + n0 + 16 * i +
                                                        (lane >> 4) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            bf16x8 x[MT];
#pragma unroll
            for (int j = 0; j < MT; ++j)
                x[j] = *reinterpret_cast<const bf16x8 *>(&s_act[(m0 + 16 * j + fr) * LD + 32 * k + fk]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][k], x[j], acc[i][j], 0, 0, 0);
            if constexpr (decltype(more)::value)
#pragma unroll
                for (int i = 0; i < 4; ++i) load_hidden(W, i, k);
        }
        __syncthreads();  // every wavefront has read the layer's inputs
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint2 *>(
                    &s_act[(m0 + 16 * j + fr) * LD + n0 + 16 * i + (lane >> 4) * 4]) =
                    hidden_bf16(acc[i][j], bias[i], a.slope);
        __syncthreads();
    };
    for (int l = 1; l + 2 < a.layers; ++l) hidden(l, std::true_type{});
    if (a.layers > 2) hidden(a.layers - 2, std::false_type{});
    // output layer (5 columns): 16 rows per wavefront
    {
        const int l = a.layers - 1, m = 16 * wave + fr;
        const uint16_t *W =
            a.packed + WN * 4 * 2 * 512 + (int64_t)(a.layers - 2) * H * H + lane * 8;
        f32x4 o = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const bf16x8 wk = *reinterpret_cast<const bf16x8 *>(W + 512 * k);
            const bf16x8 x = *reinterpret_cast<const bf16x8 *>(&s_act[m * LD + 32 * k + fk]);
            o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wk, x, o, 0, 0, 0);
        }
        const int row = row0 + m;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = (lane >> 4) * 4 + r;
            if (c < 5 && row < rows) a.y[(int64_t)row * 5 + c] = o[r] + a.p[a.b_off[l] + c];
        }
    }
}

unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

int64_t packed_net_elems(int layers, int hidden) {
    return (int64_t)(hidden / 16) * 2 * 512 + (int64_t)(layers - 2) * hidden * hidden +
           (int64_t)(hidden / 32) * 512;
}

size_t actor_fused_lds_bytes(int layers, const int *kpad, const int *npad, int kmax) {
    return ((size_t)32 * (kmax + 8) + (size_t)actor_fused_wmax(layers, kpad, npad)) *
               sizeof(uint16_t) +
           16 * 2 * sizeof(float);
}

int actor_fused_wmax(int layers, const int *kpad, const int *npad) {
    int wmax = 0;
    for (int l = 0; l < layers; ++l) wmax = std::max(wmax, (kpad[l] + 8) * npad[l]);
    return (wmax + 7) & ~7;  // keeps the action floats after it 16-byte aligned
}

hipError_t launch_actor_fused(const ActorArgs &a, hipStream_t s) {
    if (a.N <= 0) return hipSuccess;
    const size_t lds = actor_fused_lds_bytes(a.layers, a.kpad, a.npad, a.kmax);
    hipLaunchKernelGGL(actor_fused_kernel, dim3((unsigned)((a.N + 15) / 16)), dim3(kActorThreads), lds,
                       s, a);
    return hipGetLastError();
}

bool forward_noise_supported(int hidden) { return hidden == 128 || hidden == 256; }

hipError_t launch_forward_noise(const ForwardNoiseArgs &a, int hidden, hipStream_t s) {
    const int64_t rows = (int64_t)a.n * a.per;
    if (rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)((rows + kFwdRows - 1) / kFwdRows));
    if (hidden == 256)
        hipLaunchKernelGGL(forward_noise_kernel<256>, grid, dim3(kFwdThreads), 0, s, a);
    else if (hidden == 128)
        hipLaunchKernelGGL(forward_noise_kernel<128>, grid, dim3(kFwdThreads), 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// Products of at least this many 64 x 64 blocks (two per CU) take those: they
// read each operand half as often.  A 256-wide forward pass of 4,096 rows (256
// blocks) 54 us in small blocks against 61, of 8,192 rows (512) 83 against 65.
constexpr int64_t kLargeBlocks = 512;

hipError_t launch_gemm(const GemmArgs &g, hipStream_t s) {
    if (!g.a_kmajor) return hipErrorInvalidValue;  // launch_gradient's products
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    const int64_t blocks = (int64_t)((g.M + kBM - 1) / kBM) * ((g.N + kBN - 1) / kBN);
    if (blocks < kLargeBlocks) {
        const dim3 sg((unsigned)((g.N + kSB - 1) / kSB), (unsigned)((g.M + kSB - 1) / kSB));
        if (g.b_kmajor)
            hipLaunchKernelGGL(gemm_small_kernel<true>, sg, dim3(256), 0, s, g);
        else
            hipLaunchKernelGGL(gemm_small_kernel<false>, sg, dim3(256), 0, s, g);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((g.N + kBN - 1) / kBN), (unsigned)((g.M + kBM - 1) / kBM));
    if (g.b_kmajor)
        hipLaunchKernelGGL(gemm_kernel<true>, grid, dim3(kGemmThreads), 0, s, g);
    else
        hipLaunchKernelGGL(gemm_kernel<false>, grid, dim3(kGemmThreads), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_gradient(const GradientArgs &a, hipStream_t s) {
    int64_t blocks = 0;
    for (int l = 0; l < a.gemms; ++l)
        blocks += (int64_t)((a.gemm[l].N + kSB - 1) / kSB) * ((a.gemm[l].M + kSB - 1) / kSB);
    for (int l = 0; l < a.sums; ++l) blocks += (a.sum[l].N + kColWidth - 1) / kColWidth;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(gradient_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_sq_loss(int M, int D, const float *Y, const float *T, const float *w,
                          float *L, float *dYf, uint16_t *dYb, hipStream_t s) {
    if (M == 0) return hipSuccess;
    hipLaunchKernelGGL(sq_loss_kernel, dim3(blocks_for(M, 256)), dim3(256), 0, s, M, D, Y, T, w,
                       L, dYf, dYb);
    return hipGetLastError();
}

hipError_t launch_adamw(int64_t n, float *p, uint16_t *pb, const float *g, float *m, float *v,
                        const uint8_t *decay_mask, float lr, float b1, float b2, float eps,
                        float wd, int64_t t, const PackedNet &f, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const float bc1 = (float)(1.0 - pow((double)b1, (double)t));
    const float bc2 = (float)(1.0 - pow((double)b2, (double)t));
    hipLaunchKernelGGL(adamw_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, p, pb, g, m, v,
                       decay_mask, lr, b1, b2, eps, wd, bc1, bc2, f);
    return hipGetLastError();
}

hipError_t launch_actor_input(int N, int m, const float *obs, const float *beta, uint16_t *x,
                              hipStream_t s) {
    const int64_t n = (int64_t)N * (m + 4);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(actor_input_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, N, m, obs,
                       beta, x);
    return hipGetLastError();
}

hipError_t launch_actor_noise(int N, float *act, float std, const uint32_t *step_ctr, int step_off,
                              uint32_t key0, uint32_t key1, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(actor_noise_kernel, dim3(blocks_for(N, 256)), dim3(256), 0, s, N, act, std,
                       step_ctr, step_off, key0, key1);
    return hipGetLastError();
}

hipError_t launch_to_bf16(int64_t n, const float *x, uint16_t *y, const PackedNet &f,
                          hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, x, y, f);
    return hipGetLastError();
}

}  // namespace navsim
