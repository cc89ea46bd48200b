// Surrogate MLP (protocol -> predicted fitness) with hand-written BF16 MFMA
// kernels: 128 -> 512 -> 512 -> 512 -> 1, GELU(x) = x Phi(x) on the hidden
// layers, BF16 weights and activations into v_mfma_f32_16x16x32_bf16 with FP32
// accumulation, FP32 master weights and Adam.  The surrogate only pre-screens
// GA offspring; the full simulation evaluates whatever it lets through.
//
// Net buffer (caller-owned, gga_mlp_net_bytes()):
//   header (normalisation mu, sigma) | params f32 | adam m | adam v | grads |
//   bf16 copies W_l [K][N] and W_l^T [N][K] for the three MFMA layers.
// Parameter order: W1 [128][512], b1, W2 [512][512], b2, W3 [512][512], b3,
// w4 [512], b4 [1].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gga_device.h"
#include "gga_internal.h"
#include "mlp_internal.h"

namespace gga {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int PADK = 8;   // LDS rows of BK + PADK bf16 (the pad spreads banks)

// Phi(x), the standard normal CDF, through erf(|x| / sqrt 2) in the rational
// form of Abramowitz & Stegun 7.1.26 (Hastings): erf(a) = 1 - p(t) exp(-a^2),
// t = 1 / (1 + 0.3275911 a), |error| <= 1.5e-7, so Phi is within 7.5e-8 (plus
// fp32 rounding) everywhere.  Branch-free: one reciprocal and one exp2 against
// the two-branch polynomial of the library erff.  e receives exp(-x^2 / 2),
// which the derivative also needs.
__device__ __forceinline__ float phi_as(float x, float& e) {
    const float a = fabsf(x) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, a, 1.0f));
    const float p =
        t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
    e = __builtin_amdgcn_exp2f(-a * a * 1.4426950408889634f);
    return 0.5f + copysignf(0.5f * fmaf(-p, e, 1.0f), x);
}
// GELU(x) = x Phi(x) = relu(x) - |x| p(t) exp(-x^2 / 2) / 2 with the same
// rational erf (x Phi(x) = x/2 + |x| erf(|x| / sqrt 2) / 2): 11 VALU operations
// and two transcendentals, the 1/2 and 1/sqrt 2 folded into the constants.
// GELU'(x) = Phi(x) + x phi(x), phi(x) = exp(-x^2 / 2) / sqrt(2 pi).
__device__ __forceinline__ float gelu_f(float x) {
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.2316418882f, ax, 1.0f));
    const float q =
        t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0.5307027145f, -0.7265760135f), 0.7107068705f), -0.142248368f),
                 0.127414796f);
    const float e = __builtin_amdgcn_exp2f(x * x * -0.7213475204f);
    return fmaf(-ax * q, e, fmaxf(x, 0.0f));
}
__device__ __forceinline__ float gelu_grad_f(float x) {
    float e;
    const float p = phi_as(x, e);
    return fmaf(x * 0.39894228040143268f, e, p);
}

// One bf16x8 vector of an operand tile: elements (r, k0..k0+7) of a matrix
// X(r, k) = X[r*s_r + k*s_k] with `rows` x `K` bounds, zero outside.
__device__ __forceinline__ bf16x8 load8(const bf16* X, int s_r, int s_k, int rows, int K, int r, int k0) {
    bf16x8 v;
    if (s_k == 1 && r < rows && k0 + 8 <= K && ((s_r & 7) == 0)) {
        v = *reinterpret_cast<const bf16x8*>(X + (size_t)r * s_r + k0);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + e;
            v[e] = (r < rows && k < K) ? X[(size_t)r * s_r + (size_t)k * s_k] : (bf16)0.0f;
        }
    }
    return v;
}

// C = A (M x K) * B (K x N) with element A(m,k) = A[m*sa_m + k*sa_k] and
// B(k,n) = B[k*sb_k + n*sb_n].  256 threads (2 x 2 waves) compute a
// (32 WT) x (32 WT) tile, each wave WT x WT blocks of MFMA 16x16x32, over
// k-tiles of BK.  The operand tiles are double-buffered in LDS: the global
// loads of k-tile t + 1 are in flight while the MFMAs of k-tile t run.
template <int WT, int BK>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(MlpGemm g) {
    constexpr int TM = 32 * WT;                          // tile rows (= tile columns)
    constexpr int VPT = TM * BK / 8 / 256;               // bf16x8 vectors per thread per operand
    __shared__ bf16 As[2][TM][BK + PADK];
    __shared__ bf16 Bs[2][TM][BK + PADK];                // stored as [n][k]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
    const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TM / 2);
    floatx4 acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ra[VPT], rb[VPT];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * 256, r = idx / (BK / 8), k = (idx % (BK / 8)) * 8;
            ra[v] = load8(g.A, g.sa_m, g.sa_k, g.M, g.K, m0 + r, k0 + k);
            rb[v] = load8(g.B, g.sb_n, g.sb_k, g.N, g.K, n0 + r, k0 + k);   // B^T(n, k) = B(k, n)
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * 256, r = idx / (BK / 8), k = (idx % (BK / 8)) * 8;
            *reinterpret_cast<bf16x8*>(&As[buf][r][k]) = ra[v];
            *reinterpret_cast<bf16x8*>(&Bs[buf][r][k]) = rb[v];
        }
    };
    const int nk = (g.K + BK - 1) / BK;
    fetch(0);
    stash(0);
    __syncthreads();
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    for (int t = 0; t < nk; ++t) {
        const int buf = t & 1;
        if (t + 1 < nk) fetch((t + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 32) {
            bf16x8 b[WT];
#pragma unroll
            for (int j = 0; j < WT; ++j) b[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf][wn + j * 16 + fr][kk + fk]);
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(&As[buf][wm + i * 16 + fr][kk + fk]);
#pragma unroll
                for (int j = 0; j < WT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[j], acc[i][j], 0, 0, 0);
            }
        }
        if (t + 1 < nk) stash(buf ^ 1);                  // the other buffer: last read before the previous barrier
        __syncthreads();
    }
    // D[4*(lane/16) + r][lane%16] of every 16x16 block
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm + i * 16 + (lane >> 4) * 4 + r;
                const int col = n0 + wn + j * 16 + (lane & 15);
                if (row >= g.M || col >= g.N) continue;
                float v = acc[i][j][r] + (g.bias ? g.bias[col] : 0.0f);
                if (g.mode == MLP_FWD) {
                    g.Z[(size_t)row * g.ldz + col] = v;
                    g.H[(size_t)row * g.ldh + col] = (bf16)gelu_f(v);
                } else if (g.mode == MLP_BWD) {
                    g.H[(size_t)row * g.ldh + col] = (bf16)(v * gelu_grad_f(g.Z[(size_t)row * g.ldz + col]));
                } else {
                    g.C[(size_t)row * g.ldc + col] = v;
                }
            }
}

// The same product when both operands run along K in memory (A [M][sa_m],
// B^T [N][sb_n]; every layer of the forward pass and the data gradient of the
// backward pass), K a multiple of 32 and N of the tile width: unguarded
// 16-byte loads (rows beyond M clamp to row M - 1 and are not stored), and the
// MFMA operands swapped so that each lane ends with four consecutive columns
// of one row, stored as one 16-byte (f32) or 8-byte (bf16) write.  The tile
// epilogue is fixed at compile time (MODE).  Workgroups are numbered so that
// the N / TM column tiles of one row block run on one XCD (blocks are dealt
// round-robin over the 8 XCDs), which then reads that row block once into its
// L2.  The accumulators start from the bias.  At most 122 VGPRs (no AGPRs),
// so four workgroups share a CU with k-steps of 32 (their LDS tiles fill its
// 160 KB), two with the small tile's steps of 128.
template <int WT, int BK, int MODE>
__global__ __launch_bounds__(256, 2) void gemm_nt_kernel(MlpGemm g) {
    constexpr int TM = 32 * WT, VPT = TM * BK / 8 / 256, CPR = BK / 8;
    __shared__ bf16 As[2][TM][BK + PADK];
    __shared__ bf16 Bs[2][TM][BK + PADK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ntn = g.N / TM;
    int bid = blockIdx.x;
    if ((gridDim.x & 7) == 0) bid = (bid & 7) * (gridDim.x >> 3) + (bid >> 3);
    const int m0 = (bid / ntn) * TM, n0 = (bid - (bid / ntn) * ntn) * TM;
    const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TM / 2);
    floatx4 acc[WT][WT];                                  // [column block][row block], from the bias
#pragma unroll
    for (int i = 0; i < WT; ++i) {
        floatx4 b0 = floatx4{0.f, 0.f, 0.f, 0.f};
        if (g.bias) {
            const float4 bb = *reinterpret_cast<const float4*>(g.bias + n0 + wn + i * 16 + (lane >> 4) * 4);
            b0 = floatx4{bb.x, bb.y, bb.z, bb.w};
        }
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = b0;
    }
    const bf16* pa[VPT];
    const bf16* pb[VPT];
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
        const int idx = tid + v * 256, r = idx / CPR, k = (idx % CPR) * 8;
        pa[v] = g.A + (size_t)min(m0 + r, g.M - 1) * g.sa_m + k;
        pb[v] = g.B + (size_t)(n0 + r) * g.sb_n + k;
    }
    bf16x8 ra[VPT], rb[VPT];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            ra[v] = *reinterpret_cast<const bf16x8*>(pa[v] + k0);
            rb[v] = *reinterpret_cast<const bf16x8*>(pb[v] + k0);
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int idx = tid + v * 256, r = idx / CPR, k = (idx % CPR) * 8;
            *reinterpret_cast<bf16x8*>(&As[buf][r][k]) = ra[v];
            *reinterpret_cast<bf16x8*>(&Bs[buf][r][k]) = rb[v];
        }
    };
    const int nk = g.K / BK;
    fetch(0);
    stash(0);
    __syncthreads();
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    for (int t = 0; t < nk; ++t) {
        const int buf = t & 1;
        if (t + 1 < nk) fetch((t + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 32) {
            bf16x8 a[WT];
#pragma unroll
            for (int j = 0; j < WT; ++j) a[j] = *reinterpret_cast<const bf16x8*>(&As[buf][wm + j * 16 + fr][kk + fk]);
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const bf16x8 b = *reinterpret_cast<const bf16x8*>(&Bs[buf][wn + i * 16 + fr][kk + fk]);
#pragma unroll
                for (int j = 0; j < WT; ++j)                // D^T block: rows n, columns m
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[j], acc[i][j], 0, 0, 0);
            }
        }
        if (t + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    // lane: row m0 + wm + 16 j + (lane & 15), columns n .. n + 3, n = n0 + wn + 16 i + 4 (lane >> 4)
#pragma unroll
    for (int j = 0; j < WT; ++j) {
        const int row = m0 + wm + j * 16 + (lane & 15);
        if (row >= g.M) continue;
#pragma unroll
        for (int i = 0; i < WT; ++i) {
            const int col = n0 + wn + i * 16 + (lane >> 4) * 4;
            float o[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            if (MODE == MLP_PLAIN) {
                *reinterpret_cast<float4*>(g.C + (size_t)row * g.ldc + col) = make_float4(o[0], o[1], o[2], o[3]);
                continue;
            }
            if (MODE == MLP_FWD)
                *reinterpret_cast<float4*>(g.Z + (size_t)row * g.ldz + col) = make_float4(o[0], o[1], o[2], o[3]);
            if (MODE == MLP_BWD) {
                const float4 z = *reinterpret_cast<const float4*>(g.Z + (size_t)row * g.ldz + col);
                o[0] *= gelu_grad_f(z.x); o[1] *= gelu_grad_f(z.y); o[2] *= gelu_grad_f(z.z); o[3] *= gelu_grad_f(z.w);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = gelu_f(o[q]);
            }
            bf16x4 h;
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = (bf16)o[q];
            *reinterpret_cast<bf16x4*>(g.H + (size_t)row * g.ldh + col) = h;
        }
    }
}

// Column sums over the batch of a [B][MLP_HID] bf16 matrix: chunk c of
// MLP_RED_CHUNKS adds its rows, each lane 8 consecutive columns (one 16-byte
// load per row) in 4 row groups of one wave each, combined in LDS in a fixed
// order into part[c]; grad_sum_kernel adds the chunks in order.  Row b is
// weighted by w[b] when w is given, and column MLP_HID then holds the sum of w.
struct ColSums {
    const bf16* D[2];
    const float* w[2];
    float* part[2];              // [MLP_RED_CHUNKS][MLP_HID + 1]
    int B;
};
__device__ __forceinline__ void colsum_chunk(const ColSums& a, int which, int c, float* lds) {
    float (*red)[MLP_HID] = reinterpret_cast<float (*)[MLP_HID]>(lds);
    float* redw = lds + 4 * MLP_HID;
    const bf16* D = which ? a.D[1] : a.D[0];
    const float* w = which ? a.w[1] : a.w[0];
    float* part = (which ? a.part[1] : a.part[0]) + (size_t)c * (MLP_HID + 1);
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6, col = lane * 8;
    const int rows = (a.B + MLP_RED_CHUNKS - 1) / MLP_RED_CHUNKS;
    const int b0 = c * rows, b1 = min(a.B, b0 + rows);
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float sw = 0.0f;
#pragma unroll 4
    for (int b = b0 + grp; b < b1; b += 4) {
        const float wb = w ? w[b] : 1.0f;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(D + (size_t)b * MLP_HID + col);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += (float)v[e] * wb;
        sw += wb;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[grp][col + e] = s[e];
    if (lane == 0) redw[grp] = sw;
    __syncthreads();
    for (int n = threadIdx.x; n < MLP_HID; n += 256) part[n] = ((red[0][n] + red[1][n]) + red[2][n]) + red[3][n];
    if (w && threadIdx.x == 0) part[MLP_HID] = ((redw[0] + redw[1]) + redw[2]) + redw[3];
}

// C = A (M x K) * B (K x N) when both operands run along M and N in memory
// (A(m, k) = A[k sa_k + m], B(k, n) = B[k sb_k + n]: the weight gradients
// H^T dZ), over the k range [k0, k1) of split blockIdx.y, M and N multiples of
// 64.  A thread loads 8 x 8 elements of one operand (8 rows of k, 16 bytes of
// each, whole 128-byte lines per 8 lanes), transposes them in registers and
// writes them as 16-byte parts of the [row][k] LDS tiles the MFMA fragments
// read; rows of k past k1 load as zero.  Part c of row m lies at part
// c ^ tn_swizzle(m), which keeps writes (rows 8 apart) and fragment reads (16
// consecutive rows) from meeting in a bank.  Each split writes its own f32
// slice C + split * ldp (a fixed-order sum over the splits follows when there
// are several).  Blocks past the tiles take the column sums that fall due with
// the product (see colsum_chunk), beside it instead of in launches of their own.
// Bound: the latency of its few k-steps.  With the transposed elements written
// one by one (16-bit LDS writes, k-steps of 32) 512 x 512 x 4,096 took 21 us,
// now 10, column sums included.
__device__ __forceinline__ int tn_swizzle(int m) { return ((m & 7) ^ ((m >> 3) & 7)) | (((m >> 3) & 1) << 3); }
__global__ __launch_bounds__(256) void gemm_tn_kernel(MlpGemm g, int kchunk, long ldp, ColSums sums) {
    constexpr int WT = 2, TM = 64, BK = 128;
    __shared__ __attribute__((aligned(16))) bf16 tile[2][2][TM][BK];      // [operand][buffer]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntn = g.N / TM, past = (int)blockIdx.x - ntn * (g.M / TM);
    if (past >= 0) {
        if (blockIdx.y == 0)
            colsum_chunk(sums, past / MLP_RED_CHUNKS, past % MLP_RED_CHUNKS, reinterpret_cast<float*>(&tile[0][0][0][0]));
        return;
    }
    const int m0 = (blockIdx.x / ntn) * TM, n0 = (blockIdx.x - (blockIdx.x / ntn) * ntn) * TM;
    const int kb = blockIdx.y * kchunk, ke = min(g.K, kb + kchunk);
    const int wm = (wave >> 1) * (TM / 2), wn = (wave & 1) * (TM / 2);
    const int op = wave >> 1;                              // waves 0 and 1 load A, 2 and 3 B
    const int mc = tid & 7, kc = (tid & 127) >> 3;         // the thread's 8 columns and 8 rows of k
    const bf16* src = op ? g.B + n0 : g.A + m0;
    const long stride = op ? g.sb_k : g.sa_k;
    floatx4 acc[WT][WT];                                  // [column block][row block]
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 v[8];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = k0 + kc * 8 + r;
            const bf16x8 z = {};
            v[r] = k < ke ? *reinterpret_cast<const bf16x8*>(src + (size_t)k * stride + mc * 8) : z;
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bf16x8 t;
#pragma unroll
            for (int r = 0; r < 8; ++r) t[r] = v[r][e];
            const int m = mc * 8 + e;
            *reinterpret_cast<bf16x8*>(&tile[op][buf][m][(kc ^ tn_swizzle(m)) * 8]) = t;
        }
    };
    const int nk = (ke - kb + BK - 1) / BK;
    if (nk > 0) {
        fetch(kb);
        stash(0);
    }
    __syncthreads();
    const int fr = lane & 15, fq = lane >> 4;
    for (int t = 0; t < nk; ++t) {
        const int buf = t & 1;
        if (t + 1 < nk) fetch(kb + (t + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
            auto fragment = [&](int o, int m) {
                return *reinterpret_cast<const bf16x8*>(&tile[o][buf][m][((kk * 4 + fq) ^ tn_swizzle(m)) * 8]);
            };
            bf16x8 a[WT];
#pragma unroll
            for (int j = 0; j < WT; ++j) a[j] = fragment(0, wm + j * 16 + fr);
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const bf16x8 b = fragment(1, wn + i * 16 + fr);
#pragma unroll
                for (int j = 0; j < WT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[j], acc[i][j], 0, 0, 0);
            }
        }
        if (t + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }
    float* C = g.C + (size_t)blockIdx.y * ldp;
#pragma unroll
    for (int j = 0; j < WT; ++j) {
        const int row = m0 + wm + j * 16 + (lane & 15);
#pragma unroll
        for (int i = 0; i < WT; ++i) {
            const int col = n0 + wn + i * 16 + (lane >> 4) * 4;
            *reinterpret_cast<float4*>(C + (size_t)row * g.ldc + col) =
                make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
    }
}

// The sums that follow a weight gradient, all in one launch and each in a fixed
// order: gW over the splits (4 entries per thread, the first `wblocks` blocks;
// none when the product wrote gW itself), gb over the chunks of its column
// sums, and behind the last layer's gradient gw4 and gb4 over theirs and the
// loss over the blocks of out_kernel.
struct MlpSums {
    const float* part;           // [S][n]
    int S, wblocks;
    long n;
    float* gW;
    const float* col[2];         // [MLP_RED_CHUNKS][MLP_HID + 1]
    float *gb, *gw4, *gb4;
    const float* sq;             // [nsq]
    int nsq, B;
    float* loss;
};
__global__ __launch_bounds__(256) void grad_sum_kernel(MlpSums a) {
    const int block = (int)blockIdx.x - a.wblocks;
    if (block < 0) {
        const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
        if (i >= a.n) return;
        float4 acc = *reinterpret_cast<const float4*>(a.part + i);
        for (int s = 1; s < a.S; ++s) {
            const float4 v = *reinterpret_cast<const float4*>(a.part + (size_t)s * a.n + i);
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
        *reinterpret_cast<float4*>(a.gW + i) = acc;
        return;
    }
    constexpr int BB = MLP_HID / 256;                      // blocks of a column vector
    const int which = block / BB, n = block % BB * 256 + (int)threadIdx.x;
    auto chunks = [&](const float* part, int at) {
        float s = 0.0f;
#pragma unroll 16
        for (int c = 0; c < MLP_RED_CHUNKS; ++c) s += part[(size_t)c * (MLP_HID + 1) + at];
        return s;
    };
    if (which == 0) {
        a.gb[n] = chunks(a.col[0], n);
    } else if (which == 1) {
        a.gw4[n] = chunks(a.col[1], n);
    } else {                                               // one block: thread 0 and, for the loss, all
        __shared__ float red[256];
        if (threadIdx.x == 0) a.gb4[0] = chunks(a.col[1], MLP_HID);
        red[threadIdx.x] = (int)threadIdx.x < a.nsq ? a.sq[threadIdx.x] : 0.0f;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0 && a.loss) a.loss[0] = red[0] / (float)a.B;
    }
}

// Features f0 .. f0 + 7 of protocol b (f0 a multiple of 8): for fraction j < 40,
// (dose/5, gap/60, 1) if present.  The dose and delay loads depend only on K,
// so they are in flight together with the load of nfrac[b].
__device__ __forceinline__ bf16x8 features(const float* dose, const int32_t* gap, const int32_t* nfrac, int b, int K,
                                           int f0) {
    const int j0 = f0 / 3, jmax = min(MLP_FRAC, K);
    float d[4], g[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool in = j0 + q < jmax;
        d[q] = in ? dose[(size_t)b * K + j0 + q] * (1.0f / 5.0f) : 0.0f;
        g[q] = in ? (float)gap[(size_t)b * K + j0 + q] * (1.0f / 60.0f) : 0.0f;
    }
    const int nf = min(jmax, nfrac[b]);
    bf16x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int f = f0 + e, j = f / 3, part = f - 3 * j, q = j - j0;
        const float v = part == 0 ? d[q] : part == 1 ? g[q] : 1.0f;
        x[e] = (bf16)(j < nf ? v : 0.0f);
    }
    return x;
}

// One thread per 8 consecutive features, stored as one 16-byte vector.
__global__ void encode_kernel(const float* dose, const int32_t* gap, const int32_t* nfrac, int B, int K,
                              bf16* X) {
    constexpr int V = MLP_IN / 8;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= B * V) return;
    const int b = idx / V, f0 = (idx - b * V) * 8;
    *reinterpret_cast<bf16x8*>(X + (size_t)b * MLP_IN + f0) = features(dose, gap, nfrac, b, K, f0);
}

// A whole prediction in one launch.  A workgroup takes 16 MB protocols through
// all layers with their activations in LDS (one buffer, overwritten layer by
// layer: a layer's outputs are complete in the accumulators first).  Wave w
// computes columns [64 w, 64 w + 64) of every layer; no other wave of the
// workgroup needs those weights, so it fetches them from L2 itself, 128 values
// of k ahead (the next layer's too), and passes them through its own LDS strip
// into the MFMA fragments' order.  The sums run as in gemm_nt_kernel (from the
// bias, k ascending by 32), the output layer per 64 columns and then over the
// eight waves in order.
// Bound: for one workgroup per CU the weights, 1.2 MB from L2 per workgroup
// (8 us at 64 bytes a cycle; loading the fragments directly, 16 lanes on 16
// lines, ran at 17 bytes a cycle: 36 us against 19), and for many the GELUs'
// VALU work (13 us per 64 protocols) after the products.  A launch per layer
// with the activations through device memory took 152 us for 65,536 protocols
// and 33 for 5,000, this 131 and 23.  (Two workgroups of 32 protocols on a CU,
// one's GELUs beside the other's products, fetch the weights twice as often:
// 168 us.)
constexpr int FUSED_PITCH = MLP_HID + PADK;
template <int MB>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
predict_kernel(MlpNet net, const float* dose, const int32_t* gap, const int32_t* nfrac, int B, int K, float* pred) {
    constexpr int ROWS = 16 * MB;
    // k in steps of 64, the two fragments of a 128-byte line together: 2 of the first layer, then 8 and 8
    constexpr int END0 = MLP_IN / 64, END1 = END0 + MLP_HID / 64, END2 = END1 + MLP_HID / 64;
    __shared__ __attribute__((aligned(16))) bf16 act[ROWS][FUSED_PITCH];
    __shared__ __attribute__((aligned(16))) bf16 stage[8][64 * 64];   // per wave: a step's weights
    __shared__ float red[8][ROWS];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = (int)blockIdx.x * ROWS;
    const int fr = lane & 15, fk = (lane >> 4) * 8, n0 = wave * 64;
    // step's weights of the wave's 64 columns: 8 lanes a 128-byte line, 8 columns an access
    bf16x8 wq[2][8];
    auto weights = [&](int step, bf16x8 (&q)[8]) {
        const int l = step < END0 ? 0 : step < END1 ? 1 : 2, kd = step < END0 ? MLP_IN : MLP_HID;
        const bf16* base = net.WT[0];
        if (l == 1) base = net.WT[1];
        if (l == 2) base = net.WT[2];
        base += (size_t)n0 * kd + (step - (l == 0 ? 0 : l == 1 ? END0 : END1)) * 64;
        const uint32_t at = (uint32_t)((lane >> 3) * kd + (lane & 7) * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = *reinterpret_cast<const bf16x8*>(base + (size_t)i * 8 * kd + at);
    };
    // Staging: column r's 16-byte part c at part c ^ (r / 2 mod 8), so that neither
    // the writes nor the fragment reads (16 columns, one part) meet in a bank.  Lanes
    // read what other lanes of the wave wrote: the wave's LDS accesses execute in
    // order, so a wavefront fence on either side of the reads, which costs no
    // instruction, is all the hand-over needs.
    bf16* const st = stage[wave];
    auto part = [&](int r, int c) { return st + r * 64 + ((c ^ (r >> 1)) & 7) * 8; };
    weights(0, wq[0]);
    weights(1, wq[1]);
    for (int v = tid; v < ROWS * (MLP_IN / 8); v += 512) {
        const int r = v / (MLP_IN / 8), f0 = v % (MLP_IN / 8) * 8;
        *reinterpret_cast<bf16x8*>(&act[r][f0]) = features(dose, gap, nfrac, min(b0 + r, B - 1), K, f0);
    }
    floatx4 acc[4][MB];                                   // [column block][row block]
    auto start = [&](const float* bias) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 bb = *reinterpret_cast<const float4*>(bias + n0 + i * 16 + (lane >> 4) * 4);
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[i][j] = floatx4{bb.x, bb.y, bb.z, bb.w};
        }
    };
    start(net.b[0]);
    __syncthreads();                                      // the features are in LDS
    typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
    int k0 = 0;                                           // the step's first k in its layer
#pragma nounroll
    for (int step = 0; step < END2; step += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int i = 0; i < 8; ++i) *reinterpret_cast<bf16x8*>(part(i * 8 + (lane >> 3), lane & 7)) = wq[b][i];
            if (step + 2 + b < END2) weights(step + 2 + b, wq[b]);   // also the next layer's first
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8 a[MB], w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const bf16x8*>(part(i * 16 + fr, h * 4 + (lane >> 4)));
#pragma unroll
                for (int j = 0; j < MB; ++j) a[j] = *reinterpret_cast<const bf16x8*>(&act[j * 16 + fr][k0 + b * 64 + h * 32 + fk]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < MB; ++j)          // D^T block: rows n, columns m
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], a[j], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_sched_barrier(0);
        }
        k0 += 128;
        if (step + 2 == END0 || step + 2 == END1) {
            k0 = 0;
            __syncthreads();                              // the layer's inputs are read
            // lane: row 16 j + (lane & 15), columns n0 + 16 i + 4 (lane >> 4) .. + 3
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < MB; ++j) {
                    bf16x4 h;
#pragma unroll
                    for (int q = 0; q < 4; ++q) h[q] = (bf16)gelu_f(acc[i][j][q]);
                    *reinterpret_cast<bf16x4*>(&act[j * 16 + fr][n0 + i * 16 + (lane >> 4) * 4]) = h;
                }
            start(step + 2 == END0 ? net.b[1] : net.b[2]);
            __syncthreads();                              // the next layer's inputs are in LDS
        }
    }
#pragma unroll
    for (int j = 0; j < MB; ++j) {                        // H3 . w4, H3 rounded to bf16
        float dot = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 w = *reinterpret_cast<const float4*>(net.w4 + n0 + i * 16 + (lane >> 4) * 4);
            dot = fmaf((float)(bf16)gelu_f(acc[i][j][0]), w.x, dot);
            dot = fmaf((float)(bf16)gelu_f(acc[i][j][1]), w.y, dot);
            dot = fmaf((float)(bf16)gelu_f(acc[i][j][2]), w.z, dot);
            dot = fmaf((float)(bf16)gelu_f(acc[i][j][3]), w.w, dot);
        }
        dot += __shfl_xor(dot, 16, 64);
        dot += __shfl_xor(dot, 32, 64);
        if (lane < 16) red[wave][j * 16 + lane] = dot;
    }
    __syncthreads();
    if (tid < ROWS && b0 + tid < B) {
        float y = 0.0f;
#pragma unroll
        for (int w = 0; w < 8; ++w) y += red[w][tid];
        pred[b0 + tid] = (y + net.b4[0]) * net.norm[1] + net.norm[0];
    }
}

// The output layer of a training step, forward and backward, and the loss: per
// row b (one wave, every 64th column a lane) y = H3[b] . w4 + b4, e = y - t'
// with t' = (t - mu) / sigma, dy = 2 e / B and dZ3[b] = dy w4 gelu'(Z3[b]); per
// block of `rows` rows (at most 256 blocks) the sum of e^2.  One pass over H3
// and Z3; separate launches for y, the loss and dZ3 took 18 us for 4,096 rows,
// this 7.
__global__ __launch_bounds__(256) void out_kernel(const bf16* H3, const float* Z3, const float* w4, const float* b4,
                                                  const float* t, const float* norm, int B, int rows, float* y, float* dy,
                                                  bf16* dZ3, float* sq) {
    __shared__ float red[4];
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int r0 = (int)blockIdx.x * rows, r1 = min(B, r0 + rows);
    float w[8], se = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = w4[lane + 64 * e];
    const float mu = norm[0], sigma = norm[1], bias = b4[0];
    for (int b = r0 + grp; b < r1; b += 4) {
        const size_t at = (size_t)b * MLP_HID + lane;
        float h[8], z[8], s = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h[e] = (float)H3[at + 64 * e];
            z[e] = Z3[at + 64 * e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s += h[e] * w[e];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        const float yb = s + bias, err = yb - (t[b] - mu) / sigma, d = 2.0f * err / (float)B;
        if (lane == 0) {
            y[b] = yb;
            dy[b] = d;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) dZ3[at + 64 * e] = (bf16)(d * w[e] * gelu_grad_f(z[e]));
        se += err * err;
    }
    if (lane == 0) red[grp] = se;
    __syncthreads();
    if (threadIdx.x == 0) sq[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Adam with bias correction over the flat parameter vector, and the bf16 copies
// W [K][N] and W^T [N][K] of the three MFMA layers.  Blocks of 32 x 64 weights
// (W^T leaves through LDS in whole rows), then blocks of 256 of the other
// parameters.  One launch instead of one for Adam and one per layer, which read
// the weights again and wrote W^T two bytes a line: 17 us, now 8.
constexpr int ADAM_K = 32, ADAM_N = 64;
constexpr int adam_tiles(int K) { return K / ADAM_K * (MLP_HID / ADAM_N); }
constexpr int ADAM_TILES = adam_tiles(MLP_IN) + 2 * adam_tiles(MLP_HID);
constexpr int ADAM_REST = 4 * MLP_HID + 1;                // biases, w4, b4
__global__ __launch_bounds__(256) void adam_kernel(MlpNet net, float lr) {
    const float t = (float)*net.step;                   // bias corrections of step t
    const float c1 = 1.0f - powf(0.9f, t), c2 = 1.0f - powf(0.999f, t);
    auto update = [&](long i, float gi, float m0, float v0, float p0) {
        const float mi = 0.9f * m0 + 0.1f * gi;
        const float vi = 0.999f * v0 + 0.001f * gi * gi;
        net.m[i] = mi;
        net.v[i] = vi;
        return net.p[i] = p0 - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    };
    int tile = (int)blockIdx.x;
    if (tile >= ADAM_TILES) {
        int j = (tile - ADAM_TILES) * 256 + (int)threadIdx.x;
        if (j >= ADAM_REST) return;
        const int l = j / MLP_HID;                      // b1, b2, b3, then w4 and b4, which follow b3
        const long i = (l == 0 ? net.b[0] + j : l == 1 ? net.b[1] + j % MLP_HID : l == 2 ? net.b[2] + j % MLP_HID
                                                                                : net.w4 + (j - 3 * MLP_HID)) - net.p;
        update(i, net.g[i], net.m[i], net.v[i], net.p[i]);
        return;
    }
    __shared__ bf16 s_t[ADAM_N][ADAM_K + 2];
    int l = 0;
    while (tile >= adam_tiles(l ? MLP_HID : MLP_IN)) tile -= adam_tiles(l++ ? MLP_HID : MLP_IN);
    const int K = l ? MLP_HID : MLP_IN;
    float* W = l == 0 ? net.Wf[0] : l == 1 ? net.Wf[1] : net.Wf[2];
    bf16* Wb = l == 0 ? net.W[0] : l == 1 ? net.W[1] : net.W[2];
    bf16* WT = l == 0 ? net.WT[0] : l == 1 ? net.WT[1] : net.WT[2];
    const int k0 = tile / (MLP_HID / ADAM_N) * ADAM_K, n0 = tile % (MLP_HID / ADAM_N) * ADAM_N;
    constexpr int PER = ADAM_K * ADAM_N / 256;
    float in[PER][4];                                   // all loads before the first store
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = q * 256 + (int)threadIdx.x;
        const long i = W - net.p + (long)(k0 + e / ADAM_N) * MLP_HID + n0 + e % ADAM_N;
        in[q][0] = net.g[i];
        in[q][1] = net.m[i];
        in[q][2] = net.v[i];
        in[q][3] = net.p[i];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = q * 256 + (int)threadIdx.x, k = e / ADAM_N, n = e % ADAM_N;
        const long at = (long)(k0 + k) * MLP_HID + n0 + n;
        const bf16 v = (bf16)update(W - net.p + at, in[q][0], in[q][1], in[q][2], in[q][3]);
        Wb[at] = v;
        s_t[n][k] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = q * 256 + (int)threadIdx.x, n = e / ADAM_K, k = e % ADAM_K;
        WT[(long)(n0 + n) * K + k0 + k] = s_t[n][k];
    }
}

// bf16 copies W [K][N] and W^T [N][K] of a K x N layer.
__global__ void refresh_kernel(const float* W, int K, int N, bf16* Wb, bf16* WTb) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= K * N) return;
    const int k = idx / N, n = idx - k * N;
    const bf16 v = (bf16)W[idx];
    Wb[idx] = v;
    WTb[(size_t)n * K + k] = v;
}

// Weights uniform on +-1/sqrt(fan_in) from Philox blocks (i, 0x4D4C5000, layer, 0);
// biases and Adam state zero.
__global__ void init_kernel(float* p, float* m, float* v, float* g, long n, uint32_t k0, uint32_t k1) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    long off = i;
    int layer = -1;
    float fan_in = 1.0f;
    const long sizes[8] = {(long)MLP_IN * MLP_HID, MLP_HID, (long)MLP_HID * MLP_HID, MLP_HID,
                           (long)MLP_HID * MLP_HID, MLP_HID, MLP_HID, 1};
    const float fans[8] = {(float)MLP_IN, 0.f, (float)MLP_HID, 0.f, (float)MLP_HID, 0.f, (float)MLP_HID, 0.f};
    for (int t = 0; t < 8; ++t) {
        if (off < sizes[t]) { layer = t; fan_in = fans[t]; break; }
        off -= sizes[t];
    }
    float w = 0.0f;
    if (fan_in > 0.0f) {
        const Block4 b = philox10((uint32_t)i, 0x4D4C5000u, (uint32_t)layer, 0u, k0, k1);
        const float u = ((float)(b.w0 >> 8) + 0.5f) * (1.0f / 16777216.0f);
        w = (2.0f * u - 1.0f) / sqrtf(fan_in);
    }
    p[i] = w;
    m[i] = 0.0f;
    v[i] = 0.0f;
    g[i] = 0.0f;
}

// mu, sigma of n targets (one block, float64 accumulation).
__global__ __launch_bounds__(256) void norm_kernel(const float* t, int n, float* norm) {
    __shared__ double s1[256], s2[256];
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) { a += t[i]; b += (double)t[i] * t[i]; }
    s1[threadIdx.x] = a;
    s2[threadIdx.x] = b;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) { s1[threadIdx.x] += s1[threadIdx.x + w]; s2[threadIdx.x] += s2[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mu = n ? s1[0] / n : 0.0;
        const double var = n ? s2[0] / n - mu * mu : 1.0;
        norm[0] = (float)mu;
        norm[1] = (float)(var > 1e-12 ? sqrt(var) : 1.0);
    }
}

unsigned blocks_for(long n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

namespace {
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Operands that run along K, K a multiple of 32 (of 128 in the small tile's form
// of a layer, whose K is 128 or 512), N of the tile width, and 16-byte alignment
// of every row the epilogue and the loads touch.
bool nt_eligible(const MlpGemm& g, int TM) {
    if (g.sa_k != 1 || g.sb_k != 1 || g.K <= 0 || g.K % 32 || g.N % TM) return false;
    if (g.sa_m % 8 || g.sb_n % 8 || !aligned16(g.A) || !aligned16(g.B)) return false;
    if (g.bias && !aligned16(g.bias)) return false;
    if (g.mode == MLP_PLAIN) return aligned16(g.C) && g.ldc % 4 == 0;
    if ((TM == 64 && g.K % 128) || !aligned16(g.Z) || g.ldz % 4) return false;
    return aligned16(g.H) && g.ldh % 4 == 0;
}

template <int WT, int BK, bool LAYERS = true>
void launch_nt(const MlpGemm& g, hipStream_t s) {
    const dim3 grid(blocks_for(g.M, 32 * WT) * (g.N / (32 * WT)));
    if (g.mode == MLP_PLAIN) {
        hipLaunchKernelGGL((gemm_nt_kernel<WT, BK, MLP_PLAIN>), grid, dim3(256), 0, s, g);
    } else if constexpr (LAYERS) {
        if (g.mode == MLP_FWD)
            hipLaunchKernelGGL((gemm_nt_kernel<WT, BK, MLP_FWD>), grid, dim3(256), 0, s, g);
        else
            hipLaunchKernelGGL((gemm_nt_kernel<WT, BK, MLP_BWD>), grid, dim3(256), 0, s, g);
    }
}
}  // namespace

// Both operands along M and N, M and N multiples of 64, 16-byte aligned rows.
bool tn_eligible(const MlpGemm& g) {
    if (g.mode != MLP_PLAIN || g.sa_m != 1 || g.sb_n != 1 || g.K <= 0 || g.M % 64 || g.N % 64) return false;
    if (g.sa_k % 8 || g.sb_k % 8 || !aligned16(g.A) || !aligned16(g.B) || g.bias) return false;
    return aligned16(g.C) && g.ldc % 4 == 0;
}

// 128 x 128 tiles when they still give the chip two workgroups per CU, else 64 x 64
int gemm_tile(const MlpGemm& g) { return (long)blocks_for(g.N, 128) * blocks_for(g.M, 128) >= 512 ? 128 : 64; }

hipError_t launch_gemm(const MlpGemm& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    const bool large = gemm_tile(g) == 128;
    if (nt_eligible(g, large ? 128 : 64)) {
        // The small tile's k-steps are bound by their loads' latency, so they are as
        // long as K allows: a training step of 64 rows takes 68 us with steps of
        // 128 against 76 with 32, one of 4,096 104 against 111, of 8,192 165 and 166.
        if (large) launch_nt<4, 32>(g, s);
        else if (g.K % 128 == 0) launch_nt<2, 128>(g, s);
        else if (g.K % 64 == 0) launch_nt<2, 64, false>(g, s);
        else launch_nt<2, 32, false>(g, s);
        return hipGetLastError();
    }
    if (tn_eligible(g)) {
        hipLaunchKernelGGL(gemm_tn_kernel, dim3((g.M / 64) * (g.N / 64), 1), dim3(256), 0, s, g, g.K, 0L, ColSums{});
        return hipGetLastError();
    }
    if (large)
        hipLaunchKernelGGL((gemm_bf16_kernel<4, 32>), dim3(blocks_for(g.N, 128), blocks_for(g.M, 128)), dim3(256), 0, s,
                           g);
    else
        hipLaunchKernelGGL((gemm_bf16_kernel<2, 32>), dim3(blocks_for(g.N, 64), blocks_for(g.M, 64)), dim3(256), 0, s,
                           g);
    return hipGetLastError();
}

hipError_t mlp_predict(const MlpNet& net, const float* dose, const int32_t* gap, const int32_t* nfrac, int B, int K,
                       float* pred, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    // As few protocols per workgroup as still leave each CU at most one: a round of
    // workgroups takes 19 us with 16 protocols each, 23 with 32, 33 with 64.
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    auto launch = [&](auto* kernel, int rows) {
        hipLaunchKernelGGL(kernel, dim3(blocks_for(B, rows)), dim3(512), 0, s, net, dose, gap, nfrac, B, K, pred);
    };
    if (B <= 16LL * cus) launch(predict_kernel<1>, 16);
    else if (B <= 32LL * cus) launch(predict_kernel<2>, 32);
    else launch(predict_kernel<4>, 64);
    return hipGetLastError();
}

// The hidden layers of a training step: every layer's Z and H into w.
hipError_t mlp_forward(const MlpNet& net, const float* dose, const int32_t* gap, const int32_t* nfrac, int B,
                       int K, const MlpWork& w, hipStream_t s) {
    hipLaunchKernelGGL(encode_kernel, dim3(blocks_for((long)B * (MLP_IN / 8), 256)), dim3(256), 0, s, dose, gap,
                       nfrac, B, K, w.X);
    hipError_t e = hipGetLastError();
    const bf16* in = w.X;
    int kin = MLP_IN;
    for (int l = 0; l < 3 && e == hipSuccess; ++l) {
        MlpGemm g{};
        g.M = B; g.N = MLP_HID; g.K = kin;
        g.A = in; g.sa_m = kin; g.sa_k = 1;
        g.B = net.WT[l]; g.sb_k = 1; g.sb_n = kin;           // B(k, n) = W^T[n][k]
        g.bias = net.b[l];
        g.mode = MLP_FWD;
        g.Z = w.Z[l]; g.ldz = MLP_HID;
        g.H = w.H[l]; g.ldh = MLP_HID;
        e = launch_gemm(g, s);
        in = w.H[l];
        kin = MLP_HID;
    }
    return e;
}

// The output layer and the loss, then the gradients of every layer.  A weight
// gradient (K = batch rows) is split over S workgroups per tile so that the
// 16-64 tiles of a 512-wide layer fill the chip, S = B / 512 up to 8, its
// partials in the spent Z3 buffer until they are summed in split order.
hipError_t mlp_backward(const MlpNet& net, int B, const float* target, const MlpWork& w, float* loss,
                        hipStream_t s) {
    // The output layer's column sums and squares lie where the first layer's
    // gradient goes last (MLP_IN MLP_HID floats): they are spent by then.
    static_assert((long)MLP_IN * MLP_HID >= (long)MLP_RED_CHUNKS * (MLP_HID + 1) + 256, "scratch in gW[0]");
    const int rows = std::max(16, (B + 255) / 256), nout = (B + rows - 1) / rows;
    float* const out = net.gW[0];
    float* const sq = out + MLP_RED_CHUNKS * (MLP_HID + 1);
    hipLaunchKernelGGL(out_kernel, dim3(nout), dim3(256), 0, s, w.H[2], w.Z[2], net.w4, net.b4, target, net.norm, B, rows,
                       w.y, w.dy, w.dZ[0], sq);
    hipError_t e = hipGetLastError();
    // layer l = 2, 1, 0: dZ_l in dZ[cur]; weight and bias gradients, then dZ_{l-1}
    int cur = 0;
    for (int l = 2; l >= 0 && e == hipSuccess; --l) {
        const int kin = l == 0 ? MLP_IN : MLP_HID;
        MlpGemm g{};
        g.M = kin; g.N = MLP_HID; g.K = B;                    // dW_l = H_in^T dZ_l
        g.A = l == 0 ? w.X : w.H[l - 1]; g.sa_m = 1; g.sa_k = kin;
        g.B = w.dZ[cur]; g.sb_k = MLP_HID; g.sb_n = 1;
        g.mode = MLP_PLAIN;
        g.C = net.gW[l]; g.ldc = MLP_HID;
        if (!tn_eligible(g)) return hipErrorInvalidValue;
        const long mn = (long)g.M * g.N;
        int S = std::min(MLP_SPLITS, std::max(1, B / 512));
        const int kchunk = ((B + S - 1) / S + 31) / 32 * 32;
        S = (B + kchunk - 1) / kchunk;
        if (S > 1) g.C = w.Z[2];                              // S M N <= B MLP_HID floats
        // bias gradients, and with the last layer's dw4 = H3^T dy and db4 = sum dy
        const ColSums sums{{w.dZ[cur], w.H[2]}, {nullptr, w.dy}, {w.part, out}, B};
        const unsigned cols = (l == 2 ? 2 : 1) * MLP_RED_CHUNKS;
        hipLaunchKernelGGL(gemm_tn_kernel, dim3((g.M / 64) * (g.N / 64) + cols, S), dim3(256), 0, s, g, kchunk, mn, sums);
        MlpSums a{};
        a.part = w.Z[2]; a.S = S; a.n = mn; a.gW = net.gW[l];
        a.wblocks = S > 1 ? (int)blocks_for(mn / 4, 256) : 0;
        a.col[0] = w.part; a.col[1] = out;
        a.gb = net.gb[l]; a.gw4 = net.gw4; a.gb4 = net.gb4;
        a.sq = sq; a.nsq = nout; a.B = B; a.loss = loss;
        const unsigned blocks = a.wblocks + (l == 2 ? 2 * (MLP_HID / 256) + 1 : MLP_HID / 256);
        hipLaunchKernelGGL(grad_sum_kernel, dim3(blocks), dim3(256), 0, s, a);
        e = hipGetLastError();
        if (l == 0 || e != hipSuccess) break;
        MlpGemm d{};
        d.M = B; d.N = MLP_HID; d.K = MLP_HID;                // dZ_{l-1} = (dZ_l W_l^T) . gelu'(Z_{l-1})
        d.A = w.dZ[cur]; d.sa_m = MLP_HID; d.sa_k = 1;
        d.B = net.W[l]; d.sb_k = 1; d.sb_n = MLP_HID;         // B(k, n) = W_l[n][k]
        d.mode = MLP_BWD;
        d.Z = w.Z[l - 1]; d.ldz = MLP_HID;
        d.H = w.dZ[1 - cur]; d.ldh = MLP_HID;
        e = launch_gemm(d, s);
        cur = 1 - cur;
    }
    return e;
}

hipError_t mlp_adam_refresh(const MlpNet& net, int step, float lr, hipStream_t s) {
    // the net's step counter: set to `step`, or advanced by one when step is 0
    hipError_t e = launch_counter(net.step, step > 0 ? step : 1, step > 0 ? 0 : 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(adam_kernel, dim3(ADAM_TILES + blocks_for(ADAM_REST, 256)), dim3(256), 0, s, net, lr);
    return hipGetLastError();
}

hipError_t mlp_refresh_layer(const MlpNet& net, int l, hipStream_t s) {
    const int K = l == 0 ? MLP_IN : MLP_HID;
    hipLaunchKernelGGL(refresh_kernel, dim3(blocks_for((long)K * MLP_HID, 256)), dim3(256), 0, s, net.Wf[l], K,
                       MLP_HID, net.W[l], net.WT[l]);
    return hipGetLastError();
}

hipError_t mlp_init(const MlpNet& net, uint64_t seed, hipStream_t s) {
    const long n = MLP_PARAMS;
    hipLaunchKernelGGL(init_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, net.p, net.m, net.v, net.g, n,
                       (uint32_t)seed, (uint32_t)(seed >> 32));
    hipError_t e = hipGetLastError();
    for (int l = 0; l < 3 && e == hipSuccess; ++l) e = mlp_refresh_layer(net, l, s);
    return e;
}

hipError_t mlp_set_norm(const MlpNet& net, const float* t, int n, hipStream_t s) {
    hipLaunchKernelGGL(norm_kernel, dim3(1), dim3(256), 0, s, t, n, net.norm);
    return hipGetLastError();
}

}  // namespace gga
