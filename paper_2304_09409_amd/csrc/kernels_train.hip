// kernels_train.hip -- training-mode backward (Sec. II.B), FP64: the fitting nets with their tangent and
// their reverse pass, the loss, the packing of the parameters, Adam. The decomposition is in
// dpk_train.h, the embedding nets in kernels_tre.hip.
//
// Every layer y = w_hat tanh(x W + b) + skip(x) of the fitting net carries its tangent (y, ydot); the
// adjoint pair (ybar, ydotbar) gives
//   zbar = w_hat (1 - a^2) ybar - 2 w_hat a (1 - a^2) zdot ydotbar,  zdotbar = w_hat (1 - a^2) ydotbar,
//   Wbar += x zbar^T + xdot zdotbar^T,  bbar += zbar,  w_hatbar += a ybar + (1 - a^2) zdot ydotbar,
//   xbar = W zbar + skip^T ybar,  xdotbar = W zdotbar + skip^T ydotbar.
// The rows are the atoms, grouped by type; one launch covers every type (blockIdx.z). The layers are row
// GEMMs on v_mfma_f64_16x16x4f64 with both products of a weight tile (value and tangent) in one pass and
// the layer's arithmetic in the epilogue: forward the activation, in reverse the adjoint of the layer
// below with its bias and w_hat sums, so that no elementwise pass stands between two GEMMs. The next
// K-chunk of every operand is read into registers before the products of the current one.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dpk_device.h"
#include "dpk_train.h"

namespace dpk {
namespace {

// Offsets inside one fitting net's block of the parameter vector: layers (W, b, w_hat) 1600 -> 240 ->
// 240 -> 240 -> 1.
constexpr int64_t TF_W[4] = {0, (int64_t)DD * FW + 2 * FW, (int64_t)DD * FW + 4 * FW + FW * FW,
                             (int64_t)DD * FW + 6 * FW + 2 * FW * FW};
constexpr int64_t TF_NET = TF_W[3] + FW + 2;
__host__ __device__ constexpr int tf_in(int l) { return l == 0 ? DD : FW; }   // inputs of layer l = 0, 1, 2
__host__ __device__ constexpr int64_t tf_w(int l)
{
    return l == 0 ? TF_W[0] : l == 1 ? TF_W[1] : l == 2 ? TF_W[2] : TF_W[3];
}

// ---------------------------------------------------------------------------------------------
// D = T T_<^T and its tangent, one block per atom
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_trf_desc(TrfArgs A)
{
    __shared__ __attribute__((aligned(16))) double sT[E2][4], sTd[E2][4];
    const size_t a = blockIdx.x;
    for (int e = threadIdx.x; e < E2 * 4; e += 256) {
        sT[e >> 2][e & 3] = A.T[a * E2 * 4 + e];
        sTd[e >> 2][e & 3] = A.Td[a * E2 * 4 + e];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < DD; e += 256) {
        const int m = e >> 4, n = e & 15;
        double d = 0.0, dd = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d += sT[m][k] * sT[n][k];
            dd += sTd[m][k] * sT[n][k] + sT[m][k] * sTd[n][k];
        }
        A.D[a * DD + e] = d;
        A.Dd[a * DD + e] = dd;
    }
}

// Its adjoint: Tb[p] = sum_n Db[p][n] T[n] + Ddb[p][n] Td[n], Tdb[p] = sum_n Ddb[p][n] T[n], and for p < 16
// also the sums over m of the transposed terms; over N_c, in the order of TRE_TB.
__global__ void __launch_bounds__(256) k_trf_desc_adj(TrfArgs A)
{
    __shared__ __attribute__((aligned(16))) double sT[E2][4], sTd[E2][4];
    __shared__ double sDb[E2][AX + 1], sDdb[E2][AX + 1], s_r[4][64], s_rd[4][64];
    const size_t a = blockIdx.x;
    for (int e = threadIdx.x; e < E2 * 4; e += 256) {
        sT[e >> 2][e & 3] = A.T[a * E2 * 4 + e];
        sTd[e >> 2][e & 3] = A.Td[a * E2 * 4 + e];
    }
    for (int e = threadIdx.x; e < DD; e += 256) {
        sDb[e >> 4][e & 15] = A.Db[a * DD + e];
        sDdb[e >> 4][e & 15] = A.Ddb[a * DD + e];
    }
    __syncthreads();
    {
        // the transposed terms: entry (p, k) of the first 16 rows, a quarter of the m each
        const int q = threadIdx.x >> 6, p = (threadIdx.x >> 2) & 15, k = threadIdx.x & 3;
        double tb = 0.0, tdb = 0.0;
        for (int m = 25 * q; m < 25 * q + 25; ++m) {
            tb += sDb[m][p] * sT[m][k] + sDdb[m][p] * sTd[m][k];
            tdb += sDdb[m][p] * sT[m][k];
        }
        s_r[q][threadIdx.x & 63] = tb;
        s_rd[q][threadIdx.x & 63] = tdb;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E2 * 4; e += 256) {
        const int p = e >> 2, k = e & 3;
        double tb = 0.0, tdb = 0.0;
#pragma unroll
        for (int n = 0; n < AX; ++n) {
            tb += sDb[p][n] * sT[n][k] + sDdb[p][n] * sTd[n][k];
            tdb += sDdb[p][n] * sT[n][k];
        }
        if (p < AX)
            for (int q = 0; q < 4; ++q) {
                tb += s_r[q][e];
                tdb += s_rd[q][e];
            }
        int g = 0, u = 0;
        emb_reg3(p, g, u);
        double* o = A.Tb + a * TRE_TB + (16 * (u >> 2) + g + 4 * (u & 3)) * 8 + k;
        o[0] = tb * A.inv_nc;
        o[4] = tdb * A.inv_nc;
    }
    for (int e = threadIdx.x; e < TRE_TB; e += 256) {
        const int r = e >> 3;
        if (emb_feat(3, r & 3, 4 * (r >> 4) + ((r & 15) >> 2)) < 0) A.Tb[a * TRE_TB + e] = 0.0;
    }
}

// ---------------------------------------------------------------------------------------------
// Row GEMM, C = X B and C2 = X2 B, on TM x TM tiles (four waves of a quarter each). LDS rows are padded
// by one double (the 16 rows a wave reads at once fall in distinct banks).
//   TRF_FWD  layer l: X = the layer's input, B = W; epilogue a, y, zd, yd;
//   TRF_BWD  layer l (1 or 2) to the pre-activation of layer l - 1: X = zbar_l, B = W^T;
//   TRF_IN   layer 0 to D: X = zbar_0, B = W^T, stored.
// TM = 64 with 32-deep K-chunks where that fills the device, else 32 with 64-deep ones.
// Bound: the FP64 unit and the reads' latency, two blocks per CU. 12,288 atoms: forward layers 1,445 -> 738
// us, layer 0 to D 608 -> 409, with the edge test moved from the reads to the LDS writes (the products
// waited for the next chunk), two blocks per CU and the column tiles of a row tile on one XCD. 64-wide tiles
// from one block per CU on: below that the 32-wide ones give four times the blocks (192 atoms, forward 28 us
// per layer).
// ---------------------------------------------------------------------------------------------
enum { TRF_FWD, TRF_BWD, TRF_IN };

template <int MODE, int TM>
__global__ void __launch_bounds__(256, 2) k_trf_gemm(TrfArgs A, int l, int nt)
{
    constexpr int KC = TM == 64 ? 32 : 64, IT = TM / 32, NLD = TM * KC / 256;
    __shared__ double sA[TM][KC + 1], sA2[TM][KC + 1], sB[KC][TM + 1];
    // The column tiles of a row tile run on one XCD, one after the other: X is read from memory once.
    const int xi = blockIdx.x >> 3, m0 = (xi / nt * 8 + (blockIdx.x & 7)) * TM, n0 = xi % nt * TM;
    const int ty = blockIdx.y, r0 = A.rows[ty], M = A.rows[ty + 1] - r0;
    if (m0 >= M) return;
    const int K = MODE == TRF_FWD ? tf_in(l) : FW, N = MODE == TRF_IN ? DD : FW;
    const double* X = (MODE != TRF_FWD ? A.zb[l] : l == 0 ? A.D : A.y[l - 1]) + (size_t)r0 * K;
    const double* X2 = (MODE != TRF_FWD ? A.zdb[l] : l == 0 ? A.Dd : A.yd[l - 1]) + (size_t)r0 * K;
    const int64_t net = A.fit0 + ty * TF_NET;
    const double* W = A.theta + net + tf_w(l);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lg = lane >> 4, lc = lane & 15;
    const int wr = wave >> 1, wc = wave & 1;
    double ra[NLD], ra2[NLD], rb[NLD];
    // Reads past the edges are clamped here and cleared on the way to LDS: nothing waits for them before
    // the products of the chunk at hand.
    auto load = [&](int k0) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q, r = idx / KC, kk = idx % KC;
            const size_t o = (size_t)min(m0 + r, M - 1) * K + min(k0 + kk, K - 1);
            ra[q] = X[o];
            ra2[q] = X2[o];
            // B[k][n] = W[k][n] forward, W[n][k] in reverse
            const int kb = MODE == TRF_FWD ? idx / TM : idx % KC, c = MODE == TRF_FWD ? idx % TM : idx / KC;
            const int n = min(n0 + c, N - 1), k2 = min(k0 + kb, K - 1);
            rb[q] = MODE == TRF_FWD ? W[(size_t)k2 * N + n] : W[(size_t)n * K + k2];
        }
        keep_loads();
    };
    d4 acc[IT][IT], acc2[IT][IT];
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int j = 0; j < IT; ++j) acc[i][j] = acc2[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    load(0);
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += KC) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q, r = idx / KC, kk = idx % KC;
            const bool in = m0 + r < M && k0 + kk < K;
            sA[r][kk] = in ? ra[q] : 0.0;
            sA2[r][kk] = in ? ra2[q] : 0.0;
            const int kb = MODE == TRF_FWD ? idx / TM : kk, c = MODE == TRF_FWD ? idx % TM : r;
            sB[kb][c] = k0 + kb < K && n0 + c < N ? rb[q] : 0.0;
        }
        __syncthreads();
        load(min(k0 + KC, K - 1));
#pragma unroll
        for (int ks = 0; ks < KC; ks += 4) {
            double a[IT], a2[IT], b[IT];
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                a[i] = sA[wr * 16 * IT + i * 16 + lc][ks + lg];
                a2[i] = sA2[wr * 16 * IT + i * 16 + lc][ks + lg];
                b[i] = sB[ks + lg][wc * 16 * IT + i * 16 + lc];
            }
#pragma unroll
            for (int i = 0; i < IT; ++i)
#pragma unroll
                for (int j = 0; j < IT; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
                    acc2[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[i], b[j], acc2[i][j], 0, 0, 0);
                }
        }
        __syncthreads();
    }
    const double cE = A.coef->cE;
    const double *bias = W + (size_t)tf_in(l) * FW, *wh = bias + FW;   // (FWD: of layer l)
    const int lb = l - 1;                                              // (BWD: the layer below)
    const double* whb = MODE == TRF_BWD ? A.theta + net + tf_w(lb) + (size_t)tf_in(lb) * FW + FW : nullptr;
    const double *w4 = A.theta + net + tf_w(3), wh4 = w4[FW + 1];
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const int n = n0 + wc * 16 * IT + j * 16 + lc;
        double sb = 0.0, sh = 0.0;
#pragma unroll
        for (int i = 0; i < IT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wr * 16 * IT + i * 16 + lg + 4 * r;
                if (m >= M || n >= N) continue;
                const double c = acc[i][j][r], c2 = acc2[i][j][r];
                const size_t o = (size_t)(r0 + m) * N + n;
                if constexpr (MODE == TRF_FWD) {
                    const double a = tanh(c + bias[n]);
                    const double sx = l == 0 ? 0.0 : X[(size_t)m * K + n], sxd = l == 0 ? 0.0 : X2[(size_t)m * K + n];
                    A.a[l][o] = a;
                    A.y[l][o] = wh[n] * a + sx;
                    A.zd[l][o] = c2;
                    A.yd[l][o] = wh[n] * (1.0 - a * a) * c2 + sxd;
                } else if constexpr (MODE == TRF_BWD) {
                    // adjoint of layer lb's output: the product and the skip of layer l
                    const double yb = c + (l == 2 ? cE * wh4 * w4[n] : A.yb[o]), ydb = c2 + (l == 2 ? wh4 * w4[n] : A.ydb[o]);
                    const double a = A.a[lb][o], gd = 1.0 - a * a, gzy = gd * A.zd[lb][o] * ydb;
                    const double zb = whb[n] * (gd * yb - 2.0 * a * gzy);
                    if (l == 2) {
                        A.yb[o] = yb;
                        A.ydb[o] = ydb;
                    }
                    A.zb[lb][o] = zb;
                    A.zdb[lb][o] = whb[n] * gd * ydb;
                    sb += zb;
                    sh += a * yb + gzy;
                } else {
                    A.Db[o] = c;
                    A.Ddb[o] = c2;
                }
            }
        if constexpr (MODE == TRF_BWD) {
            sb += __shfl_xor(sb, 16);
            sb += __shfl_xor(sb, 32);
            sh += __shfl_xor(sh, 16);
            sh += __shfl_xor(sh, 32);
            if (lg == 0 && n < N) {
                double* gb = A.grad + net + tf_w(lb) + (size_t)tf_in(lb) * FW;
                unsafeAtomicAdd(&gb[n], sb);
                unsafeAtomicAdd(&gb[FW + n], sh);
            }
        }
    }
}

// Output layer o = y3 W4 + b4, E_i = w_hat4 o: the adjoints of its input are cE w_hat4 W4 and w_hat4 W4 for
// every row; those of layer 3's pre-activation, and the sums of both layers' vectors. A thread per
// column, OUT_ROWS rows per block.
constexpr int OUT_ROWS = 16;
__global__ void __launch_bounds__(256) k_trf_out(TrfArgs A)
{
    const int ty = blockIdx.y, r0 = A.rows[ty], M = A.rows[ty + 1] - r0;
    const int m0 = blockIdx.x * OUT_ROWS, m1 = min(M, m0 + OUT_ROWS), n = threadIdx.x;
    if (m0 >= M) return;
    const int64_t net = A.fit0 + ty * TF_NET;
    const double *w4 = A.theta + net + tf_w(3), b4 = w4[FW], wh4 = w4[FW + 1], cE = A.coef->cE;
    double* g4 = A.grad + net + tf_w(3);
    const int64_t v3 = net + tf_w(2) + (int64_t)FW * FW;   // b3, w_hat3
    double so = 0.0;
    if (n < FW) {
        const double w = w4[n], wh = A.theta[v3 + FW + n], ydb = wh4 * w, yb = cE * ydb;
        double s1 = 0.0, s2 = 0.0, sb = 0.0, sh = 0.0;
#pragma unroll 4
        for (int m = m0; m < m1; ++m) {
            const size_t o = (size_t)(r0 + m) * FW + n;
            const double a = A.a[2][o], gd = 1.0 - a * a, gzy = gd * A.zd[2][o] * ydb;
            const double zb = wh * (gd * yb - 2.0 * a * gzy);
            s1 += A.y[2][o];
            s2 += A.yd[2][o];
            A.zb[2][o] = zb;
            A.zdb[2][o] = wh * gd * ydb;
            sb += zb;
            sh += a * yb + gzy;
        }
        unsafeAtomicAdd(&g4[n], wh4 * (cE * s1 + s2));
        unsafeAtomicAdd(&A.grad[v3 + n], sb);
        unsafeAtomicAdd(&A.grad[v3 + FW + n], sh);
        so = w * (cE * s1 + s2);   // this column's share of sum over the rows of cE o + odot
    }
    __shared__ double s_o[4];
    for (int k = 1; k < 64; k <<= 1) so += __shfl_xor(so, k);
    if ((threadIdx.x & 63) == 0) s_o[threadIdx.x >> 6] = so;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsafeAtomicAdd(&g4[FW], cE * wh4 * (m1 - m0));
        unsafeAtomicAdd(&g4[FW + 1], s_o[0] + s_o[1] + s_o[2] + s_o[3] + cE * b4 * (m1 - m0));
    }
}

// Weight gradients of the three hidden layers, Wbar = X^T Zb + Xd^T Zdb over the rows: 64 x 64 tiles, the
// rows in ranges; FP64 atomics into the gradient. Bound: the FP64 unit (350 us of products at 12,288 atoms)
// and the latency of the rows' reads, two blocks per CU: 552 us, 1,031 with the tiles of a range on all XCDs
// and the edge test on arrival (see k_trf_gemm).
constexpr int WG_T1 = (DD / 64) * 4, WG_T2 = 16, WG_TILES = WG_T1 + 2 * WG_T2;
__global__ void __launch_bounds__(256, 2) k_trf_wgrad(TrfArgs A, int splits, int grp)
{
    constexpr int TB = 64, KC = 16, NLD = TB * KC / 256;
    __shared__ double sA[KC][TB + 1], sB[KC][TB + 1], sA2[KC][TB + 1], sB2[KC][TB + 1];
    const int ty = blockIdx.y, row0 = A.rows[ty], M = A.rows[ty + 1] - row0;
    const int per = ((M + splits - 1) / splits + KC - 1) / KC * KC;
    const int xi = blockIdx.x / grp, r0 = (xi / WG_TILES * grp + blockIdx.x % grp) * per, r1 = min(M, r0 + per);
    if (r0 >= r1) return;
    const int t = xi % WG_TILES, l = t < WG_T1 ? 0 : t < WG_T1 + WG_T2 ? 1 : 2, tl = l == 0 ? t : (t - WG_T1) % WG_T2;
    const int K = tf_in(l), k0 = (tl >> 2) * TB, n0 = (tl & 3) * TB;
    const double *X = (l == 0 ? A.D : A.y[l - 1]) + (size_t)row0 * K, *X2 = (l == 0 ? A.Dd : A.yd[l - 1]) + (size_t)row0 * K;
    const double *Z = A.zb[l] + (size_t)row0 * FW, *Z2 = A.zdb[l] + (size_t)row0 * FW;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lg = lane >> 4, lc = lane & 15;
    const int wr = wave >> 1, wc = wave & 1;
    double ra[NLD], ra2[NLD], rb[NLD], rb2[NLD];
    auto load = [&](int m0) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q, m = m0 + (idx >> 6), c = idx & 63;
            const size_t mm = min(m, r1 - 1), ok = mm * K + min(k0 + c, K - 1), on = mm * FW + min(n0 + c, FW - 1);
            ra[q] = X[ok];
            ra2[q] = X2[ok];
            rb[q] = Z[on];
            rb2[q] = Z2[on];
        }
        keep_loads();
    };
    d4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    load(r0);
#pragma unroll 1
    for (int m0 = r0; m0 < r1; m0 += KC) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q, mm = idx >> 6, c = idx & 63;
            const bool kin = m0 + mm < r1 && k0 + c < K, nin = m0 + mm < r1 && n0 + c < FW;
            sA[mm][c] = kin ? ra[q] : 0.0;
            sA2[mm][c] = kin ? ra2[q] : 0.0;
            sB[mm][c] = nin ? rb[q] : 0.0;
            sB2[mm][c] = nin ? rb2[q] : 0.0;
        }
        __syncthreads();
        load(m0 + KC);
#pragma unroll
        for (int ks = 0; ks < KC; ks += 4) {
            double a[2], b[2], a2[2], b2[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = sA[ks + lg][wr * 32 + i * 16 + lc];
                b[i] = sB[ks + lg][wc * 32 + i * 16 + lc];
                a2[i] = sA2[ks + lg][wr * 32 + i * 16 + lc];
                b2[i] = sB2[ks + lg][wc * 32 + i * 16 + lc];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[i], b2[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();
    }
    double* G = A.grad + A.fit0 + ty * TF_NET + tf_w(l);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = k0 + wr * 32 + i * 16 + lg + 4 * r, n = n0 + wc * 32 + j * 16 + lc;
                if (k < K && n < FW) unsafeAtomicAdd(&G[(size_t)k * FW + n], acc[i][j][r]);
            }
}

template <int MODE>
void gemm(const TrfArgs& a, int l, int ncu, hipStream_t s)
{
    const int N = MODE == TRF_IN ? DD : FW;
    const int64_t b64 = (int64_t)((N + 63) / 64) * ((a.n + 63) / 64);
    auto grid = [&](int tm) { return dim3((a.max_rows + 8 * tm - 1) / (8 * tm) * 8 * ((N + tm - 1) / tm), a.nt); };
    if (b64 >= (ncu > 0 ? ncu : 256))
        hipLaunchKernelGGL((k_trf_gemm<MODE, 64>), grid(64), dim3(256), 0, s, a, l, (N + 63) / 64);
    else
        hipLaunchKernelGGL((k_trf_gemm<MODE, 32>), grid(32), dim3(256), 0, s, a, l, (N + 31) / 32);
}

// ---------------------------------------------------------------------------------------------
// Loss
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_tr_direction(TrLossArgs A)
{
    __shared__ double s_p[4];
    const int k = blockIdx.x * 256 + threadIdx.x;
    double lf = 0.0;
    if (k < A.n) {
        const double q = A.q ? A.q[k] : 1.0;
        for (int c = 0; c < 3; ++c) {
            double v = 0.0;
            if (A.fl) {
                const double d = A.F[3 * (size_t)k + c] - A.fl[3 * (size_t)k + c];
                lf += q * d * d;
                v = -2.0 * A.pf * q * d / (3.0 * A.n) * A.weight;
            }
            A.vdir[3 * (size_t)k + c] = v;
        }
    }
    for (int m = 1; m < 64; m <<= 1) lf += __shfl_xor(lf, m);
    if ((threadIdx.x & 63) == 0) s_p[threadIdx.x >> 6] = lf;
    __syncthreads();
    if (threadIdx.x == 0) A.part[blockIdx.x] = s_p[0] + s_p[1] + s_p[2] + s_p[3];
}

__global__ void __launch_bounds__(64) k_tr_loss(TrLossArgs A, int nblocks)
{
    double lf = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 64) lf += A.part[b];
    for (int m = 1; m < 64; m <<= 1) lf += __shfl_xor(lf, m);
    if (threadIdx.x) return;
    TrCoef* c = A.coef;
    const double N = A.n;
    double le = 0.0, lv = 0.0;
    c->cE = 0.0;
    if (A.has_e) {
        const double d = c->ev[0] - A.el;
        le = d * d / N;
        c->cE = 2.0 * A.pe * d / N * A.weight;
    }
    for (int k = 0; k < 9; ++k) {
        c->CV[k] = 0.0;
        if (A.has_v) {
            const double d = c->ev[1 + k] - A.vl[k];
            lv += d * d;
            c->CV[k] = -2.0 * A.pv * d / (9.0 * N) * A.weight;
        }
    }
    lv /= 9.0 * N;
    lf /= 3.0 * N;
    c->loss[0] = A.pe * le + A.pf * lf + A.pv * lv;
    c->loss[1] = le;
    c->loss[2] = lf;
    c->loss[3] = lv;
}

// ---------------------------------------------------------------------------------------------
// Packing, Adam
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_tr_map(const double* packed, int64_t n, int* map)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) map[i] = (int)packed[i] - 1;
}

__global__ void __launch_bounds__(256) k_tr_pack(const double* theta, const int* map, int64_t n, double* packed)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) packed[i] = map[i] >= 0 ? theta[map[i]] : 0.0;
}

__global__ void __launch_bounds__(256) k_tr_adam(int64_t n, double* th, double* g, double* m, double* v, double lr,
                                                 double b1, double b2, double eps, double c1, double c2)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double gi = g[i];
        const double mi = b1 * m[i] + (1.0 - b1) * gi, vi = b2 * v[i] + (1.0 - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        th[i] -= lr * (mi / c1) / (sqrt(vi / c2) + eps);
        g[i] = 0.0;
    }
}

}  // namespace

void trf_run(const TrfArgs& a, int ncu, hipStream_t s)
{
    hipLaunchKernelGGL(k_trf_desc, dim3(a.n), dim3(256), 0, s, a);
    for (int l = 0; l < 3; ++l) gemm<TRF_FWD>(a, l, ncu, s);
    hipLaunchKernelGGL(k_trf_out, dim3((a.max_rows + OUT_ROWS - 1) / OUT_ROWS, a.nt), dim3(256), 0, s, a);
    gemm<TRF_BWD>(a, 2, ncu, s);
    gemm<TRF_BWD>(a, 1, ncu, s);
    gemm<TRF_IN>(a, 0, ncu, s);
    // Row ranges in groups of 8: all tiles of a range on one XCD, which reads its rows once. Short ranges
    // would only add atomics: one range below 2048 rows.
    const int grp = a.max_rows < 2048 ? 1 : 8;
    const int splits = grp * (int)std::max<int64_t>(1, std::min<int64_t>(a.max_rows / (256 * grp), 4LL * ncu / (WG_TILES * grp * a.nt)));
    hipLaunchKernelGGL(k_trf_wgrad, dim3(WG_TILES * splits, a.nt), dim3(256), 0, s, a, splits, grp);
    hipLaunchKernelGGL(k_trf_desc_adj, dim3(a.n), dim3(256), 0, s, a);
}

int tr_loss_blocks(int n) { return (n + 255) / 256; }

void tr_loss(const TrLossArgs& a, hipStream_t s)
{
    const int nb = tr_loss_blocks(a.n);
    hipLaunchKernelGGL(k_tr_direction, dim3(nb), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_tr_loss, dim3(1), dim3(64), 0, s, a, nb);
}

void tr_map(const double* packed, int64_t n, int* map, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_tr_map, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, packed, n, map);
}

void tr_pack(const double* theta, const int* map, int64_t n, double* packed, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_tr_pack, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, map, n, packed);
}

void tr_adam(int64_t n, double* theta, double* g, double* m, double* v, double lr, double b1, double b2, double eps,
             double c1, double c2, hipStream_t s)
{
    if (n <= 0) return;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_tr_adam, dim3(blocks), dim3(256), 0, s, n, theta, g, m, v, lr, b1, b2, eps, c1, c2);
}

}  // namespace dpk
