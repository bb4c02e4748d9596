// kernels_tre.hip -- training-mode backward through the embedding nets (Sec. II.B), FP64.
//
// The loss gradient is the derivative of cE E + sum_ij g_ij . rdot_ij (dpk_train.h): a forward-mode
// tangent along the pair displacements rdot_ij, then reverse mode through the model and its tangent.
// The net's input is the scalar s, so its tangent is sdot times the unit tangent d/ds.
//   k_tre_tan    Td = N_c^-1 sum_j (sdot Gd_j (x) R_j + G_j (x) Rdot_j), with G and Gd = dG/ds
//                re-evaluated per chunk of 16 neighbours as in the inference kernels;
//   k_tre_adj    per chunk: the adjoints (ybar, ydbar) of G and sdot Gd from (Tbar, Tdbar), reverse
//                through the three layers, z = x W + b, a = tanh z, y = w_hat a + skip(x):
//                  zbar = w_hat (1 - a^2) ybar - 2 w_hat a (1 - a^2) zdot ydbar, zdbar = w_hat (1 - a^2) ydbar,
//                  hbar = a ybar + (1 - a^2) zdot ydbar (w_hat's gradient),
//                  xbar = W zbar + skip^T ybar, xdbar = W zdbar + skip^T ydbar;
//                the operands of the weight gradients go to memory as they stand in registers;
//   k_tre_wgrad  Wbar_l = sum over the pairs of x zbar^T + xdot zdbar^T, and bbar_l as the row of a
//                padding feature of x that is set to 1.
// Layouts as in the embedding kernels: features in registers and lane groups, one pair per lane column,
// in the skip-aligned order, so every skip and its transpose stay in a lane. One wave per SIMD (up to
// 512 registers: the layers' values, the running adjoints and the w_hat sums).
// Bound: the FP64 unit (k_tre_tan 252, k_tre_adj 532 products of 65 cycles per chunk, k_tre_wgrad 320, of
// which 32 are waves 3 and 7 repeating their tile of W3, whose sum is dropped; plus the vector work, with one
// wave per SIMD to hide its latencies) and, for k_tre_wgrad, reading the 65 KiB per chunk that k_tre_adj
// wrote (4.2 TB/s). 12,288 atoms (73,800 chunks), the means of several runs: k_tre_tan 1,110-1,200 us,
// k_tre_adj 1,990-2,060, k_tre_wgrad 1,130-1,180; 192 atoms 43, 90 and 80. With whole atoms per wave, and one
// copy of the gradient, 192 atoms took 106, 239 and 106.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dpk_device.h"
#include "dpk_internal.h"
#include "dpk_launch.h"
#include "dpk_train.h"
#include "emb_device.h"

namespace dpk {
namespace {

typedef PF64 P;
typedef EmbCfg<PF64> Cfg;
typedef P::frag frag;
typedef double d2 __attribute__((ext_vector_type(2)));
constexpr int NW = 4;                          // waves per block, one per SIMD
constexpr int NU1 = Cfg::NU1, NU2 = Cfg::NU2;  // registers in use of layers 1 and 2 (of 8 and 16)
// Padding registers whose lane group 0 carries the constant 1 of the bias gradients
constexpr int ONE1 = NU1, ONE2 = NU2;
static_assert(ONE1 < 8 && ONE2 < 16, "padding registers");
// One chunk's operands: registers [u][64 lanes] of each quantity
// (padding registers are left out where the rows or columns they make are not read: a tile that runs over
// into the next quantity fills such rows only)
constexpr int D_Z3 = 0, D_ZD3 = 28, D_Z2 = 56, D_ZD2 = D_Z2 + NU2, D_Y2 = D_ZD2 + NU2, D_YD2 = D_Y2 + NU2 + 1,
              D_Y1 = D_YD2 + NU2 + 1, D_YD1 = D_Y1 + 8;
static_assert((D_YD1 + 8) * 64 == TRE_CHUNK, "operand block of a chunk");
// Offsets inside one net's block of the parameter vector
constexpr int G_W1 = 0, G_B1 = 25, G_H1 = 50, G_W2 = 75, G_B2 = G_W2 + E0 * E1, G_H2 = G_B2 + E1, G_W3 = G_H2 + E1,
              G_B3 = G_W3 + E1 * E2, G_H3 = G_B3 + E2, G_NET = TRE_NET;
static_assert(G_H3 + E2 == G_NET, "parameters of a net");

// Environment row and its tangent of one pair: r_ij, rdot_ij = v_j - v_i + CV r_ij.
struct Pair {
    double s, sd, R[4], Rd[4];
};
__device__ __forceinline__ void pair_env(const EmbArgs& A, const TrCoef* co, double inv_w, double x, double y, double z,
                                         const double* vj, const double* vi, bool valid, Pair& o)
{
    o.s = o.sd = 0.0;
    for (int k = 0; k < 4; ++k) o.R[k] = o.Rd[k] = 0.0;
    if (!valid) return;
    const double r = sqrt(x * x + y * y + z * z), ir = 1.0 / r;
    double s, ds, d[3];
    switch_fn(r, ir, A.rs, A.rc, inv_w, s, ds);
    const double sr = s * ir, ux = x * ir, uy = y * ir, uz = z * ir;
    for (int k = 0; k < 3; ++k) d[k] = vj[k] - vi[k] + co->CV[3 * k] * x + co->CV[3 * k + 1] * y + co->CV[3 * k + 2] * z;
    const double q = ux * d[0] + uy * d[1] + uz * d[2], c = (ds - sr) * q;   // q: rate of change of r
    o.s = s;
    o.sd = ds * q;
    o.R[0] = s; o.R[1] = sr * x; o.R[2] = sr * y; o.R[3] = sr * z;
    o.Rd[0] = o.sd; o.Rd[1] = c * ux + sr * d[0]; o.Rd[2] = c * uy + sr * d[1]; o.Rd[3] = c * uz + sr * d[2];
}

// Per-wave walk over the chunks [c, end) of one net. The items of the next chunk are loaded while the
// current one is worked on, in two steps, since vdir_j needs the neighbour's index: fetch() at its start,
// fetch_v() in its middle. Nothing then waits for a load behind the stores of the current chunk (the
// counter of vector memory operations is in order). The map is read one chunk further ahead.
struct TreWalk {
    int c, end;
    int4 m;                      // the chunk's map entry
    double x, y, z, vj[3], vi[3];
    int4 m1, m2;                 // of the next chunk and the one after it
    double nx, ny, nz, nvj[3], nvi[3];
    int nj;
    __device__ __forceinline__ int4 map(const TreArgs& K, int k) const { return K.cmap[min(k, end - 1)]; }
    __device__ __forceinline__ int4 uniform(int4 v) const
    {
        return int4{__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
                    __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w)};
    }
    // (a lane past its atom's neighbours reads another slot of the atom's row, which holds finite values)
    __device__ __forceinline__ void fetch(const TreArgs& K, int tj, int c16)
    {
        m1 = uniform(m2);
        m2 = map(K, c + 2);
        const size_t slot = (size_t)m1.x * K.e.nc + min(K.e.off[tj] + m1.z + c16, K.e.nc - 1);
        const double* v = K.e.nl_r + 3 * slot;
        nx = v[0];
        ny = v[1];
        nz = v[2];
        nj = K.e.nl_j[slot];
        keep_loads();
    }
    __device__ __forceinline__ void fetch_v(const TreArgs& K)
    {
        for (int k = 0; k < 3; ++k) {
            nvj[k] = K.vdir[3 * (size_t)max(nj, 0) + k];
            nvi[k] = K.vdir[3 * (size_t)m1.y + k];
        }
        keep_loads();
    }
    __device__ __forceinline__ void take()
    {
        m = m1;
        x = nx;
        y = ny;
        z = nz;
        for (int k = 0; k < 3; ++k) {
            vj[k] = nvj[k];
            vi[k] = nvi[k];
        }
    }
    // c < end
    __device__ __forceinline__ void start(const TreArgs& K, int tj, int c16, int lo, int hi)
    {
        c = lo - 1;
        end = hi;
        m2 = map(K, lo);
        fetch(K, tj, c16);
        fetch_v(K);
        c = lo;
        take();
    }
};

// Where this block adds its sums of a net. All blocks add to every address of a net, and adds to one cache
// line take turns: on one copy of the gradient they took most of k_tre_adj and k_tre_wgrad of a small frame
// (192 atoms 187 and 110 us; 89 and 80 on 32 copies, each of the blocks of one XCD only).
__device__ __forceinline__ double* replica(const TreArgs& K, int net)
{
    return K.rep + ((size_t)(blockIdx.x % K.nrep) * K.nets + net) * G_NET;
}

// The chunk range of wave `wave` of this block in the net (ti, tj); false if the block has none there.
__device__ __forceinline__ bool net_range(const TreArgs& K, int ti, int tj, int wave, int& lo, int& hi)
{
    const int nt = K.e.ntypes, n = K.e.natoms, side = K.e.type_one_side;
    const int64_t ld = n + 1, total = K.coff[(nt - 1) * ld + n];
    const int b0 = (int)(total * blockIdx.x / gridDim.x), b1 = (int)(total * (blockIdx.x + 1) / gridDim.x);
    const int c0 = max(b0, K.coff[tj * ld + (side ? 0 : K.toff[ti])]), c1 = min(b1, K.coff[tj * ld + (side ? n : K.toff[ti + 1])]);
    if (c0 >= c1) return false;
    lo = c0 + (int)((int64_t)(c1 - c0) * wave / NW);
    hi = c0 + (int)((int64_t)(c1 - c0) * (wave + 1) / NW);
    return true;
}

__global__ void __launch_bounds__(64 * NW, 1) k_tre_tan(TreArgs K)
{
    const EmbArgs& A = K.e;
    __shared__ double s_vec[EVEC];
    __shared__ __attribute__((aligned(16))) char s_w2[N2P * Cfg::ROW2];
    __shared__ __attribute__((aligned(16))) char s_w3[N3P * Cfg::ROW3];
    // layer 2 and its unit tangent, neighbour-major, for the skip into the untransposed layer 3
    __shared__ double s_z2[NW][2][16][Z2S];
    __shared__ __attribute__((aligned(16))) double s_R[NW][16][10];   // R, Rdot, sdot (a pad) per pair
    __shared__ double s_th[TH_N];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const double inv_w = 1.0 / (A.rc - A.rs);
    tanh_tab_fill(s_th);
    for (int tj = 0; tj < A.ntypes; ++tj)
        for (int ti = 0; ti < (A.type_one_side ? 1 : A.ntypes); ++ti) {
            int lo, hi;
            if (!net_range(K, ti, tj, wave, lo, hi)) continue;   // (uniform over the block)
            __syncthreads();
            stage_net<P>(A, A.type_one_side ? tj : ti * A.ntypes + tj, s_vec, s_w2, s_w3);
            __syncthreads();
            if (lo >= hi) continue;
            TreWalk w;
            w.start(K, tj, c16, lo, hi);
            d4 Tacc[7];
            for (int t = 0; t < 7; ++t) zero4(Tacc[t]);
            for (;;) {
                w.fetch(K, tj, c16);
                Pair pr;
                pair_env(A, K.coef, inv_w, w.x, w.y, w.z, w.vj, w.vi, w.m.z + c16 < w.m.w, pr);
                const double s = pr.s;
                wave_sync();
                if (g == 0) {
                    for (int k = 0; k < 4; ++k) {
                        s_R[wave][c16][k] = pr.R[k];
                        s_R[wave][c16][4 + k] = pr.Rd[k];
                    }
                    s_R[wave][c16][8] = pr.sd;
                }
                frag B1[Cfg::NC1], B1d[Cfg::NC1];
                double z1[8], z1d[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    z1[u] = z1d[u] = 0;
                    if (u >= NU1) continue;
                    const int k = P::kidx(u / 4, g, u % 4);
                    const double w1 = s_vec[EV_W1 + k], wh = s_vec[EV_WH1 + k];
                    const double t1 = P::act(s * w1 + s_vec[EV_B1 + k], s_th);
                    z1[u] = wh * t1;
                    z1d[u] = wh * (1 - t1 * t1) * w1;
                }
#pragma unroll
                for (int c = 0; c < Cfg::NC1; ++c) {
                    B1[c] = P::make(&z1[4 * c]);
                    B1d[c] = P::make(&z1d[4 * c]);
                }
                d4 acc2[4], acc2d[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    zero4(acc2[t]);
                    zero4(acc2d[t]);
#pragma unroll
                    for (int c = 0; c < Cfg::NC1; ++c) {
                        const frag W = lds_frag<P>(s_w2, Cfg::ROW2, 16 * t + c16, 4 * c + g);
                        P::mma(acc2[t], W, B1[c], Cfg::ku(NU1, c));
                        P::mma(acc2d[t], W, B1d[c], Cfg::ku(NU1, c));
                    }
                }
                wave_sync();
                double zt[16], ztd[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    zt[u] = ztd[u] = 0;
                    if (u >= NU2) continue;
                    const int n = 16 * (u >> 2) + P::orow(g, u & 3);
                    const double t2 = P::act_b(acc2[u >> 2][u & 3], s_vec[EV_B2 + n], s_th), wh = s_vec[EV_WH2 + n];
                    zt[u] = wh * t2 + z1[u >> 1];
                    ztd[u] = wh * (1 - t2 * t2) * acc2d[u >> 2][u & 3] + z1d[u >> 1];
                    s_z2[wave][0][c16][n] = zt[u];
                    s_z2[wave][1][c16][n] = ztd[u];
                }
                frag A3[Cfg::NC2], A3d[Cfg::NC2];
#pragma unroll
                for (int c = 0; c < Cfg::NC2; ++c) {
                    A3[c] = P::make(&zt[4 * c]);
                    A3d[c] = P::make(&ztd[4 * c]);
                }
                w.fetch_v(K);
                auto mm3 = [&](int tm, d4& o, d4& od) {
                    zero4(o);
                    zero4(od);
#pragma unroll
                    for (int c = 0; c < Cfg::NC2; ++c) {
                        const frag Bw = lds_frag<P>(s_w3, Cfg::ROW3, 16 * tm + c16, 4 * c + g);
                        P::mma(o, A3[c], Bw, Cfg::ku(NU2, c));
                        P::mma(od, A3d[c], Bw, Cfg::ku(NU2, c));
                    }
                };
                const int gc = P::ogrp(c16), rc = P::oreg(c16);
                auto epi3 = [&](int tm, const d4& o, const d4& od) {
                    const int m = 16 * tm + c16;
                    const int u2 = (4 * tm + rc) >> 1;
                    const int n2 = 16 * (u2 >> 2) + P::orow(gc, u2 & 3);
                    const double wh = s_vec[EV_WH3 + m], bb = s_vec[EV_B3 + m];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int q = P::orow(g, r);

                        const double t3 = P::act_b(o[r], bb, s_th);
                        const double G = wh * t3 + s_z2[wave][0][q][n2];
                        const double Gd = (wh * (1 - t3 * t3) * od[r] + s_z2[wave][1][q][n2]) * s_R[wave][q][8];
#pragma unroll
                        for (int k = 0; k < 4; ++k) Tacc[tm][k] += Gd * s_R[wave][q][k] + G * s_R[wave][q][4 + k];
                    }
                };
                wave_sync();
                d4 a3[2], a3d[2];
                mm3(0, a3[0], a3d[0]);
#pragma unroll
                for (int tm = 0; tm < 7; ++tm) {
                    if (tm + 1 < 7) mm3(tm + 1, a3[(tm + 1) & 1], a3d[(tm + 1) & 1]);
                    epi3(tm, a3[tm & 1], a3d[tm & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const bool more = w.c + 1 < w.end;
                if (!more || w.m1.x != w.m.x) {
                    // the atom's (or the wave's) last chunk here: its share of Td
#pragma unroll
                    for (int tm = 0; tm < 7; ++tm) {
                        const double tv[4] = {Tacc[tm][0], Tacc[tm][1], Tacc[tm][2], Tacc[tm][3]};
                        const double v = sum_groups4(tv);
                        const int f = emb_feat(3, gc, 4 * tm + rc);
                        if (f >= 0) unsafeAtomicAdd(&K.Td[((size_t)w.m.x * E2 + f) * 4 + ksel(g)], v * A.inv_nc);
                        zero4(Tacc[tm]);
                    }
                }
                if (!more) break;
                ++w.c;
                w.take();
            }
        }
}

// A fragment of W itself (rows = the layer's inputs) from the staged W^T: input 16 t + c16, outputs
// 16 c + orow(g, v) (row pitch rowb, K order of the staged rows).
__device__ __forceinline__ frag lds_frag_t(const char* base, int rowb, int t, int c, int g, int c16)
{
    const char* p = base + (16 * c + g) * rowb + (4 * t + (c16 & 3)) * P::GB + (c16 >> 2) * 8;
    frag f;
#pragma unroll
    for (int v = 0; v < 4; ++v) f.v[v] = *reinterpret_cast<const double*>(p + 4 * v * rowb);
    return f;
}

__global__ void __launch_bounds__(64 * NW, 1) k_tre_adj(TreArgs K)
{
    const EmbArgs& A = K.e;
    __shared__ double s_vec[EVEC];
    __shared__ __attribute__((aligned(16))) char s_w2[N2P * Cfg::ROW2];
    __shared__ __attribute__((aligned(16))) char s_w3[N3P * Cfg::ROW3];
    // Tbar and Tdbar of the wave's current atom by layer-3 row position (padding rows zero)
    __shared__ __attribute__((aligned(16))) double s_tb[NW][N3P][8];
    __shared__ double s_th[TH_N];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const double inv_w = 1.0 / (A.rc - A.rs);
    tanh_tab_fill(s_th);
    for (int tj = 0; tj < A.ntypes; ++tj)
        for (int ti = 0; ti < (A.type_one_side ? 1 : A.ntypes); ++ti) {
            const int net = A.type_one_side ? tj : ti * A.ntypes + tj;
            int lo, hi;
            if (!net_range(K, ti, tj, wave, lo, hi)) continue;   // (uniform over the block)
            __syncthreads();
            stage_net<P>(A, net, s_vec, s_w2, s_w3);
            __syncthreads();
            if (lo >= hi) continue;
            TreWalk w;
            w.start(K, tj, c16, lo, hi);
            int atom = -1;   // whose adjoints s_tb holds
            // sums over the wave's pairs of this net: w_hat's gradient of every layer, and W1's and b1's
            double h3[28], h2[NU2], h1[NU1], gw1[NU1], gb1[NU1];
#pragma unroll
            for (int u = 0; u < 28; ++u) h3[u] = 0.0;
#pragma unroll
            for (int u = 0; u < NU2; ++u) h2[u] = 0.0;
#pragma unroll
            for (int u = 0; u < NU1; ++u) h1[u] = gw1[u] = gb1[u] = 0.0;
            while (w.c < w.end) {
                wave_sync();
                if (w.m.x != atom) {
                    atom = w.m.x;
                    const double2* tb = reinterpret_cast<const double2*>(K.Tb + (size_t)atom * TRE_TB);
                    double2 v[TRE_TB / 128];
#pragma unroll
                    for (int q = 0; q < TRE_TB / 128; ++q) v[q] = tb[lane + 64 * q];
#pragma unroll
                    for (int q = 0; q < TRE_TB / 128; ++q) reinterpret_cast<double2*>(&s_tb[wave][0][0])[lane + 64 * q] = v[q];
                    wave_sync();
                }
                int lo = lane;
                asm volatile("" : "+v"(lo));   // (or the 17 store offsets are kept in registers over the loop)
                double* dump = K.dump + (size_t)w.c * TRE_CHUNK + lo;
                auto put = [&](int at, int u, double v) { __builtin_nontemporal_store(v, &dump[(at + u) * 64]); };
                Pair pr;
                pair_env(A, K.coef, inv_w, w.x, w.y, w.z, w.vj, w.vi, w.m.z + c16 < w.m.w, pr);
                const double s = pr.s, sd = pr.sd;
                // forward: the layers' tanh outputs and unit tangents
                double t1[8], z1[8], z1d[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    t1[u] = z1[u] = z1d[u] = 0;
                    if (u < NU1) {
                        const int k = P::kidx(u / 4, g, u % 4);
                        const double w1 = s_vec[EV_W1 + k], wh = s_vec[EV_WH1 + k];
                        t1[u] = P::act(s * w1 + s_vec[EV_B1 + k], s_th);
                        z1[u] = wh * t1[u];
                        z1d[u] = wh * (1 - t1[u] * t1[u]) * w1;
                    }
                    put(D_Y1, u, u == ONE1 ? (g == 0 ? 1.0 : 0.0) : z1[u]);
                    put(D_YD1, u, sd * z1d[u]);
                }
                d4 acc2[4], zd2[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    zero4(acc2[t]);
                    zero4(zd2[t]);
#pragma unroll
                    for (int c = 0; c < Cfg::NC1; ++c) {
                        const frag W = lds_frag<P>(s_w2, Cfg::ROW2, 16 * t + c16, 4 * c + g);
                        P::mma(acc2[t], W, P::make(&z1[4 * c]), Cfg::ku(NU1, c));
                        P::mma(zd2[t], W, P::make(&z1d[4 * c]), Cfg::ku(NU1, c));
                    }
                }
                double t2[16], zt[16], ztd[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    t2[u] = zt[u] = ztd[u] = 0;
                    if (u < NU2) {
                        const int n = 16 * (u >> 2) + P::orow(g, u & 3);
                        const double wh = s_vec[EV_WH2 + n];
                        t2[u] = P::act_b(acc2[u >> 2][u & 3], s_vec[EV_B2 + n], s_th);
                        zt[u] = wh * t2[u] + z1[u >> 1];
                        ztd[u] = wh * (1 - t2[u] * t2[u]) * zd2[u >> 2][u & 3] + z1d[u >> 1];
                    }
                    if (u > ONE2) continue;
                    put(D_Y2, u, u == ONE2 ? (g == 0 ? 1.0 : 0.0) : zt[u]);
                    put(D_YD2, u, sd * ztd[u]);
                }
                auto mm3 = [&](int tm, d4& o, d4& od) {
                    zero4(o);
                    zero4(od);
#pragma unroll
                    for (int c = 0; c < Cfg::NC2; ++c) {
                        const frag W = lds_frag<P>(s_w3, Cfg::ROW3, 16 * tm + c16, 4 * c + g);
                        P::mma(o, W, P::make(&zt[4 * c]), Cfg::ku(NU2, c));
                        P::mma(od, W, P::make(&ztd[4 * c]), Cfg::ku(NU2, c));
                    }
                };
                // layer 3: adjoints of the output, of the pre-activation, and the products with W3
                d4 xb[4], xdb[4];   // adjoints of layer 2's output; the skip is added to the accumulators
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    zero4(xb[t]);
                    zero4(xdb[t]);
                }
                auto epi3 = [&](int tm, const d4& o, const d4& od) {
                    d4 zb, zdb;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int u = 4 * tm + r, m = 16 * tm + P::orow(g, r);
                        const double* tb = s_tb[wave][m];
                        double yb = 0.0, ydb = 0.0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            yb += tb[k] * pr.R[k] + tb[4 + k] * pr.Rd[k];
                            ydb += tb[4 + k] * pr.R[k];
                        }
                        const double t3 = P::act_b(o[r], s_vec[EV_B3 + m], s_th), gd = 1 - t3 * t3, wh = s_vec[EV_WH3 + m];
                        const double gzy = gd * (sd * od[r]) * ydb;
                        zb[r] = wh * (gd * yb - 2 * t3 * gzy);
                        zdb[r] = wh * gd * ydb;
                        h3[u] += t3 * yb + gzy;
                        put(D_Z3, u, zb[r]);
                        put(D_ZD3, u, zdb[r]);
                        xb[u >> 3][(u >> 1) & 3] += yb;
                        xdb[u >> 3][(u >> 1) & 3] += ydb;
                    }
                    frag fb, fdb;
                    fb.v = zb;
                    fdb.v = zdb;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const frag W = lds_frag_t(s_w3, Cfg::ROW3, t, tm, g, c16);
                        P::mma(xb[t], W, fb);
                        P::mma(xdb[t], W, fdb);
                    }
                };
                d4 a3[2], a3d[2];
                mm3(0, a3[0], a3d[0]);
#pragma unroll
                for (int tm = 0; tm < 7; ++tm) {
                    if (tm + 1 < 7) mm3(tm + 1, a3[(tm + 1) & 1], a3d[(tm + 1) & 1]);
                    if (tm == 4) w.fetch(K, tj, c16);
                    epi3(tm, a3[tm & 1], a3d[tm & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                w.fetch_v(K);
                // layer 2
                d4 xb1[2], xdb1[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    zero4(xb1[t]);
                    zero4(xdb1[t]);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    d4 zb, zdb;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int u = 4 * c + r;
                        zb[r] = zdb[r] = 0.0;
                        if (u < NU2) {
                            const int n = 16 * c + P::orow(g, r);
                            const double yb = xb[c][r], ydb = xdb[c][r];
                            const double gd = 1 - t2[u] * t2[u], wh = s_vec[EV_WH2 + n], gzy = gd * (sd * zd2[c][r]) * ydb;
                            zb[r] = wh * (gd * yb - 2 * t2[u] * gzy);
                            zdb[r] = wh * gd * ydb;
                            h2[u] += t2[u] * yb + gzy;
                            xb1[u >> 3][(u >> 1) & 3] += yb;
                            xdb1[u >> 3][(u >> 1) & 3] += ydb;
                        }
                        if (u >= NU2) continue;
                        put(D_Z2, u, zb[r]);
                        put(D_ZD2, u, zdb[r]);
                    }
                    frag fb, fdb;
                    fb.v = zb;
                    fdb.v = zdb;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const frag W = lds_frag_t(s_w2, Cfg::ROW2, t, c, g, c16);
                        P::mma(xb1[t], W, fb, Cfg::ku(NU2, c));
                        P::mma(xdb1[t], W, fdb, Cfg::ku(NU2, c));
                    }
                }
                // layer 1: input s, its tangent sdot
#pragma unroll
                for (int u = 0; u < NU1; ++u) {
                    const int k = P::kidx(u / 4, g, u % 4);
                    const double yb = xb1[u >> 2][u & 3], ydb = xdb1[u >> 2][u & 3];
                    const double gd = 1 - t1[u] * t1[u], wh = s_vec[EV_WH1 + k], gzy = gd * (sd * s_vec[EV_W1 + k]) * ydb;
                    const double zb = wh * (gd * yb - 2 * t1[u] * gzy);
                    h1[u] += t1[u] * yb + gzy;
                    gb1[u] += zb;
                    gw1[u] += s * zb + sd * (wh * gd * ydb);
                }
                ++w.c;
                w.take();
            }
            // sums over the 16 pair columns, then into the gradient (feature of register u in group g)
            {
                double* gr = replica(K, net);
                auto add = [&](int off, int f, double v) {
                    for (int m = 1; m < 16; m <<= 1) v += __shfl_xor(v, m);
                    if (c16 == 0 && f >= 0) unsafeAtomicAdd(&gr[off + f], v);
                };
#pragma unroll
                for (int u = 0; u < 28; ++u) add(G_H3, emb_feat(3, g, u), h3[u]);
#pragma unroll
                for (int u = 0; u < NU2; ++u) add(G_H2, emb_feat(2, g, u), h2[u]);
#pragma unroll
                for (int u = 0; u < NU1; ++u) {
                    const int f = emb_feat(1, g, u);
                    add(G_H1, f, h1[u]);
                    add(G_B1, f, gb1[u]);
                    add(G_W1, f, gw1[u]);
                }
            }
        }
}

// Weight and bias gradients of layers 2 and 3. The chunks (grouped by net) are split evenly over the
// blocks; of a block's eight waves, wave w takes the output tiles w % 4 and w % 4 + 4 of W3 and w % 4 of W2
// for half of each chunk's pairs; the two halves meet in LDS and the sums go to the gradient with atomics.
// An operand tile is a register dump [4][64 lanes] of 16 features x 16 pairs: lane (i, g) of an MFMA takes
// feature row i and the pairs 4g..4g+3, which are consecutive there (the pairs are the summation index,
// in any order). The chunks pass through two LDS buffers, each read from memory once, a chunk ahead:
// with every wave loading its own tiles the block moved 176 KB per chunk and waited for them.
__global__ void __launch_bounds__(512, 2) k_tre_wgrad(TreArgs K)
{
    const EmbArgs& A = K.e;
    constexpr int NLD = (TRE_CHUNK / 2 + 511) / 512;
    __shared__ __attribute__((aligned(16))) double s_buf[2][TRE_CHUNK];
    static_assert(sizeof(s_buf) >= sizeof(d4) * 4 * 10 * 64, "the halves' exchange lies over the buffers");
    d4 (*s_red)[10][64] = reinterpret_cast<d4 (*)[10][64]>(&s_buf[0][0]);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), w = wave & 3, half = wave >> 2;
    const int lane = tid & 63, g = lane >> 4, c16 = lane & 15;
    const int nt = A.ntypes, n = A.natoms;
    const int64_t ld = n + 1;
    const int total = K.coff[(size_t)(nt - 1) * ld + n];
    const int b0 = (int)((int64_t)total * blockIdx.x / gridDim.x), b1 = (int)((int64_t)total * (blockIdx.x + 1) / gridDim.x);
    const int off = 64 * (c16 >> 2) + 16 * (c16 & 3) + 4 * g + 2 * half;
    for (int tj = 0; tj < nt; ++tj)
        for (int ti = 0; ti < (A.type_one_side ? 1 : nt); ++ti) {
            const int net = A.type_one_side ? tj : ti * nt + tj;
            const int n0 = K.coff[tj * ld + (A.type_one_side ? 0 : K.toff[ti])], n1 = K.coff[tj * ld + (A.type_one_side ? n : K.toff[ti + 1])];
            const int lo = max(b0, n0), hi = min(b1, n1);
            if (lo >= hi) continue;   // (uniform over the block)
            d4 a3[2][4], a2[2];       // W3: [output tile][input tile]; W2: [input tile]
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                zero4(a2[q]);
#pragma unroll
                for (int t = 0; t < 4; ++t) zero4(a3[q][t]);
            }
            const int m1 = min(w + 4, 6);   // (wave 3 has one output tile of W3: it repeats tile 6, not added)
            d2 st[NLD];
            auto load = [&](int c) {
                const d2* src = reinterpret_cast<const d2*>(K.dump + (size_t)min(c, hi - 1) * TRE_CHUNK);
#pragma unroll
                for (int q = 0; q < NLD; ++q) st[q] = src[min(tid + 512 * q, TRE_CHUNK / 2 - 1)];
                keep_loads();
            };
            auto store = [&](int b) {
#pragma unroll
                for (int q = 0; q < NLD; ++q) reinterpret_cast<d2*>(s_buf[b])[min(tid + 512 * q, TRE_CHUNK / 2 - 1)] = st[q];
            };
            load(lo);
            __syncthreads();   // (the exchange of the previous net is done)
            store(lo & 1);
            load(lo + 1);
            __syncthreads();
#pragma unroll 1
            for (int c = lo; c < hi; ++c) {
                const double* d = s_buf[c & 1];
                auto tile = [&](int u0) { return *reinterpret_cast<const d2*>(d + u0 * 64 + off); };
                auto mma = [&](const d2& x, const d2& y, d4& acc) {
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, acc, 0, 0, 0);
                };
#pragma unroll
                for (int p = 0; p < 2; ++p) {   // the values, then the tangents
                    const d2 z0 = tile((p ? D_ZD3 : D_Z3) + 4 * w), z1 = tile((p ? D_ZD3 : D_Z3) + 4 * m1);
                    const d2 q = tile((p ? D_ZD2 : D_Z2) + 4 * w);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const d2 y = tile((p ? D_YD2 : D_Y2) + 4 * t);
                        mma(y, z0, a3[0][t]);
                        mma(y, z1, a3[1][t]);
                        if (t < 2) mma(tile((p ? D_YD1 : D_Y1) + 4 * t), q, a2[t]);
                    }
                }
                store((c + 1) & 1);
                load(c + 2);
                __syncthreads();
            }
            __syncthreads();
            if (half)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    s_red[w][t][lane] = a3[0][t];
                    s_red[w][4 + t][lane] = a3[1][t];
                    if (t < 2) s_red[w][8 + t][lane] = a2[t];
                }
            __syncthreads();
            if (!half) {
                double* gr = replica(K, net);
                // rows g + 4r of input tile t, column c16 of output tile m: W[input][output], or the bias
                // where the input is the padding register that holds 1
                auto out = [&](int l, int t, int m, const d4& v, const d4& o, int W, int B, int width) {
                    const int fo = emb_feat(l, c16 & 3, 4 * m + (c16 >> 2));
                    if (fo < 0) return;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int u = 4 * t + r, fi = emb_feat(l - 1, g, u);
                        if (fi >= 0) unsafeAtomicAdd(&gr[W + fi * width + fo], v[r] + o[r]);
                        else if (g == 0 && u == (l == 3 ? ONE2 : ONE1)) unsafeAtomicAdd(&gr[B + fo], v[r] + o[r]);
                    }
                };
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    out(3, t, w, a3[0][t], s_red[w][t][lane], G_W3, G_B3, E2);
                    if (w + 4 < 7) out(3, t, w + 4, a3[1][t], s_red[w][4 + t][lane], G_W3, G_B3, E2);
                    if (t < 2) out(2, t, w, a2[t], s_red[w][8 + t][lane], G_W2, G_B2, E1);
                }
            }
        }
}

// Chunk offsets: coff[tj][a] = the first chunk of atom a's block of neighbours of type tj (chunks of 16
// kept neighbours, by neighbour type, then atom); coff[tj][n] ends the type. One block.
__global__ void __launch_bounds__(1024) k_tre_offsets(int n, int nt, const int* nnei, int* coff)
{
    __shared__ int s_w[16];
    __shared__ int s_base;
    if (threadIdx.x == 0) s_base = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int tj = 0; tj < nt; ++tj)
        for (int a0 = 0; a0 < n; a0 += 1024) {
            __syncthreads();
            const int a = a0 + threadIdx.x;
            const int own = a < n ? (nnei[(size_t)a * nt + tj] + 15) >> 4 : 0;
            int v = own;
            for (int m = 1; m < 64; m <<= 1) {
                const int o = __shfl_up(v, m);
                if (lane >= m) v += o;
            }
            if (lane == 63) s_w[wave] = v;
            __syncthreads();
            int pre = s_base, all = 0;
            for (int q = 0; q < 16; ++q) {
                if (q < wave) pre += s_w[q];
                all += s_w[q];
            }
            if (a < n) coff[(size_t)tj * (n + 1) + a] = pre + v - own;
            __syncthreads();
            if (threadIdx.x == 0) {
                s_base += all;
                if (a0 + 1024 >= n) coff[(size_t)tj * (n + 1) + n] = s_base;
            }
        }
}

// The chunk map (atom, its caller index, first neighbour, number of neighbours in the block) and Td = 0.
__global__ void __launch_bounds__(256) k_tre_map(TreArgs K)
{
    const int n = K.e.natoms, nt = K.e.ntypes;
    for (int64_t k = blockIdx.x * 256 + threadIdx.x; k < (int64_t)n * E2 * 4; k += 256 * gridDim.x) {
        K.Td[k] = 0.0;
        if (k >= (int64_t)n * nt) continue;
        const int tj = (int)(k / n), a = (int)(k % n);
        const int np = K.e.nnei[(size_t)a * nt + tj], c = K.coff[tj * (int64_t)(n + 1) + a];
        for (int q = 0; 16 * q < np; ++q) K.cmap[c + q] = int4{a, K.e.perm[a], 16 * q, np};
    }
}

// The offsets of the chunks [c0, c0 + m) taken alone: what net_range and k_tre_wgrad see of a window is a
// frame of its own. (The first chunk as an argument of the kernels took them 7 % longer, by its registers.)
__global__ void __launch_bounds__(256) k_tre_window(int64_t len, const int* coff, int c0, int m, int* woff)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < len) woff[i] = min(max(coff[i] - c0, 0), m);
}

// The copies added to the gradient, and cleared for the next frame.
__global__ void __launch_bounds__(256) k_tre_collect(TreArgs K)
{
    const int i = blockIdx.x * 256 + threadIdx.x, m = K.nets * G_NET;
    if (i >= m) return;
    double v = 0.0;
#pragma unroll 8
    for (int k = 0; k < K.nrep; ++k) {
        v += K.rep[(size_t)k * m + i];
        K.rep[(size_t)k * m + i] = 0.0;
    }
    K.grad[i] += v;
}

}  // namespace

void tre_offsets(int n, int nt, const int* nnei, int* coff, hipStream_t s)
{
    hipLaunchKernelGGL(k_tre_offsets, dim3(1), dim3(1024), 0, s, n, nt, nnei, coff);
}

// One block per CU, each with an even share of the chunks (of two or three nets at most where there are
// many): four waves, one per SIMD.
void tre_tangent(const TreArgs& k, hipStream_t s)
{
    const int blocks = k.e.ncu > 0 ? k.e.ncu : 256;
    hipLaunchKernelGGL(k_tre_map, dim3(std::min<int64_t>(((int64_t)k.e.natoms * E2 * 4 + 255) / 256, 8 * blocks)), dim3(256), 0, s, k);
    hipLaunchKernelGGL(k_tre_tan, dim3(blocks), dim3(64 * NW), 0, s, k);
}

void tre_gradient(const TreArgs& k, hipStream_t s)
{
    const int blocks = k.e.ncu > 0 ? k.e.ncu : 256;
    const int64_t len = (int64_t)k.e.ntypes * (k.e.natoms + 1);
    for (int c0 = 0; c0 < k.chunks; c0 += k.window) {
        TreArgs w = k;
        if (k.window < k.chunks) {
            w.coff = k.woff;
            w.cmap = k.cmap + c0;
            hipLaunchKernelGGL(k_tre_window, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, len, k.coff, c0,
                               std::min(k.window, k.chunks - c0), k.woff);
        }
        hipLaunchKernelGGL(k_tre_adj, dim3(blocks), dim3(64 * NW), 0, s, w);
        hipLaunchKernelGGL(k_tre_wgrad, dim3(blocks), dim3(512), 0, s, w);
    }
    hipLaunchKernelGGL(k_tre_collect, dim3((k.nets * G_NET + 255) / 256), dim3(256), 0, s, k);
}

}  // namespace dpk
