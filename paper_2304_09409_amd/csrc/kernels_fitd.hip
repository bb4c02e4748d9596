// kernels_fitd.hip -- fitting net on the 16x16x4 MFMA: the FP64 path of every descriptor, and the
// FP32 kernel of the descriptors of M values (se_e2_r, se_e3).
//
// Fitting net F_0 (Sec. II.A.2, eq. fitting_energy) for every atom, forward E_i and the input
// gradient dE_i/dT through D = T T_<^T (Sec. II.A.1).
//
// A block holds 16 atoms of one species and eight waves. Wave w owns the 16-row output tiles w and
// w + 8 (< 15) of every layer, and in the input gradient the D rows w, w + 8, ... Each weight fragment
// is read by one wave of the block, straight from global memory (fragment-major: 1 KB coalesced per
// load) into a ring of K-chunks of registers; no barrier stands between a weight and its use. The
// activations are the shared operand: a layer's output tile t is, in registers, K-chunk t of the next
// layer's B operand, so it goes to LDS as that fragment, and the block meets at two barriers per layer.
// D is formed from T in groups of G K-chunks, one group ahead of its use.
// Bound: the FP64 unit, which the matrix and the vector instructions share (a v_mfma_f64_16x16x4f64
// takes 65 cycles, each FP64 vector instruction adds its 4). 16 atoms need 3,900 x 4 products on four
// SIMDs, 104 us at 2.4 GHz. Two blocks share a CU (128 registers, four waves per SIMD) when there are
// more blocks than CUs, so that one's epilogues and barriers run beside the other's products;
// otherwise a block has its CU to itself and looks further ahead (256 registers). Measured (FP64, us):
//   atoms                       192  3,072  12,288  24,000
//   64-atom blocks, weights staged through LDS (two barriers per 16-wide K-chunk; before)
//                                 -    864     746       -
//   16-atom blocks, deep        172    179     520   1,032
//   16-atom blocks, shared CU   188    190     486     950
//   32-atom blocks, deep        298    296     600     917   (48-atom: 455, 453, 925, 973)
// and for a descriptor of M values in FP32, 2,997 atoms: 282 before, 45 now. Small frames of the M x M_<
// descriptor run in steps (launch_p): 192 atoms 105 us.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "dpk_device.h"
#include "dpk_internal.h"
#include "dpk_launch.h"

namespace dpk {
namespace {

constexpr int FD_NW = 8, FD_TPW = 2;   // waves per block, output tiles per wave
constexpr int FD_FR = 256;             // values of one fragment (64 lanes x 4)

struct D64 {
    typedef double acc;
    typedef d4 accv;
    static constexpr bool F64 = true;
    __device__ static int orow(int g, int r) { return g + 4 * r; }
    // a lane's four values of a fragment: two 16-byte halves, each contiguous over the wave
    __device__ static accv ld(const acc* f, int lane) {
        typedef double d2 __attribute__((ext_vector_type(2)));
        const d2 a = *reinterpret_cast<const d2*>(f + 2 * lane), b = *reinterpret_cast<const d2*>(f + 128 + 2 * lane);
        return accv{a[0], a[1], b[0], b[1]};
    }
    __device__ static void st(acc* f, int lane, const accv& x) {
        typedef double d2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<d2*>(f + 2 * lane) = d2{x[0], x[1]};
        *reinterpret_cast<d2*>(f + 128 + 2 * lane) = d2{x[2], x[3]};
    }
    __device__ static void mma(accv& d, const accv& a, const accv& b) {
#pragma unroll
        for (int v = 0; v < 4; ++v) d = __builtin_amdgcn_mfma_f64_16x16x4f64(a[v], b[v], d, 0, 0, 0);
    }
    __device__ static acc act(acc x, const double* th) { return tanh_tab(x, th); }
};

struct S32 {
    typedef float acc;
    typedef f4 accv;
    static constexpr bool F64 = false;
    __device__ static int orow(int g, int r) { return 4 * g + r; }
    __device__ static accv ld(const acc* f, int lane) { return *reinterpret_cast<const accv*>(f + 4 * lane); }
    __device__ static void st(acc* f, int lane, const accv& x) { *reinterpret_cast<accv*>(f + 4 * lane) = x; }
    __device__ static void mma(accv& d, const accv& a, const accv& b) {
#pragma unroll
        for (int v = 0; v < 4; ++v) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v], b[v], d, 0, 0, 0);
    }
    __device__ static acc act(acc x, const double*) { return tanh_fast(x); }
};

// RAD: a descriptor of M values D_m = T[m][0]; layer 1 has K = 100 (padded to 112, zero weights past
// 100) and the input gradient is dT[m] = (dE/dD_m, 0, 0, 0).
// DEEP: two waves per SIMD and a long lookahead, for a grid that leaves CUs idle.
// PH: the whole net, or for small frames (launch_p) one of the steps that spread the two products with W1
// over FD_SUB blocks per tile: layer 1 by output tiles, the 240-wide layers, dD and dT by rows, and the sum
// of the rows n < 16 of dT. Between them the block's scratch holds a1, then part 1 and the part-2 sums (the
// third and fourth in the slot of a3), and ga1 in the slot of a2.
enum { FD_ALL, FD_L1, FD_MID, FD_DD, FD_SUM };
constexpr int FD_SUB = 4;

template <class P, bool RAD, bool ENS, bool DEEP, int PH = FD_ALL>
__global__ void __launch_bounds__(64 * FD_NW, DEEP ? 2 : 4) k_fitd(FitArgs A_)
{
    const FitArgs A = ENS ? model_args(A_) : A_;
    typedef typename P::acc acc;
    typedef typename P::accv accv;
    constexpr int NA = 16, NW = FD_NW, TPW = PH == FD_L1 ? 1 : FD_TPW, FR = FD_FR;
    constexpr int PD = DEEP ? 5 : 3;                   // weight lookahead (K-chunks)
    constexpr int G = DEEP ? 5 : 4;                    // layer 1: chunks per D group,
    constexpr int P1 = RAD ? PD : G;                   // and its lookahead
    static_assert(15 % PD == 0 && E2 % G == 0 && G % (RAD ? G : P1) == 0, "whole ring turns");
    static_assert(P::F64 || RAD, "the FP32 path of the M x M_< descriptor keeps its own summation order");
    // B operands by K-chunk (layer 1: two groups of G chunks); at the end the part-2 sums of dT,
    // [4][64 lanes][16]
    __shared__ __attribute__((aligned(16))) acc s_b[4096];
    // T rows n < 16 of the block's atoms and part 1 of their dT (rows padded to 17 entries)
    __shared__ __attribute__((aligned(16))) acc s_tq[RAD ? 1 : NA][17][4];
    __shared__ __attribute__((aligned(16))) acc s_p1[RAD ? 1 : NA][17][4];
    __shared__ acc s_e[NW][NA];
    __shared__ double s_th[P::F64 ? TH_N : 1];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform (scalar registers)
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    // Species-aligned tiling: species t has ceil(count_t / NA) blocks of its own. Block b runs on XCD
    // b % 8, and each XCD takes a contiguous range of the blocks that hold atoms (the grid is an upper
    // bound; the surplus ones leave here, the same number on every XCD: with the range taken over the
    // whole grid one XCD got a block more than its 32 CUs hold in three rounds on the 12,288-atom box,
    // 670 instead of 520 us)
    static_assert(PH == FD_ALL || !RAD, "the steps are those of the M x M_< descriptor");
    const int ngrid = PH == FD_L1 || PH == FD_DD ? gridDim.x / FD_SUB : gridDim.x;   // (a multiple of 8)
    const int sub = blockIdx.x / ngrid, bx = blockIdx.x - sub * ngrid;
    int a0 = -1, ti = 0, a1 = 0, blk = 0;
    {
        int real = 0;
        for (int t = 0; t < A.ntypes; ++t) real += (A.toff[t + 1] - A.toff[t] + NA - 1) / NA;
        const int xcd = bx & 7, at = bx >> 3, per = real >> 3, rem = real & 7;
        if (at >= per + (xcd < rem)) return;
        blk = xcd * per + min(xcd, rem) + at;
        int tb = blk;
        for (int t = 0; t < A.ntypes; ++t) {
            const int lo = A.toff[t], hi = A.toff[t + 1], nb = (hi - lo + NA - 1) / NA;
            if (tb < nb) {
                a0 = lo + tb * NA;
                a1 = hi;
                ti = t;
                break;
            }
            tb -= nb;
        }
    }
    if (a0 < 0) return;
    if constexpr (P::F64 && PH != FD_DD && PH != FD_SUM) tanh_tab_fill(s_th);
    const acc* Tg = reinterpret_cast<const acc*>(A.T);
    acc* dTg = reinterpret_cast<acc*>(A.dT);
    // tanh outputs (layer l, tile t): this lane's four values, read back by the same lane (the FP32
    // energy sum reads other waves', after a barrier)
    acc* scr = reinterpret_cast<acc*>(A.act) + (size_t)blk * (45 * FR);
    auto sptr = [&](int l, int t) { return reinterpret_cast<accv*>(scr + (l * 15 + t) * FR + 4 * lane); };
    auto sb = [&](int c) { return s_b + c * FR; };
    const acc* fv = reinterpret_cast<const acc*>(A.fvec) + (size_t)ti * FVEC;
    const acc* W = reinterpret_cast<const acc*>(A.fmat) + (size_t)ti * FM_SIZE;
    // tiles ftile(i) = first + 8 i < 15 (layer 1 on its own: four per block, of one wave each)
    const int first = PH == FD_L1 ? min(4 * sub + (wave & 3), 14) : wave;
    const int nown = PH == FD_L1 ? (wave < 4 && 4 * sub + wave < 15) : (15 - wave + NW - 1) / NW;
    auto ftile = [&](int i) { return first + NW * i; };
    // (a wave without a tile i reads its first tile again: every read is unconditional, since a read
    // skipped by a branch makes the compiler wait for every read in flight)
    auto wtile = [&](int i) { return i < nown ? ftile(i) : first; };
    const int at = a0 + c16;                           // this lane's atom (its column of every tile)
    const bool mine = at < a1;
    const acc* Ta = Tg + (size_t)min(at, a1 - 1) * (E2 * 4);
    auto vec = [&](int off, int t, int r) { return fv[off + 16 * t + P::orow(g, r)]; };

    accv acc_[TPW];
    accv ring[P1 > PD ? P1 : PD][TPW];
    auto wld = [&](int64_t mo, int c, int t) { return P::ld(W + mo + ((int64_t)c * 15 + t) * FR, lane); };
    // the first np chunks of a 15-tile product, requested before the preceding epilogue and barrier
    auto prefetch = [&](int64_t mo, auto np) {
#pragma unroll
        for (int d = 0; d < np.value; ++d)
#pragma unroll
            for (int i = 0; i < TPW; ++i) ring[d][i] = wld(mo, d, wtile(i));
    };
    auto zero_acc = [&]() {
#pragma unroll
        for (int i = 0; i < TPW; ++i) acc_[i] = accv{0, 0, 0, 0};
    };
    // one K-chunk: products of ring slot `sl` with the B fragment b, then the slot is refilled with
    // chunk cn of the product
    auto chunk = [&](int sl, int64_t mo, int cn, const acc* b) {
        accv Ac[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) Ac[i] = ring[sl][i];
#pragma unroll
        for (int i = 0; i < TPW; ++i) ring[sl][i] = wld(mo, cn, wtile(i));
        keep_loads();
        const accv B = P::ld(b, lane);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) P::mma(acc_[i], Ac[i], B);
    };
    auto gemm = [&](int64_t mo) {   // 240-wide input: 15 chunks
        zero_acc();
#pragma unroll 1
        for (int c0 = 0; c0 < 15; c0 += PD)
#pragma unroll
            for (int d = 0; d < PD; ++d) chunk(d, mo, min(c0 + d + PD, 14), sb(c0 + d));
    };
    const std::integral_constant<int, PD> npd;

    // T rows n < 16 of the block's atoms
    auto stage_tq = [&]() {
        if (threadIdx.x < NA * 16) {
            const int al = threadIdx.x >> 4, n = threadIdx.x & 15;
            *reinterpret_cast<accv*>(&s_tq[al][n][0]) =
                *reinterpret_cast<const accv*>(Tg + ((size_t)min(a0 + al, a1 - 1) * E2 + n) * 4);
        }
    };
    // ------------------------------------------------------------ layer 1
    if constexpr (PH == FD_ALL || PH == FD_L1) prefetch(FM_W1T, std::integral_constant<int, P1>());
    if constexpr (PH != FD_ALL && PH != FD_L1) {
    } else if constexpr (RAD) {
        // D_m = T[m][0] as the B fragments of K-chunks 0..6
        if (wave < RAD_K / 16) {
            accv x;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * wave + P::orow(g, v);
                x[v] = Ta[(m < E2 ? m : 0) * 4];
                if (m >= E2) x[v] = 0;
            }
            P::st(sb(wave), lane, x);
        }
        __syncthreads();
        zero_acc();
#pragma unroll
        for (int c = 0; c < RAD_K / 16; ++c) chunk(c % P1, FM_W1T, min(c + P1, RAD_K / 16 - 1), sb(c));
    } else {
        stage_tq();
        // wave w < G forms the D fragment of chunk w of a group: lane group g holds D[c][orow(g, v)],
        // D[m][n] = sum_k T[m][k] T[n][k]
        accv Tm = *reinterpret_cast<const accv*>(Ta + min(wave, E2 - 1) * 4);
        auto dform = [&](int p) {
            if (wave < G) {
                accv d;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const accv tn = *reinterpret_cast<const accv*>(&s_tq[c16][P::orow(g, v)][0]);
                    d[v] = Tm[0] * tn[0] + Tm[1] * tn[1] + Tm[2] * tn[2] + Tm[3] * tn[3];
                }
                P::st(sb(p * G + wave), lane, d);
            }
        };
        __syncthreads();
        dform(0);
        zero_acc();
        __syncthreads();
#pragma unroll 1
        for (int grp = 0; grp < E2 / G; ++grp) {
            const int p = grp & 1;
            Tm = *reinterpret_cast<const accv*>(Ta + min((grp + 1) * G + wave, E2 - 1) * 4);
#pragma unroll
            for (int d = 0; d < G; ++d) chunk(d % P1, FM_W1T, min(grp * G + d + P1, E2 - 1), sb(p * G + d));
            if (grp + 1 < E2 / G) dform(p ^ 1);
            __syncthreads();
        }
    }
    // a1 = tanh(W1 D + b1), h1 = wh1 a1; layers 2, 3: a = tanh(W h + b), h += wh a. The layer's input
    // h is read back from this lane's own fragments, which its output then replaces
    if constexpr (PH != FD_DD && PH != FD_SUM) {
    if constexpr (PH == FD_MID) {
        prefetch(FM_W2T, npd);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                const accv av = *sptr(0, t);
                accv h;
#pragma unroll
                for (int r = 0; r < 4; ++r) h[r] = vec(FV_WH1, t, r) * av[r];
                P::st(sb(t), lane, h);
            }
        __syncthreads();
    }
    acc e = 0;   // FP64: this lane's share of w4 . h3
#pragma unroll 1
    for (int layer = PH == FD_MID ? 2 : 1; layer <= (PH == FD_L1 ? 1 : 3); ++layer) {
        if (layer > 1) gemm(layer == 2 ? FM_W2T : FM_W3T);
        if (PH != FD_L1) {
            prefetch(layer == 1 ? FM_W2T : layer == 2 ? FM_W3T : FM_W3, npd);
            __syncthreads();
        }
        const int ob = layer == 1 ? FV_B1 : layer == 2 ? FV_B2 : FV_B3;
        const int ow = layer == 1 ? FV_WH1 : layer == 2 ? FV_WH2 : FV_WH3;
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                accv av, h = {0, 0, 0, 0};
                if (layer > 1) h = P::ld(sb(t), lane);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    av[r] = P::act(acc_[i][r] + vec(ob, t, r), s_th);
                    h[r] = vec(ow, t, r) * av[r] + h[r];
                }
                *sptr(layer - 1, t) = av;
                if (PH == FD_L1) continue;
                if (layer < 3) P::st(sb(t), lane, h);
                else if constexpr (P::F64)
#pragma unroll
                    for (int r = 0; r < 4; ++r) e += h[r] * vec(FV_W4, t, r);
            }
        if (layer < 3) __syncthreads();
    }
    if constexpr (PH == FD_L1) return;
    // ------------------------------------------------------------ energy E_i = wh4 (w4 . h3 + b4) and
    // backward: gh3 = wh4 w4, ga3 = gh3 wh3 (1 - a3^2); gh_{l-1} = W_l^T ga_l + gh_l,
    // ga_l = gh_l wh_l (1 - a_l^2)
    const acc wh4 = fv[FV_WH4];
    if constexpr (P::F64) {
        const acc es = sum_groups(e);
        if (g == 0) s_e[wave][c16] = es;
    } else {
        __syncthreads();   // every wave's tanh outputs
        if (wave == 0) {
            // one wave adds the features in order
            acc es = 0;
#pragma unroll 1
            for (int t = 0; t < 15; ++t) {
                const accv x1 = *sptr(0, t), x2 = *sptr(1, t), x3 = *sptr(2, t);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const acc h3 = vec(FV_WH3, t, r) * x3[r] + vec(FV_WH2, t, r) * x2[r] + vec(FV_WH1, t, r) * x1[r];
                    es += h3 * vec(FV_W4, t, r);
                }
            }
            es += __shfl_xor(es, 16);
            es += __shfl_xor(es, 32);
            if (g == 0 && mine) A.Ei[at] = wh4 * (es + fv[FV_B4]);
        }
        __syncthreads();   // (layer 3's slots are overwritten with gh2 below)
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i)
        if (i < nown) {
            const int t = ftile(i);
            const accv x3 = *sptr(2, t);
            accv ga;
#pragma unroll
            for (int r = 0; r < 4; ++r) ga[r] = wh4 * vec(FV_W4, t, r) * vec(FV_WH3, t, r) * (1 - x3[r] * x3[r]);
            P::st(sb(t), lane, ga);
        }
    __syncthreads();
    if (P::F64 && threadIdx.x < NA && a0 + (int)threadIdx.x < a1) {
        acc es = 0;
        for (int w = 0; w < NW; ++w) es += s_e[w][threadIdx.x];
        A.Ei[a0 + threadIdx.x] = wh4 * (es + fv[FV_B4]);
    }
#pragma unroll 1
    for (int layer = 3; layer >= 2; --layer) {
        gemm(layer == 3 ? FM_W3 : FM_W2);
        if (layer == 3) prefetch(FM_W2, npd);
        __syncthreads();
        const int ow = layer == 3 ? FV_WH2 : FV_WH1;
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                const accv x = *sptr(layer - 2, t);
                accv ga, gh;
                if (layer == 2) gh = *sptr(2, t);   // gh2, in the slot of a3
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    gh[r] = layer == 3 ? acc_[i][r] + wh4 * vec(FV_W4, t, r) : acc_[i][r] + gh[r];
                    ga[r] = gh[r] * vec(ow, t, r) * (1 - x[r] * x[r]);
                }
                if (layer == 3) *sptr(2, t) = gh;
                P::st(sb(t), lane, ga);
                if (PH == FD_MID && layer == 2) P::st(scr + (15 + t) * FR, lane, ga);
            }
        __syncthreads();
    }
    if constexpr (PH == FD_MID) return;
    }
    // ------------------------------------------------------------ dD = W1 ga1 and dT
    // D rows m = wave + 8 j (RAD: 16-row tiles of dE/dD_m); the weight fragments of the next PD steps,
    // also across a row boundary, are in flight
    auto p1g = [&](int al, int n) { return reinterpret_cast<accv*>(scr + (al * 16 + n) * 4); };
    auto q2g = [&](int k, int al, int n) {
        return reinterpret_cast<accv*>(scr + (k < 2 ? 1024 * (1 + k) : 30 * FR + 1024 * (k - 2)) + (al * 16 + n) * 4);
    };
    if constexpr (PH == FD_SUM) {
        const int al = threadIdx.x >> 4, n = threadIdx.x & 15;
        if (threadIdx.x < 256 && a0 + al < a1) {
            accv v = *p1g(al, n);
#pragma unroll
            for (int k = 0; k < FD_SUB; ++k) v += *q2g(k, al, n);
            *reinterpret_cast<accv*>(dTg + ((size_t)(a0 + al) * E2 + n) * 4) = v;
        }
        return;
    }
    if constexpr (PH == FD_DD) {
        for (int x = threadIdx.x; x < 15 * FR / 4; x += 64 * NW)
            reinterpret_cast<accv*>(s_b)[x] = reinterpret_cast<const accv*>(scr + 15 * FR)[x];
        stage_tq();
        __syncthreads();
    }
    constexpr int NM = RAD ? RAD_K / 16 : E2, MS = PH == FD_DD ? NW * FD_SUB : NW;
    const int m0 = PH == FD_DD ? wave + NW * sub : wave;   // rows m0 + MS j
    auto wrow = [&](int m, int c) { return P::ld(W + FM_W1 + ((int64_t)m * 15 + c) * FR, lane); };   // (by tile)
    accv rd[PD];
#pragma unroll
    for (int d = 0; d < PD; ++d) rd[d] = wrow(min(m0, NM - 1), d);
    accv q2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) q2[r] = accv{0, 0, 0, 0};
#pragma unroll 1
    for (int m = m0; m < NM; m += MS) {
        accv dd = {0, 0, 0, 0}, tm = {0, 0, 0, 0};
        if constexpr (!RAD) tm = *reinterpret_cast<const accv*>(Ta + m * 4);   // for the epilogue
#pragma unroll 1
        for (int c0 = 0; c0 < 15; c0 += PD)
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                const int c = c0 + d;
                const accv Ac = rd[d];
                rd[d] = c + PD < 15 ? wrow(m, c + PD) : wrow(min(m + MS, NM - 1), c + PD - 15);
                keep_loads();
                P::mma(dd, Ac, P::ld(sb(c), lane));
            }
        if constexpr (RAD) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * m + P::orow(g, r);
                if (mine && row < E2) *reinterpret_cast<accv*>(dTg + ((size_t)at * E2 + row) * 4) = accv{dd[r], 0, 0, 0};
            }
        } else {
            // dT[m] += sum_n dD[m][n] T[n] (part 1, over the lane groups) and, for n < 16,
            // dT[n] += sum_m dD[m][n] T[m] (part 2, q2: over the waves at the end)
            acc part[4] = {0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const accv tn = *reinterpret_cast<const accv*>(&s_tq[c16][P::orow(g, r)][0]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    part[k] += dd[r] * tn[k];
                    q2[r][k] += dd[r] * tm[k];
                }
            }
            const acc pk = sum_groups4(part);   // lane group g: component ksel(g)
            if (m < 16) {
                if constexpr (PH == FD_DD) (*p1g(c16, m))[ksel(g)] = pk;
                else s_p1[c16][m][ksel(g)] = pk;
            } else if (mine) {
                dTg[((size_t)at * E2 + m) * 4 + ksel(g)] = pk;
            }
        }
    }
    if constexpr (!RAD) {
        // rows n < 16 of dT: part 1 plus the eight waves' part 2, through LDS
        accv* slot = reinterpret_cast<accv*>(s_b + ((wave & 3) * 64 + lane) * 16);
        __syncthreads();   // ga1 is no longer read
        if (wave >= 4)
#pragma unroll
            for (int r = 0; r < 4; ++r) slot[r] = q2[r];
        __syncthreads();
        if (wave < 4)
#pragma unroll
            for (int r = 0; r < 4; ++r) slot[r] = slot[r] + q2[r];
        __syncthreads();
        if (threadIdx.x < 256) {
            const int al = threadIdx.x >> 4, n = threadIdx.x & 15;
            const int gg = P::F64 ? n & 3 : n >> 2, r = P::F64 ? n >> 2 : n & 3;
            accv v = {0, 0, 0, 0};
            if constexpr (PH != FD_DD) v = *reinterpret_cast<const accv*>(&s_p1[al][n][0]);
#pragma unroll
            for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const accv*>(s_b + (w * 64 + gg * 16 + al) * 16 + 4 * r);
            if constexpr (PH == FD_DD) *q2g(sub, al, n) = v;
            else if (a0 + al < a1) *reinterpret_cast<accv*>(dTg + ((size_t)(a0 + al) * E2 + n) * 4) = v;
        }
    }
}

// The steps, one launch each.
template <class P, bool ENS>
void launch_steps(const FitArgs& a, dim3 grid, hipStream_t s)
{
    const dim3 wide(grid.x * FD_SUB, grid.y), block(64 * FD_NW);
    hipLaunchKernelGGL((k_fitd<P, false, ENS, true, FD_L1>), wide, block, 0, s, a);
    hipLaunchKernelGGL((k_fitd<P, false, ENS, true, FD_MID>), grid, block, 0, s, a);
    hipLaunchKernelGGL((k_fitd<P, false, ENS, true, FD_DD>), wide, block, 0, s, a);
    hipLaunchKernelGGL((k_fitd<P, false, ENS, true, FD_SUM>), grid, block, 0, s, a);
}

template <class P, bool RAD>
void launch_p(const FitArgs& a, hipStream_t s)
{
    const bool ens = a.nmodels > 1;
    const int blocks = (a.natoms + 15) / 16 + a.ntypes;
    const dim3 grid((blocks + 7) / 8 * 8, ens ? a.nmodels : 1), block(64 * FD_NW);
    // a CU holds one deep block or two of the others
    const bool deep = (int64_t)((a.natoms + 15) / 16) * grid.y <= (a.ncu > 0 ? a.ncu : 256);
    // In steps while two blocks per CU hold the split phases: FP64, 192 atoms 105 us against 175 in one
    // launch, 1,020 144 against 171, 1,800 146 against 174; past that they lose (2,400: 184 and 175).
    if constexpr (!RAD)
        if ((int64_t)blocks * grid.y * FD_SUB <= 2 * (a.ncu > 0 ? a.ncu : 256)) {
            if (ens) launch_steps<P, true>(a, grid, s);
            else launch_steps<P, false>(a, grid, s);
            return;
        }
    if (ens && deep) hipLaunchKernelGGL((k_fitd<P, RAD, true, true>), grid, block, 0, s, a);
    else if (ens) hipLaunchKernelGGL((k_fitd<P, RAD, true, false>), grid, block, 0, s, a);
    else if (deep) hipLaunchKernelGGL((k_fitd<P, RAD, false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_fitd<P, RAD, false, false>), grid, block, 0, s, a);
}

}  // namespace

void launch_fitd(bool f64, const FitArgs& a, hipStream_t s)
{
    if (a.natoms <= 0) return;
    if (f64 && a.radial) launch_p<D64, true>(a, s);
    else if (f64) launch_p<D64, false>(a, s);
    else launch_p<S32, true>(a, s);
}

}  // namespace dpk
