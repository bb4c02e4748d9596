// kernels_fit.hip -- fitting net of the BF16 paths (split BF16 and plain BF16).
//
// Fitting net F_0 (Sec. II.A.2, eq. fitting_energy) for every atom, forward E_i and the input
// gradient dE_i/dT through D = T T_<^T (Sec. II.A.1). The products run on
// v_mfma_f32_16x16x32_bf16, which issues twice the K of the 16x16x16 form in the same cycles.
//
// Work split: a block holds NAT tiles of 16 atoms and eight waves; wave w owns the 16-row feature
// tiles w and w + 8 (< 15) of every layer for all atoms of the block; the backward dD product is split
// by role (below). Weights are read by exactly one wave each, straight from global memory
// (fragment-major, one coalesced 1 KB load per plane), several K-chunks ahead. The B operands (D for
// layer 1, then h_l or ga_l) are shared through LDS as split BF16 fragments; a layer's output tiles 2c
// and 2c+1 fill the two halves of K-chunk c of the next layer (the weights' K order matches, see XF_*
// in dpk_internal.h). D is formed from T by the waves of its atom tile, a group of K-chunks ahead, so
// layer 1 has one barrier per group.
// Blocks are placed so that each XCD (block b runs on XCD b % 8) works on a contiguous range of
// atoms: with atoms sorted by species, an XCD's L2 mostly holds one species' weights.
// Bound: the streaming of the weights (4.16 MB per block; small frames) and, in the 64-atom shape, the
// matrix unit with the LDS reads of the B operands. Measured (mixed; before the split by role, the longer
// lookahead and, for small frames, the steps, in brackets): 192 atoms 51 us (91), 12,288 atoms 119 us
// (128), 110,592 atoms 798 us (900).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "dpk_device.h"
#include "dpk_internal.h"
#include "dpk_launch.h"

namespace dpk {
namespace {

typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

struct F8 {
    bf8 h, l;
};

constexpr int FX_G = 4;    // layer-1 K-chunks per D group
constexpr int FX_PD = 4;   // weight lookahead (K-chunks) of the 240-wide layers

// The net in one launch, or for small frames (launch_fitx) in steps, so that the two products with W1,
// three quarters of the weights, are spread over FX_SUB blocks per atom tile: layer 1 split by output
// features, the 240-wide layers, dD and dT split by the rows m = sub (mod 4). Every sum keeps its order: the
// results are those of the one launch. A last small launch adds the part-2 partials to the rows m < 16.
// (Left to the last block of a tile to finish, its fences, which write an XCD's L2 back, took longer the
// more blocks there were: 37 us for 600 atoms, 89 for 1,890.) Between the launches a block's scratch holds,
// per layer slot: slot 0 the activations of layer 1 and afterwards part 1 of the rows m < 16 and a place for
// stores that have no atom; slot 1 the part-2 partials; slot 2 ga1.
enum { FX_ALL, FX_L1, FX_MID, FX_DD, FX_SUM };
constexpr int FX_SUB = 4;

// acc += a b with a, b split as hi + lo: lo*hi + hi*lo + hi*hi (SPLIT), or hi*hi only.
template <bool SPLIT>
__device__ __forceinline__ void mma32(f4& c, const F8& a, const F8& b)
{
    if constexpr (SPLIT) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, c, 0, 0, 0);
    }
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, c, 0, 0, 0);
}

// One lane's part of a fragment: hi at lane*8, lo at 512 + lane*8 (global memory or LDS).
template <bool SPLIT>
__device__ __forceinline__ F8 ld_frag(const __bf16* f, int lane)
{
    F8 r;
    r.h = *reinterpret_cast<const bf8*>(f + lane * 8);
    if constexpr (SPLIT) r.l = *reinterpret_cast<const bf8*>(f + 512 + lane * 8);
    else r.l = bf8{};
    return r;
}

// Buffer-resource loads of the (read-only) weights: the per-lane part of an address is one VGPR
// offset (lane * 16 B) shared by all loads, the fragment offset a scalar. Keeps 64-bit per-lane
// addresses out of the register file; loads past num_records read 0.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
// Weight fragment f of the buffer r (fragment-major, XF_ELEMS BF16 values = 2 KB each).
template <bool SPLIT>
__device__ __forceinline__ F8 ld_wfrag(rsrc_t r, int lane16, int f)
{
    F8 x;
    x.h = __builtin_bit_cast(bf8, __builtin_amdgcn_raw_buffer_load_b128(r, lane16, f * 2048, 0));
    if constexpr (SPLIT) x.l = __builtin_bit_cast(bf8, __builtin_amdgcn_raw_buffer_load_b128(r, lane16, f * 2048 + 1024, 0));
    else x.l = bf8{};
    return x;
}

// Write four values (half `half` of a lane's eight) of a fragment in LDS, split into hi and lo.
template <bool SPLIT>
__device__ __forceinline__ void st_half(__bf16* f, int lane, int half, const float* x)
{
    bf4 hi, lo;
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        bf16x2_t h, l;
        split_bf16x2(x[r], x[r + 1], h, l);
        hi[r] = h[0]; hi[r + 1] = h[1];
        lo[r] = l[0]; lo[r + 1] = l[1];
    }
    *reinterpret_cast<bf4*>(f + lane * 8 + half * 4) = hi;
    if constexpr (SPLIT) *reinterpret_cast<bf4*>(f + 512 + lane * 8 + half * 4) = lo;
}

template <int NAT, bool SPLIT, int NW, bool ENS, int PH>
__global__ void __launch_bounds__(64 * NW) k_fitx(FitArgs A_)
{
    const FitArgs A = ENS ? model_args(A_) : A_;
    constexpr int NA = 16 * NAT;                       // atoms per block
    constexpr int FR = XF_ELEMS, PD = FX_PD;
    constexpr int TPW = PH == FX_L1 ? 1 : (15 + NW - 1) / NW;   // feature tiles per wave (at most)
    constexpr int NWA = NW / NAT;                      // waves sharing one atom tile's D fragments
    static_assert(NW % NAT == 0 && NW >= 4, "wave layout");
    static_assert(XF_NCH2 % PD == 0, "prefetch ring slots are compile-time");
    // B operands [K-chunk][atom tile] (layer 1: two groups of FX_G chunks); at the end the
    // per-wave dT partials (floats) of the D rows n < 16.
    __shared__ __attribute__((aligned(16))) __bf16 s_b[XF_NCH2 * NAT * FR];
    __shared__ float s_e[NW][NA];
    // rows padded to 17 entries so that the 16 atoms a wave touches at once fall in distinct banks
    __shared__ __attribute__((aligned(16))) float s_p1[NA][17][4];
    __shared__ __attribute__((aligned(16))) float s_tq[NA][17][4];     // T rows n < 16 of the block's atoms
    __shared__ __attribute__((aligned(16))) float s_dd[2][4][NAT][64][4];   // D rows between the waves (dD phase)

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform (scalar registers)
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int nblk = gridDim.x, xcd = blockIdx.x & 7, per = nblk >> 3, rem = nblk & 7;
    const int pos = xcd * per + min(xcd, rem) + (blockIdx.x >> 3);
    // (the sub-blocks of one number, which read the same weights, follow each other)
    const int ntile = PH == FX_L1 || PH == FX_DD ? nblk / FX_SUB : nblk, sub = pos / ntile, blk = pos - sub * ntile;
    // tile blk of the species-aligned tiling: species t has ceil(count_t / NA) tiles of its own,
    // so that no block runs the net twice for a boundary between species (the grid holds
    // ceil(N / NA) + ntypes blocks, an upper bound; the surplus ones leave here)
    int a0 = -1, ty = 0;
    {
        int tb = blk;
        for (int t = 0; t < A.ntypes; ++t) {
            const int lo = A.toff[t], nb = (A.toff[t + 1] - lo + NA - 1) / NA;
            if (tb < nb) {
                a0 = lo + tb * NA;
                ty = t;
                break;
            }
            tb -= nb;
        }
    }
    if (a0 < 0) return;
    const int ti = ty;
    const float* Tg = reinterpret_cast<const float*>(A.T);
    float* dTg = reinterpret_cast<float*>(A.dT);
    float* scr = reinterpret_cast<float*>(A.act) + (size_t)blk * NAT * XF_ACT;
    // feature tiles ftile(i) = first + NW i < 15 (layer 1 on its own: four per block)
    const int first = PH == FX_L1 ? 4 * sub + wave : wave;
    const int nown = PH == FX_L1 ? (first < 15 ? 1 : 0) : (15 - wave + NW - 1) / NW;
    auto ftile = [&](int i) { return first + NW * i; };

    // activation scratch of (layer l, feature tile t, atom tile a): this lane's four values
    const int lane16 = lane * 16;
    // this lane's four values of (layer l, feature tile t, atom tile a) in the scratch: a
    // wave-uniform base plus the lane's 16-byte offset (read back by the same lane)
    const unsigned ulane16 = (unsigned)lane16;
    auto sptr = [&](int l, int t, int a) {
        char* base = reinterpret_cast<char*>(scr) + (unsigned)(((l * 16 + t) * NAT + a) * 1024);
        return reinterpret_cast<f4*>(base + ulane16);
    };
    auto sb = [&](int c, int a) { return s_b + (c * NAT + a) * FR; };

    const float* fv = reinterpret_cast<const float*>(A.fvec) + (size_t)ti * FVEC;
    const __bf16* W = reinterpret_cast<const __bf16*>(A.fmat) + (size_t)ti * XF_NFRAG * FR;
    const rsrc_t wrs = make_rsrc(W, XF_NFRAG * FR * 2);

    f4 acc[TPW][NAT];
    float h[TPW][NAT][4];
    auto zero_acc = [&]() {
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int a = 0; a < NAT; ++a) acc[i][a] = f4{0.f, 0.f, 0.f, 0.f};
    };
    // Weight fragment of K-chunk c of the product at wb for the wave's tile i (a wave without a
    // tile i reads its last valid tile again: every read is unconditional, since a read skipped
    // by a branch makes the compiler wait for every read in flight).
    auto wtile = [&](int i) { return min(ftile(i), 14); };
    // The first PD K-chunks of the next 240-wide product, requested before the preceding
    // epilogue and barrier so that their latency is hidden; each product step then requests
    // the chunk PD ahead (a ring of PD register slots).
    F8 Apf[PD][TPW];
    auto prefetch8 = [&](int wb) {
#pragma unroll
        for (int d = 0; d < PD; ++d)
#pragma unroll
            for (int i = 0; i < TPW; ++i) Apf[d][i] = ld_wfrag<SPLIT>(wrs, lane16, wb + d * 15 + wtile(i));
    };
    // acc[i][a] = sum over the 8 K-chunks of W(own tile i, c) B(c, a), B from s_b; Apf must
    // hold the first chunk of product wb (prefetch8)
    auto gemm8 = [&](int wb) {
        zero_acc();
        F8 Rg[PD][TPW];
#pragma unroll
        for (int d = 0; d < PD; ++d)
#pragma unroll
            for (int i = 0; i < TPW; ++i) Rg[d][i] = Apf[d][i];
#pragma unroll
        for (int c = 0; c < XF_NCH2; ++c) {
            F8 Ac[TPW];
#pragma unroll
            for (int i = 0; i < TPW; ++i) Ac[i] = Rg[c % PD][i];
            if (c + PD < XF_NCH2) {
#pragma unroll
                for (int i = 0; i < TPW; ++i) Rg[c % PD][i] = ld_wfrag<SPLIT>(wrs, lane16, wb + (c + PD) * 15 + wtile(i));
            }
            keep_loads();
            F8 B[NAT];
#pragma unroll
            for (int a = 0; a < NAT; ++a) B[a] = ld_frag<SPLIT>(sb(c, a), lane);
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (i < nown) {
#pragma unroll
                    for (int a = 0; a < NAT; ++a) mma32<SPLIT>(acc[i][a], Ac[i], B[a]);
                }
        }
    };
    auto vec4 = [&](int off, int t) { return *reinterpret_cast<const f4*>(fv + off + 16 * t + 4 * g); };

    auto stage_tq = [&]() {
        for (int idx = threadIdx.x; idx < NA * 16; idx += 64 * NW) {
            const int al = idx >> 4, n = idx & 15;
            const int at = a0 + al < A.natoms ? a0 + al : a0;
            *reinterpret_cast<f4*>(&s_tq[al][n][0]) = *reinterpret_cast<const f4*>(Tg + ((size_t)at * E2 + n) * 4);
        }
    };
    // feature tile 15 does not exist: the second half of K-chunk 7 is zero
    auto zero_tile15 = [&]() {
        const float z[4] = {0.f, 0.f, 0.f, 0.f};
        if (wave == NW - 1)
#pragma unroll
            for (int a = 0; a < NAT; ++a) st_half<SPLIT>(sb(7, a), lane, 1, z);
    };
    if constexpr (PH == FX_ALL || PH == FX_L1) {
        if constexpr (PH == FX_ALL) stage_tq();
        // ------------------------------------------------------------ layer 1: D (1600) -> 240
        // D fragment of K-chunk c for atom tile `wave`: lane group g holds D[2c][4g+r] and
        // D[2c+1][4g+r], D[m][n] = sum_k T[m][k] T[n][k] (Sec. II.A.1, D = T T_<^T).
        // wave w forms the D fragments of atom tile wa = w % NAT for the K-chunks cc = ph (mod NWA)
        const int wa = wave % NAT, ph = wave / NAT;
        const float* Tw = Tg + (size_t)(a0 + 16 * wa + c16 < A.natoms ? a0 + 16 * wa + c16 : a0) * (E2 * 4);
        float Tn[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f4 v = *reinterpret_cast<const f4*>(Tw + (4 * g + r) * 4);
#pragma unroll
            for (int k = 0; k < 4; ++k) Tn[r][k] = v[k];
        }
        // T rows 2c and 2c + 1 of this lane's atom for the chunks c = ph, ph + NWA, ... of a group, and
        // the D fragment of a chunk formed from them
        constexpr int NF = FX_G / NWA;
        static_assert(FX_G % NWA == 0, "every wave forms as many fragments of a group");
        f4 ta[NF], tb[NF];
        auto trows = [&](int grp) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const float* r = Tw + min(grp * FX_G + ph + NWA * q, XF_NCH1 - 1) * 8;
                ta[q] = *reinterpret_cast<const f4*>(r);
                tb[q] = *reinterpret_cast<const f4*>(r + 4);
            }
        };
        auto dform = [&](const f4& ta, const f4& tb, __bf16* f) {
            float d0[4], d1[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d0[r] = ta[0] * Tn[r][0] + ta[1] * Tn[r][1] + ta[2] * Tn[r][2] + ta[3] * Tn[r][3];
                d1[r] = tb[0] * Tn[r][0] + tb[1] * Tn[r][1] + tb[2] * Tn[r][2] + tb[3] * Tn[r][3];
            }
            st_half<SPLIT>(f, lane, 0, d0);
            st_half<SPLIT>(f, lane, 1, d1);
        };
        trows(0);
#pragma unroll
        for (int q = 0; q < NF; ++q) dform(ta[q], tb[q], sb(ph + NWA * q, wa));
        __syncthreads();
        {
            zero_acc();
            const int wb = XF_W1F;
            constexpr int P1 = 2 * FX_G;   // weight lookahead: the ring slots of two groups
            F8 R1[P1][TPW];
#pragma unroll
            for (int d = 0; d < P1; ++d)
#pragma unroll
                for (int i = 0; i < TPW; ++i) R1[d][i] = ld_wfrag<SPLIT>(wrs, lane16, wb + d * 15 + wtile(i));
            constexpr int NGRP = (XF_NCH1 + FX_G - 1) / FX_G;
            // One group of FX_G K-chunks. Reads retire in issue order, so the T rows of the D fragments
            // this wave forms for the next group are read at the group's start, before its weight
            // prefetches, and every read is unconditional (clamped to valid rows and fragments; a wave
            // with fewer tiles reads one it does not use): a read skipped by a branch would make the
            // compiler drain all reads in flight. The last, partial group is peeled so that its chunk
            // bounds are constants.
            auto group = [&](int grp, auto par) {
                constexpr int p = par.value;   // grp % 2
                trows(grp + 1);
#pragma unroll
                for (int cc = 0; cc < FX_G; ++cc) {
                    const int c = grp * FX_G + cc;
                    if (c < XF_NCH1) {
                        F8 Ac[TPW];
#pragma unroll
                        for (int i = 0; i < TPW; ++i) Ac[i] = R1[p * FX_G + cc][i];
                        const int c1 = min(c + P1, XF_NCH1 - 1);
#pragma unroll
                        for (int i = 0; i < TPW; ++i) R1[p * FX_G + cc][i] = ld_wfrag<SPLIT>(wrs, lane16, wb + c1 * 15 + wtile(i));
                        keep_loads();
                        F8 B[NAT];
#pragma unroll
                        for (int a = 0; a < NAT; ++a) B[a] = ld_frag<SPLIT>(sb(p * FX_G + cc, a), lane);
#pragma unroll
                        for (int i = 0; i < TPW; ++i)
                            if (i < nown) {
#pragma unroll
                                for (int a = 0; a < NAT; ++a) mma32<SPLIT>(acc[i][a], Ac[i], B[a]);
                            }
                    }
                }
                if (grp < NGRP - 1)
#pragma unroll
                    for (int q = 0; q < NF; ++q) dform(ta[q], tb[q], sb((p ^ 1) * FX_G + ph + NWA * q, wa));
                __syncthreads();
            };
            const std::integral_constant<int, 0> even;
            const std::integral_constant<int, 1> odd;
#pragma unroll 1
            for (int grp = 0; grp < NGRP - 1; grp += 2) {
                group(grp, even);
                group(grp + 1, odd);
            }
            static_assert(NGRP % 2 == 1, "the last group has an even number");
            group(NGRP - 1, even);
        }
        if constexpr (PH == FX_ALL) prefetch8(XF_W2F);
        // a1 = tanh(W1 D + b1), h1 = wh1 a1
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                const f4 b = vec4(FV_B1, t), wh = vec4(FV_WH1, t);
#pragma unroll
                for (int a = 0; a < NAT; ++a) {
                    f4 av;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        av[r] = tanh_fast(acc[i][a][r] + b[r]);
                        h[i][a][r] = wh[r] * av[r];
                    }
                    *sptr(0, t, a) = av;
                    if constexpr (PH == FX_ALL) st_half<SPLIT>(sb(t >> 1, a), lane, t & 1, h[i][a]);
                }
            }
        if constexpr (PH == FX_ALL) {
            zero_tile15();
            __syncthreads();
        }
    }
    if constexpr (PH == FX_MID) {
        prefetch8(XF_W2F);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                const f4 wh = vec4(FV_WH1, t);
#pragma unroll
                for (int a = 0; a < NAT; ++a) {
                    const f4 av = *sptr(0, t, a);
#pragma unroll
                    for (int r = 0; r < 4; ++r) h[i][a][r] = wh[r] * av[r];
                    st_half<SPLIT>(sb(t >> 1, a), lane, t & 1, h[i][a]);
                }
            }
        zero_tile15();
        __syncthreads();
    }
    if constexpr (PH == FX_ALL || PH == FX_MID) {
        // ------------------------------------------------------------ layers 2, 3: h += wh tanh(W h + b)
#pragma unroll 1
        for (int layer = 2; layer <= 3; ++layer) {
            gemm8(layer == 2 ? XF_W2F : XF_W3F);
            prefetch8(layer == 2 ? XF_W3F : XF_W3B);
            __syncthreads();
            const int ob = layer == 2 ? FV_B2 : FV_B3, ow = layer == 2 ? FV_WH2 : FV_WH3;
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (i < nown) {
                    const int t = ftile(i);
                    const f4 b = vec4(ob, t), wh = vec4(ow, t);
#pragma unroll
                    for (int a = 0; a < NAT; ++a) {
                        f4 av;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            av[r] = tanh_fast(acc[i][a][r] + b[r]);
                            h[i][a][r] += wh[r] * av[r];
                        }
                        *sptr(layer - 1, t, a) = av;
                        if (layer == 2) st_half<SPLIT>(sb(t >> 1, a), lane, t & 1, h[i][a]);
                    }
                }
            if (layer == 2) __syncthreads();
        }
        // ------------------------------------------------------------ energy E_i = wh4 (w4 . h3 + b4)
        {
            float e[NAT];
#pragma unroll
            for (int a = 0; a < NAT; ++a) e[a] = 0.f;
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (i < nown) {
                    const f4 w4 = vec4(FV_W4, ftile(i));
#pragma unroll
                    for (int a = 0; a < NAT; ++a)
#pragma unroll
                        for (int r = 0; r < 4; ++r) e[a] += w4[r] * h[i][a][r];
                }
            static_assert(NAT <= 4, "one energy sum per lane group");
            float ep[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int a = 0; a < NAT; ++a) ep[a] = e[a];
            const float es = sum_groups4(ep);
            if (ksel(g) < NAT) s_e[wave][16 * ksel(g) + c16] = es;
        }
        // ------------------------------------------------------------ backward through layers 3, 2
        // gh3 = wh4 w4, ga3 = gh3 wh3 (1 - a3^2); gh_{l-1} = W_l^T ga_l + gh_l, ga_l = gh_l wh_l (1 - a_l^2)
        const float wh4 = fv[FV_WH4];
#pragma unroll
        for (int i = 0; i < TPW; ++i)
            if (i < nown) {
                const int t = ftile(i);
                const f4 w4 = vec4(FV_W4, t), wh = vec4(FV_WH3, t);
#pragma unroll
                for (int a = 0; a < NAT; ++a) {
                    const f4 av = *sptr(2, t, a);
                    float ga[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        h[i][a][r] = wh4 * w4[r];
                        ga[r] = h[i][a][r] * wh[r] * (1.f - av[r] * av[r]);
                    }
                    st_half<SPLIT>(sb(t >> 1, a), lane, t & 1, ga);
                }
            }
        __syncthreads();
        if (threadIdx.x < NA) {
            const int at = a0 + threadIdx.x;
            if (at < A.natoms && A.itype[at] == ti)
            {
                double es = 0.0;
                for (int w = 0; w < NW; ++w) es += (double)s_e[w][threadIdx.x];
                A.Ei[at] = (double)wh4 * (es + (double)fv[FV_B4]);
            }
        }
#pragma unroll 1
        for (int layer = 3; layer >= 2; --layer) {
            gemm8(layer == 3 ? XF_W3B : XF_W2B);
            if (layer == 3) prefetch8(XF_W2B);
            __syncthreads();
            const int ow = layer == 3 ? FV_WH2 : FV_WH1;
#pragma unroll
            for (int i = 0; i < TPW; ++i)
                if (i < nown) {
                    const int t = ftile(i);
                    const f4 wh = vec4(ow, t);
#pragma unroll
                    for (int a = 0; a < NAT; ++a) {
                        const f4 av = *sptr(layer - 2, t, a);
                        float ga[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            h[i][a][r] += acc[i][a][r];
                            ga[r] = h[i][a][r] * wh[r] * (1.f - av[r] * av[r]);
                        }
                        st_half<SPLIT>(sb(t >> 1, a), lane, t & 1, ga);
                    }
                }
            __syncthreads();
        }
    }
    // what the launch of the dD phase reads and writes in the block's scratch (see FX_ALL above)
    constexpr int SLOT = 16 * NAT * 256;   // floats per layer slot
    static_assert(XF_NCH2 * NAT * XF_ELEMS * 2 == SLOT * 4, "ga1 fills a slot");
    float *p1g = scr, *q2g = scr + SLOT;
    if constexpr (PH == FX_MID) {
        for (int e = threadIdx.x; e < SLOT / 4; e += 64 * NW)
            reinterpret_cast<f4*>(scr + 2 * SLOT)[e] = reinterpret_cast<const f4*>(s_b)[e];
    }
    // rows n < 16 of dT: part 1 + the four row groups' part 2 (slot (row group, atom tile) [lane][16])
    auto add_part2 = [&](auto&& p1, const float* q2) {
        for (int idx = threadIdx.x; idx < NA * 16; idx += 64 * NW) {
            const int al = idx >> 4, n = idx & 15;
            const int at = a0 + al;
            if (at < A.natoms && A.itype[at] == ti) {
                const int a = al >> 4, lp = (n >> 2) * 16 + (al & 15), r = n & 3;
                f4 v = *reinterpret_cast<const f4*>(p1(al, n));
#pragma unroll
                for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const f4*>(q2 + ((w * NAT + a) * 64 + lp) * 16 + 4 * r);
                *reinterpret_cast<f4*>(dTg + ((size_t)at * E2 + n) * 4) = v;
            }
        }
    };
    if constexpr (PH == FX_ALL) {
        // ------------------------------------------------------------ dD = W1 ga1 and dT
        // D-row tile m of dD holds dD[m][n = 4g + r] for 16 atoms. dT[m][k] collects
        // sum_n dD[m][n] T[n][k] (part 1, reduced over lane groups) and, for rows n < 16,
        // sum_m dD[m][n] T[m][k] (part 2, q2, per wave; reduced over waves at the end).
        // Waves 0 to 3 (one per SIMD) form the D rows mw + 4p of pass p for all atom tiles of the block,
        // so that each W1 fragment is read once, and hand them through LDS (two buffers, one barrier
        // per pass) to waves 4 to 7, which form dT and write it. The products, which bound the phase,
        // then wait neither for the epilogue's dependent sums nor, on the in-order memory counter, for
        // its stores. The weights are the latency: 4.16 MB per species do not stay in an XCD's L2, and a
        // fragment takes about 2,500 cycles to arrive, so two passes of fragments are in flight. Cycles of
        // a 64-atom (32-atom) block: rows and atom tiles split over all eight waves, each doing both,
        // 124,000 (86,000); as here with 4 fragments per wave in flight 161,000 (125,000), 8: 101,000
        // (82,000), 16: 93,000 (72,000).
        float* qs = reinterpret_cast<float*>(s_b);
        {
            constexpr int NPASS = E2 / 4, PDD = 16;       // PDD: K-chunks of weights in flight (two passes)
            static_assert(NW == 8 && PDD == 2 * XF_NCH2, "four product and four epilogue waves; ring slots by pass parity");
            const int mw = wave & 3;
            auto dslot = [&](int p, int a) { return reinterpret_cast<f4*>(&s_dd[p & 1][mw][a][lane][0]); };
            if (wave < 4) {
                // the fragments of the next two passes (clamped at the end: unconditional reads)
                auto wfrag = [&](int p, int c) {
                    return ld_wfrag<SPLIT>(wrs, lane16, XF_W1B + (mw + 4 * min(p, NPASS - 1)) * XF_NCH2 + c);
                };
                F8 RD[PDD];
#pragma unroll
                for (int d = 0; d < PDD; ++d) RD[d] = wfrag(d / XF_NCH2, d % XF_NCH2);
                auto pass = [&](int p, auto par) {
                    f4 dd[NAT];
#pragma unroll
                    for (int a = 0; a < NAT; ++a) dd[a] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int c = 0; c < XF_NCH2; ++c) {
                        const int sl = par.value * XF_NCH2 + c;
                        const F8 Ac = RD[sl];
                        RD[sl] = wfrag(p + 2, c);
                        keep_loads();
                        F8 B[NAT];
#pragma unroll
                        for (int a = 0; a < NAT; ++a) B[a] = ld_frag<SPLIT>(sb(c, a), lane);
#pragma unroll
                        for (int a = 0; a < NAT; ++a) mma32<SPLIT>(dd[a], Ac, B[a]);
                    }
#pragma unroll
                    for (int a = 0; a < NAT; ++a) *dslot(p, a) = dd[a];
                    __syncthreads();
                };
                const std::integral_constant<int, 0> even;
                const std::integral_constant<int, 1> odd;
#pragma unroll 1
                for (int p = 0; p < NPASS - 1; p += 2) {
                    pass(p, even);
                    pass(p + 1, odd);
                }
                static_assert(NPASS % 2 == 1, "the last pass has an even number");
                pass(NPASS - 1, even);
                __syncthreads();   // (the epilogue waves' q2, below)
            } else {
                f4 tn[NAT][4];     // T rows 4g..4g+3 of this lane's atoms
                float q2[NAT][4][4];
                const float* Td[NAT];
                // where this lane's component of dT goes: rows of its atom, or (no such atom) one word of
                // the block's scratch, so that the stores stand under no branch: the compiler then knows
                // how many are in flight, and the T rows, read two passes ahead, wait for none of them
                float* dst[NAT];
                int dstep[NAT];
#pragma unroll
                for (int a = 0; a < NAT; ++a) {
                    const int at = a0 + 16 * a + c16;
                    const bool mined = at < A.natoms && A.itype[at] == ti;
                    Td[a] = Tg + (size_t)(at < A.natoms ? at : a0) * (E2 * 4);
                    dst[a] = mined ? dTg + (size_t)at * (E2 * 4) + ksel(g) : scr + threadIdx.x;
                    dstep[a] = mined ? 4 : 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        tn[a][r] = *reinterpret_cast<const f4*>(&s_tq[16 * a + c16][4 * g + r][0]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) q2[a][r][k] = 0.f;
                    }
                }
                f4 tm[2][NAT];     // rows T[m] of passes p and p + 1
                auto trow = [&](int p, f4* t) {
#pragma unroll
                    for (int a = 0; a < NAT; ++a)
                        t[a] = *reinterpret_cast<const f4*>(Td[a] + (mw + 4 * min(p, NPASS - 1)) * 4);
                };
                trow(0, tm[0]);
                trow(1, tm[1]);
                auto pass = [&](int p, auto slot, auto low) {   // low: rows m < 16, kept in LDS
                    const int m = mw + 4 * p;
                    __syncthreads();
                    f4 t[NAT];
#pragma unroll
                    for (int a = 0; a < NAT; ++a) t[a] = tm[slot.value][a];
                    trow(p + 2, tm[slot.value]);
#pragma unroll
                    for (int a = 0; a < NAT; ++a) {
                        const f4 dd = *dslot(p, a);
                        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                part[k] += dd[r] * tn[a][r][k];
                                q2[a][r][k] += dd[r] * t[a][k];
                            }
                        const float pk = sum_groups4(part);   // lane group g: component ksel(g)
                        if constexpr (low.value) s_p1[16 * a + c16][m][ksel(g)] = pk;
                        else dst[a][m * dstep[a]] = pk;
                    }
                };
                const std::integral_constant<int, 0> s0;
                const std::integral_constant<int, 1> s1;
                const std::true_type low;
                const std::false_type high;
                pass(0, s0, low);
                pass(1, s1, low);
                pass(2, s0, low);
                pass(3, s1, low);
#pragma unroll 1
                for (int p = 4; p < NPASS - 1; p += 2) {
                    pass(p, s0, high);
                    pass(p + 1, s1, high);
                }
                static_assert(NPASS % 2 == 1, "the last pass has an even number");
                pass(NPASS - 1, s0, high);
                // part 2 partials: slot (row group, atom tile) [lane][16], each written by one wave (the
                // product waves are done with ga1 in s_b since the last pass's barrier)
#pragma unroll
                for (int a = 0; a < NAT; ++a)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<f4*>(qs + ((mw * NAT + a) * 64 + lane) * 16 + 4 * r) =
                            f4{q2[a][r][0], q2[a][r][1], q2[a][r][2], q2[a][r][3]};
                __syncthreads();
            }
            add_part2([&](int al, int n) { return &s_p1[al][n][0]; }, qs);
        }
    }
    if constexpr (PH == FX_DD) {
        // As below, for the rows m = sub + 4 p: waves 0 to 3 form the rows of the passes p = w + 4 j of round
        // j, wave 4 + a the dT of atom tile a from the round's four rows in the order of p.
        static_assert(NW == 8 && NAT <= 4, "four product waves, an epilogue wave per atom tile");
        constexpr int NPASS = E2 / 4, NRND = (NPASS + 3) / 4;
        float* none = scr + 15 * NAT * 256;
        for (int e = threadIdx.x; e < SLOT / 4; e += 64 * NW)
            reinterpret_cast<f4*>(s_b)[e] = reinterpret_cast<const f4*>(scr + 2 * SLOT)[e];
        stage_tq();
        auto dslot = [&](int j, int w, int a) { return reinterpret_cast<f4*>(&s_dd[j & 1][w][a][lane][0]); };
        if (wave < 4) {
            auto wfrag = [&](int j, int c) {
                return ld_wfrag<SPLIT>(wrs, lane16, XF_W1B + (sub + 4 * min(wave + 4 * j, NPASS - 1)) * XF_NCH2 + c);
            };
            F8 RD[2 * XF_NCH2];
#pragma unroll
            for (int d = 0; d < 2 * XF_NCH2; ++d) RD[d] = wfrag(d / XF_NCH2, d % XF_NCH2);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NRND; ++j) {
                f4 dd[NAT];
#pragma unroll
                for (int a = 0; a < NAT; ++a) dd[a] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < XF_NCH2; ++c) {
                    const int sl = (j & 1) * XF_NCH2 + c;
                    const F8 Ac = RD[sl];
                    if (j + 2 < NRND) RD[sl] = wfrag(j + 2, c);
                    keep_loads();
                    F8 B[NAT];
#pragma unroll
                    for (int a = 0; a < NAT; ++a) B[a] = ld_frag<SPLIT>(sb(c, a), lane);
#pragma unroll
                    for (int a = 0; a < NAT; ++a) mma32<SPLIT>(dd[a], Ac, B[a]);
                }
#pragma unroll
                for (int a = 0; a < NAT; ++a) *dslot(j, wave, a) = dd[a];
                __syncthreads();
            }
        } else {
            const int a = min(wave - 4, NAT - 1), at = a0 + 16 * a + c16;
            const bool own = wave - 4 < NAT, mined = at < A.natoms && A.itype[at] == ti;
            const float* Td = Tg + (size_t)(at < A.natoms ? at : a0) * (E2 * 4);
            float* dst = mined ? dTg + (size_t)at * (E2 * 4) + ksel(g) : none + threadIdx.x;
            const int dstep = mined ? 4 : 0;
            f4 tn[4], tm[4];   // T rows 4g..4g+3 of this lane's atom; rows of the round's passes
            float q2[4][4];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                tn[r] = *reinterpret_cast<const f4*>(&s_tq[16 * a + c16][4 * g + r][0]);
#pragma unroll
                for (int k = 0; k < 4; ++k) q2[r][k] = 0.f;
            }
            auto trow = [&](int p) { return *reinterpret_cast<const f4*>(Td + (sub + 4 * min(p, NPASS - 1)) * 4); };
#pragma unroll
            for (int w = 0; w < 4; ++w) tm[w] = trow(w);
#pragma unroll
            for (int j = 0; j < NRND; ++j) {
                __syncthreads();
                if (own) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int p = w + 4 * j, m = sub + 4 * p;
                        if (p >= NPASS) continue;
                        const f4 t = tm[w], dd = *dslot(j, w, a);
                        tm[w] = trow(p + 4);
                        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                part[k] += dd[r] * tn[r][k];
                                q2[r][k] += dd[r] * t[k];
                            }
                        const float pk = sum_groups4(part);   // lane group g: component ksel(g)
                        if (p < 4) p1g[((16 * a + c16) * 16 + m) * 4 + ksel(g)] = pk;
                        else dst[m * dstep] = pk;
                    }
                }
            }
            if (own)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<f4*>(q2g + ((sub * NAT + a) * 64 + lane) * 16 + 4 * r) = f4{q2[r][0], q2[r][1], q2[r][2], q2[r][3]};
        }
    }
    if constexpr (PH == FX_SUM) add_part2([&](int al, int n) { return p1g + (al * 16 + n) * 4; }, q2g);
}

}  // namespace

template <int NAT, int NW, int PH>
static void launch_fitx_phase(bool split, int sub, const FitArgs& a, hipStream_t s)
{
    const bool ens = a.nmodels > 1;
    dim3 grid(((a.natoms + 16 * NAT - 1) / (16 * NAT) + a.ntypes) * sub, ens ? a.nmodels : 1), block(64 * NW);
    // ens: one launch for a model ensemble, blockIdx.y = model (a separate instantiation)
    if (split) {
        if (ens) hipLaunchKernelGGL((k_fitx<NAT, true, NW, true, PH>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_fitx<NAT, true, NW, false, PH>), grid, block, 0, s, a);
    } else {
        if (ens) hipLaunchKernelGGL((k_fitx<NAT, false, NW, true, PH>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_fitx<NAT, false, NW, false, PH>), grid, block, 0, s, a);
    }
}

// Block shape: 64 atoms when the frame fills the CUs, so that the weights a block streams serve more
// atoms; 32 atoms while the 64-atom blocks would leave half of the CUs idle (8,100 atoms: 86 us). In steps
// while the blocks of the split phases fit the CUs at once (a block per CU): 192 atoms 51 us against 76 in
// one launch, 1,890 atoms 59 against 77; past that the steps lose it again (3,000: 75 and 77, 4,200: 95 and
// 78).
void launch_fitx(bool split, const FitArgs& a, hipStream_t s)
{
    if (a.natoms <= 0) return;
    const int64_t blocks64 = ((int64_t)a.natoms + 63) / 64 * (a.nmodels > 1 ? a.nmodels : 1);
    const int64_t ncu = a.ncu > 0 ? a.ncu : 256, models = a.nmodels > 1 ? a.nmodels : 1;
    const int64_t blocks32 = (((int64_t)a.natoms + 31) / 32 + a.ntypes) * models;
    if (blocks32 * FX_SUB <= ncu) {
        launch_fitx_phase<2, 4, FX_L1>(split, FX_SUB, a, s);
        launch_fitx_phase<2, 8, FX_MID>(split, 1, a, s);
        launch_fitx_phase<2, 8, FX_DD>(split, FX_SUB, a, s);
        launch_fitx_phase<2, 8, FX_SUM>(split, 1, a, s);
    } else if (blocks64 * 2 <= ncu) {
        launch_fitx_phase<2, 8, FX_ALL>(split, 1, a, s);
    } else {
        launch_fitx_phase<4, 8, FX_ALL>(split, 1, a, s);
    }
}

}  // namespace dpk
