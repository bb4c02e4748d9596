// emb_device.h -- device code shared by the embedding-net kernels: the precision policies (MFMA operand
// and result layouts), the launch shapes, the staging of a net in LDS and the walk over an atom's
// neighbour chunks.
//
// Matrix-core mapping (16x16 output tiles, one 64-lane wave): an MFMA computes D[i][j] += sum_k A[i][k]
// B[k][j] over a 16-wide K-chunk. Lane l supplies row i = l%16 of A and column j = l%16 of B, with the
// lane group g = l/16 holding the K values kidx(c, g, v), v = 0..3; the output holds D[orow(g, r)][l%16]
// in register r. The two maps depend on the instruction (see the policies); with them, the output of
// one tile is the B operand of the next K-chunk without any data movement.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include "dpk_device.h"
#include "dpk_internal.h"

namespace dpk {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// Precision policies
// ---------------------------------------------------------------------------------------------

// FP64: v_mfma_f64_16x16x4f64, four instructions per 16-wide K-chunk. Output register r of lane
// group g holds row g + 4r. Weight matrices are stored with each 16-wide K-chunk permuted so that
// the four K values a lane needs (g, g+4, g+8, g+12) are contiguous.
struct PF64 {
    typedef double acc;
    typedef double wt;
    typedef d4 accv;
    static constexpr int NPL = 1;
    static constexpr int KC = 16;    // K per fragment (four instructions)
    static constexpr int VPL = 4;    // K values per lane per fragment
    static constexpr int GB = 32;    // bytes of one lane's fragment in LDS
    struct frag { d4 v; };
    __device__ static int orow(int g, int r) { return g + 4 * r; }
    __device__ static int ogrp(int row) { return row & 3; }    // inverse of orow
    __device__ static int oreg(int row) { return row >> 2; }
    __device__ static int kidx(int c, int g, int v) { return 16 * c + g + 4 * v; }
    __device__ static frag make(acc x0, acc x1, acc x2, acc x3) { frag f; f.v = d4{x0, x1, x2, x3}; return f; }
    __device__ static frag make(const acc* x) { return make(x[0], x[1], x[2], x[3]); }
    __device__ static frag lds(const char* p) { return *reinterpret_cast<const frag*>(p); }
    __device__ static frag load(const wt* p, int64_t) {
        frag f;
        f.v = *reinterpret_cast<const d4*>(p);
        return f;
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b) {
        mma(d, a, b, 4);
    }
    // the first n of the fragment's four K values per lane (the others have zero weights)
    __device__ static void mma(accv& d, const frag& a, const frag& b, int n) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (v < n) d = __builtin_amdgcn_mfma_f64_16x16x4f64(a.v[v], b.v[v], d, 0, 0, 0);
    }
    __device__ static acc act(acc x, const double* th) { return tanh_tab(x, th); }
    // tanh(x + b) from the bias as staged (unscaled)
    __device__ static acc act_b(acc x, acc b, const double* th) { return tanh_tab(x + b, th); }
    static constexpr double BIAS_SCALE = 1.0;
};

// Split BF16 on v_mfma_f32_16x16x32_bf16: each FP32 operand is hi + lo with both parts BF16; the
// product is formed as lo*hi + hi*lo + hi*hi with FP32 accumulation, about 16 significant bits per
// operand. Lane group g supplies K values 8g..8g+7 of a 32-wide chunk; they are the logical
// indices kidx(c, g, v): rows 4g..4g+3 of output tile 2c (v < 4) and of tile 2c + 1 (v >= 4), so
// that a layer's output tiles feed the next layer's K-chunk in place (weights are stored with
// their K order permuted to match). Output register r of lane group g holds row 4g + r.
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ int kidx32(int c, int g, int v) { return 32 * c + (v < 4 ? 4 * g + v : 16 + 4 * g + (v - 4)); }

struct PMIX {
    typedef float acc;
    typedef __bf16 wt;
    typedef f4 accv;
    static constexpr int NPL = 2;
    static constexpr int KC = 32, VPL = 8, GB = 32;
    struct frag { bf8 h, l; };
    __device__ static int orow(int g, int r) { return 4 * g + r; }
    __device__ static int ogrp(int row) { return row >> 2; }   // inverse of orow
    __device__ static int oreg(int row) { return row & 3; }
    __device__ static int kidx(int c, int g, int v) { return kidx32(c, g, v); }
    __device__ static frag make(const acc* x) {
        frag f;
#pragma unroll
        for (int v = 0; v < 8; v += 2) {
            bf16x2_t h, l;
            split_bf16x2(x[v], x[v + 1], h, l);
            f.h[v] = h[0]; f.h[v + 1] = h[1];
            f.l[v] = l[0]; f.l[v + 1] = l[1];
        }
        return f;
    }
    __device__ static frag load(const wt* p, int64_t plane) {
        frag f;
        f.h = *reinterpret_cast<const bf8*>(p);
        f.l = *reinterpret_cast<const bf8*>(p + plane);
        return f;
    }
    __device__ static frag lds(const char* p) {
        frag f;
        f.h = *reinterpret_cast<const bf8*>(p);
        f.l = *reinterpret_cast<const bf8*>(p + 16);
        return f;
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b) {
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, d, 0, 0, 0);
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b, int) { mma(d, a, b); }
    __device__ static acc act(acc x) { return tanh_fast(x); }
    __device__ static acc act(acc x, const double*) { return tanh_fast(x); }
    // tanh(x + b) from the bias as staged (K b)
    __device__ static acc act_b(acc x, acc kb, const double*) { return tanh_scaled(__builtin_fmaf(x, TANH_K, kb)); }
    static constexpr float BIAS_SCALE = TANH_K;
};

// Plain BF16 operands on the same instruction, one product (fast, about 1e-2 relative force error).
struct PBF16 {
    typedef float acc;
    typedef __bf16 wt;
    typedef f4 accv;
    static constexpr int NPL = 1;
    static constexpr int KC = 32, VPL = 8, GB = 16;
    struct frag { bf8 h; };
    __device__ static int orow(int g, int r) { return 4 * g + r; }
    __device__ static int ogrp(int row) { return row >> 2; }   // inverse of orow
    __device__ static int oreg(int row) { return row & 3; }
    __device__ static int kidx(int c, int g, int v) { return kidx32(c, g, v); }
    __device__ static frag make(const acc* x) {
        frag f;
#pragma unroll
        for (int v = 0; v < 8; v += 2) {
            const bf16x2_t h = __builtin_convertvector((f32x2_t){x[v], x[v + 1]}, bf16x2_t);
            f.h[v] = h[0];
            f.h[v + 1] = h[1];
        }
        return f;
    }
    __device__ static frag load(const wt* p, int64_t) {
        frag f;
        f.h = *reinterpret_cast<const bf8*>(p);
        return f;
    }
    __device__ static frag lds(const char* p) {
        frag f;
        f.h = *reinterpret_cast<const bf8*>(p);
        return f;
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b) {
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, d, 0, 0, 0);
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b, int) { mma(d, a, b); }
    __device__ static acc act(acc x) { return tanh_fast(x); }
    __device__ static acc act(acc x, const double*) { return tanh_fast(x); }
    // tanh(x + b) from the bias as staged (K b)
    __device__ static acc act_b(acc x, acc kb, const double*) { return tanh_scaled(__builtin_fmaf(x, TANH_K, kb)); }
    static constexpr float BIAS_SCALE = TANH_K;
};

// FP32 on v_mfma_f32_16x16x4f32, four instructions per 16-wide K-chunk (the FP32 precision of
// the paper's reduced-precision inference, Sec. IV). In instruction v lane group g supplies one K
// value, register v of its fragment; with kidx(c, g, v) = 16c + 4g + v that is row 4g + v of the
// previous layer's output tile c, which is exactly what output register v of lane group g holds
// (orow(g, r) = 4g + r, probed on gfx950), so a layer's output is the next layer's B operand in
// place and the weights are stored in plain K order.
struct PF32 {
    typedef float acc;
    typedef float wt;
    typedef f4 accv;
    static constexpr int NPL = 1;
    static constexpr int KC = 16, VPL = 4, GB = 16;
    struct frag { f4 v; };
    __device__ static int orow(int g, int r) { return 4 * g + r; }
    __device__ static int ogrp(int row) { return row >> 2; }   // inverse of orow
    __device__ static int oreg(int row) { return row & 3; }
    __device__ static int kidx(int c, int g, int v) { return 16 * c + 4 * g + v; }
    __device__ static frag make(acc x0, acc x1, acc x2, acc x3) { frag f; f.v = f4{x0, x1, x2, x3}; return f; }
    __device__ static frag make(const acc* x) { return make(x[0], x[1], x[2], x[3]); }
    __device__ static frag lds(const char* p) { frag f; f.v = *reinterpret_cast<const f4*>(p); return f; }
    __device__ static frag load(const wt* p, int64_t) { frag f; f.v = *reinterpret_cast<const f4*>(p); return f; }
    __device__ static void mma(accv& d, const frag& a, const frag& b) {
        mma(d, a, b, 4);
    }
    __device__ static void mma(accv& d, const frag& a, const frag& b, int n) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (v < n) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[v], b.v[v], d, 0, 0, 0);
    }
    __device__ static acc act(acc x) { return tanh_fast(x); }
    __device__ static acc act(acc x, const double*) { return tanh_fast(x); }
    // tanh(x + b) from the bias as staged (K b)
    __device__ static acc act_b(acc x, acc kb, const double*) { return tanh_scaled(__builtin_fmaf(x, TANH_K, kb)); }
    static constexpr float BIAS_SCALE = TANH_K;
};

template <class V> __device__ __forceinline__ void zero4(V& v) { v[0] = 0; v[1] = 0; v[2] = 0; v[3] = 0; }

// Rank-1 updates on the matrix cores. v_mfma_f32_4x4x1f32 runs 16 independent 4 x 4 x 1 products,
// one per block of four lanes b: register i of lane 4b + j gains A(lane 4b + i) * B(lane 4b + j).
// With a = X[lane % 4] (an entry of a 4-vector X that is the same for the lane's quad) and b the
// lane's own scalar y, register k of every lane gains X[k] * y: 16 products per instruction, none
// wasted. The forward embedding kernel contracts T += G^T R this way (its layer-3 output puts one
// feature per lane and the neighbours in registers), the backward kernel dE/dR_j = G dT and
// dE/ds_j = (dG/ds) dT (one row m per lane quad, one neighbour per lane): the FMAs leave the vector
// ALUs and the accumulators the general registers.
__device__ __forceinline__ void outer4(f4& d, float a, float b)
{
    d = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, d, 0, 0, 0);
}


// Row stride of the forward pass's neighbour-major layer-2 buffer (64 rows used): a multiple of 4
// but not of 8, so the reads at (neighbour orow(g, r), row n) of the four lane groups fall in
// different banks, and rows stay 16-B aligned, so a lane's four consecutive rows go out as one
// 128-bit store (odd strides split them into 32-bit pairs: the bank-conflict counter rose 60 %).
constexpr int Z2S = 68;

// Launch shape of the embedding kernels: the waves of a block share one staged net; a block takes A.apb
// consecutive atoms, wave w of nw the atoms w, w + nw, ... of them. embed_shape chooses apb and nw per
// launch. Every path stages W3^T in LDS. At most NW waves per block: FP64 8 (network; two per SIMD, in
// at most 256 registers) or 4 (table; three blocks per CU). The FP32-accumulating policies run:
//   * forward (network): 16 waves, four per SIMD, in at most 128 VGPRs (the contraction's
//     accumulators live in the matrix cores' operands, see outer4): the extra waves per SIMD hide
//     more of the exp/rcp, MFMA and LDS latency;
//   * forward (table): 8 waves (the polynomial path needs more registers);
//   * backward: 12 waves, three per SIMD, in at most 168 VGPRs (skips in registers, the
//     contraction on the matrix cores, the pair sums of force and virial in LDS).
constexpr int EMB_MIN = 4;   // smallest block in atoms
template <class P, bool FWD = false, bool TAB = false> struct EmbCfg {
    typedef typename P::wt wt;
    static constexpr bool F64 = sizeof(typename P::acc) == 8;
    static constexpr int NW = F64 ? (TAB ? 4 : 8) : (FWD ? (TAB ? 8 : 16) : 12);
    static constexpr int APW_MAX = F64 ? 3 : (FWD ? (TAB ? 3 : 4) : 6);
    static constexpr int E3_APW = TAB ? 1 : 2;   // three-body backward: atoms per wave (slot gradients in LDS)
    static constexpr bool W3LDS = true;
    // LDS rows of staged weights: one lane's fragment per group (VPL K values; [hi lo] for split
    // BF16), rows padded by 16 B so 16 consecutive rows fall in distinct banks.
    static constexpr int ROW2 = (K2P / P::VPL) * P::GB + 16;
    static constexpr int ROW3 = (N2P / P::VPL) * P::GB + 16;
    static constexpr int NC1 = K2P / P::KC;     // K-chunks of layer 2 (input 25, padded)
    static constexpr int NC2 = N2P / P::KC;     // K-chunks of layer 3 (input 50, padded)
    // The skip-aligned order fills registers [0, NU1) of layer 1 and [0, NU2) of layer 2 (emb_feat;
    // group 0 has the most features); the others hold zeros, so their activations and, in the 4-deep
    // instructions, their K steps are left out. K values of chunk c in use: ku(NU, c).
    static constexpr int NU1 = emb_ns(0), NU2 = 2 * emb_ns(0);
    __device__ static constexpr int ku(int nu, int c) { return nu - c * P::VPL < P::VPL ? nu - c * P::VPL : P::VPL; }
};

// Fragment of row `row`, K-group `grp` (= 4 * chunk + lane group) from a staged block with `rowb`
// bytes per row.
template <class P>
__device__ __forceinline__ typename P::frag lds_frag(const char* base, int rowb, int row, int grp)
{
    return P::lds(base + row * rowb + grp * P::GB);
}

// Stage rows x K of a per-plane row-major matrix into LDS rows of fragment groups. Every thread issues
// the loads of up to STG groups before it stores the first (a load-store loop paid one memory latency
// per group; the last groups repeat, so that no load is under a branch).
template <class P>
__device__ void stage_rows(char* dst, int rowb, const typename P::wt* src, int64_t plane, int rows, int K)
{
    typedef typename P::wt wt;
    constexpr int STG = 4;
    typedef std::conditional_t<sizeof(wt) == 8, d4, u32x4> piece;
    const int G = K / P::VPL, n = rows * G;
    const int step = blockDim.x;
    for (int b0 = 0; b0 < n; b0 += STG * step) {
        piece h[STG], l[STG];
#pragma unroll
        for (int q = 0; q < STG; ++q) {
            if (b0 + q * step >= n) break;   // (uniform)
            const int i = min(b0 + q * step + (int)threadIdx.x, n - 1), row = i / G, grp = i - row * G;
            const wt* sp = src + (int64_t)row * K + P::VPL * grp;
            h[q] = *reinterpret_cast<const piece*>(sp);
            if constexpr (P::NPL == 2) l[q] = *reinterpret_cast<const piece*>(sp + plane);
        }
#pragma unroll
        for (int q = 0; q < STG; ++q) {
            if (b0 + q * step >= n) break;
            const int i = min(b0 + q * step + (int)threadIdx.x, n - 1), row = i / G, grp = i - row * G;
            char* d = dst + row * rowb + grp * P::GB;
            *reinterpret_cast<piece*>(d) = h[q];
            if constexpr (P::NPL == 2) *reinterpret_cast<piece*>(d + 16) = l[q];
        }
    }
}

// Stage one embedding net: vector block, W2^T and (split BF16) W3^T.
template <class P>
__device__ void stage_net(const EmbArgs& A, int net, typename P::acc* s_vec, char* s_w2, char* s_w3)
{
    typedef typename P::acc acc;
    typedef typename P::wt wt;
    typedef EmbCfg<P> Cfg;
    const acc* ev = reinterpret_cast<const acc*>(A.evec) + (size_t)net * EVEC;
    // biases of layers 2 and 3 staged pre-scaled for P::act_b
    for (int i = threadIdx.x; i < EVEC; i += blockDim.x) {
        const bool bias = (i >= EV_B2 && i < EV_B2 + N2P) || (i >= EV_B3 && i < EV_B3 + N3P);
        s_vec[i] = bias ? ev[i] * (acc)P::BIAS_SCALE : ev[i];
    }
    const int nets = A.type_one_side ? A.ntypes : A.ntypes * A.ntypes;
    const wt* src = reinterpret_cast<const wt*>(A.emat) + (size_t)net * EM_SIZE;
    const int64_t plane = (int64_t)nets * EM_SIZE;
    stage_rows<P>(s_w2, Cfg::ROW2, src + EM_W2T, plane, N2P, K2P);
    if (Cfg::W3LDS) stage_rows<P>(s_w3, Cfg::ROW3, src + EM_W3T, plane, N3P, N2P);
}

// Per-wave walk over (atom, 16-neighbour chunk) work items of one (type_i, type_j) pass, with the
// next item's neighbour vector and index loaded one item ahead. With LDSW the wave's atoms' type,
// neighbour count and caller index are loaded once per pass into a small LDS table (wl) and read
// from there when the walk reaches an atom: a global load there has to wait for every vector
// memory operation in flight (force atomics, prefetches), since that counter is in order. (The
// table backward pass uses it; in the network passes it cost more registers than it saved.)
constexpr int WL_MAX = 8;   // atoms per wave at most (APW_MAX)
template <bool LDSW = false>
struct ChunkWalk {
    int i, a, np, c0;
    int ac;   // caller index of atom a (backward pass)
    bool have;
    double px, py, pz;
    int pj;
    // wl: this wave's [2][WL_MAX] LDS table (type << 16 | neighbour count of atom k; its caller index)
    template <bool J = false>
    __device__ __forceinline__ void load_atoms(int* wl, const EmbArgs& A, int a0, int a1, int wave, int nw, int apw,
                                               int tj, int lane) {
        if (!LDSW) return;
        const int a = a0 + wave + nw * lane;
        if (lane < apw) {
            wl[lane] = a < a1 ? (A.itype[a] << 16) | A.nnei[(size_t)a * A.ntypes + tj] : -1;
            if (J) wl[WL_MAX + lane] = a < a1 ? A.perm[a] : 0;
        }
        wave_sync();
    }
    template <bool J = false>
    __device__ __forceinline__ bool find_atom(const EmbArgs& A, const int* wl, int a0, int a1, int wave, int nw,
                                              int apw, int ti, int tj, bool skip_empty) {
        for (; i < apw; ++i) {
            a = a0 + wave + nw * i;
            if (a >= a1) return false;
            if constexpr (LDSW) {
                const int tn = __builtin_amdgcn_readfirstlane(wl[i]);
                if ((tn >> 16) != ti) continue;
                np = tn & 0xffff;
                if (skip_empty && np == 0) continue;
                if (J) ac = __builtin_amdgcn_readfirstlane(wl[WL_MAX + i]);
            } else {
                if (A.itype[a] != ti) continue;
                np = A.nnei[(size_t)a * A.ntypes + tj];
                if (skip_empty && np == 0) continue;
                if (J) ac = A.perm[a];
            }
            return true;
        }
        return false;
    }
    // Prefetch of the chunk's r_ij; J: also the neighbour's caller index (the backward pass adds
    // forces in caller order). The reads are unconditional and their values used as read: a lane
    // past its atom's kept neighbours reads another slot of the atom's row (clamped to the row;
    // slot 0 once the walk has ended). Every slot of every row holds finite values (padding is
    // written as zero), and the kernels use r of such a lane only under `valid` or multiplied by
    // its zero s. A read under a branch, or a select of its value, makes the compiler wait for
    // this prefetch early (reads retire in order).
    template <bool J = false>
    __device__ __forceinline__ void fetch(const EmbArgs& A, int tj, int c16) {
        const int e = min(A.off[tj] + c0 + c16, A.nc - 1);
        const size_t slot = have ? (size_t)a * A.nc + e : 0;
        const double* v = A.nl_r + 3 * slot;
        px = v[0];
        py = v[1];
        pz = v[2];
        if (J) pj = A.nl_j[slot];
    }
};

}  // namespace dpk
