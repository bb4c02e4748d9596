// dpk_train.h -- internal declarations of the training-mode backward (Sec. II.B), FP64: the kernels of
// the embedding nets (kernels_tre.hip) and of the fitting nets, the loss and Adam (kernels_train.hip),
// and the frame hooks of the inference path they start from.
//
// With g_ij = dE/dr_ij, the force and virial terms of the loss are linear in the g_ij, so
//   dL/dtheta = d/dtheta [ cE E + sum_ij g_ij . rdot_ij ],
//   cE = 2 p_E (E - E*) / N,  rdot_ij = vdir_j - vdir_i + CV r_ij,
//   vdir_k = -2 p_F q_k (F_k - F*_k) / (3N),  CV = -2 p_Xi (Xi - Xi*) / (9N),
// and sum_ij g_ij . rdot_ij is the derivative of E along the pair displacements rdot_ij: a
// forward-mode tangent through the model (s, R, G = N(s), T, D, F_0), then reverse mode through
// the model and its tangent.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dpk_internal.h"
#include "train_window.h"

struct dpk_ctx;
struct dpk_model;

namespace dpk {

// The frame as the inference launches left it (internal atom order), on the context's stream.
struct FrameNet {
    int n, nt, ncu;
    EmbArgs emb;           // geometry, packed embedding weights and cut-offs of the embedding kernels
    const int* toff;       // [nt + 1] internal type offsets (device)
    const int* nnei;       // [n][nt]
    const int* perm;       // [n] caller index of each internal atom
    const double* T;       // [n][100][4]
    const double* F;       // [n][3] caller order
    hipStream_t stream;
};
// Partition, bin and search one host frame on the context's device and stream and queue the network and
// its adjoint with the context's packed weights; E and the virial [9] go to ev (device, 10 doubles). Waits
// for the geometry only (its errors are reported here), and for the chunk offsets: coff (device, nt (n + 1))
// is filled and *chunks (pinned) their number. The context keeps the buffers until its next frame.
int frame_network(dpk_ctx* c, int64_t natoms, const double* coord, const int32_t* atype, const double* box, double* ev,
                  int* coff, int* chunks, FrameNet* f);
// The context's packed FP64 weights (device) in four buffers: embedding vectors and matrices, fitting
// vectors and matrices.
struct PackedWeights {
    double* p[4];
    int64_t n[4];
    hipStream_t stream;    // the context's stream
};
void packed_weights(dpk_ctx* c, PackedWeights* w);
const double* model_params(const dpk_model* m);   // host, in the blob's order
dpk_model* numbered_model(const dpk_model* m);    // of m's description, the parameters 1, 2, 3, ...

// Loss, its coefficients and the energy and virial of the frame (device).
struct TrCoef {
    double cE, CV[9];
    double loss[4];
    double ev[10];
};

// Packing maps: map[i] = parameter index of packed value i, or -1 (a padding zero), from weights packed
// out of the parameter vector 1, 2, 3, ...; and the packing itself.
void tr_map(const double* packed, int64_t n, int* map, hipStream_t s);
void tr_pack(const double* theta, const int* map, int64_t n, double* packed, hipStream_t s);

// vdir [n][3] (caller order) and the loss terms from the prediction; labels NULL: the term is left out.
struct TrLossArgs {
    int n;
    const double* F;              // prediction (caller order)
    const double *fl, *q;         // force labels [n][3], per-atom prefactors [n] or nullptr
    double el, vl[9];
    int has_e, has_v;
    double pe, pf, pv, weight;
    double* vdir;
    double* part;                 // [blocks] partial force loss
    TrCoef* coef;                 // ev filled on entry
};
int tr_loss_blocks(int n);
void tr_loss(const TrLossArgs& a, hipStream_t s);

// Embedding nets. Chunks of 16 kept neighbours of one atom and neighbour type; coff [nt][n + 1] their
// offsets (by neighbour type, then atom). dump: TRE_CHUNK doubles per chunk, for a window of chunks at a
// time: 66.5 KB per chunk would otherwise hold 16 kept neighbours or one alike, and a frame of many types
// with few neighbours of each needs a chunk for almost every pair (train_window.h).
constexpr int TRE_CHUNK = 130 * 64;
// Adjoints of T and Td of an atom, over N_c: [layer-3 row position][T 4, Td 4], padding rows zero
constexpr int TRE_TB = N3P * 8;
constexpr int TRE_NET = 3 * E0 + E0 * E1 + 2 * E1 + E1 * E2 + 2 * E2;   // parameters of one embedding net
// Copies of the embedding gradients that the blocks add to: a multiple of the XCDs while that is a few MB
// (with more nets fewer blocks meet at an address).
inline int tre_copies(int nets) { return nets <= 4 ? 32 : nets <= 9 ? 16 : nets <= 16 ? 8 : 1; }
struct TreArgs {
    EmbArgs e;
    const int* toff;
    const int* coff;
    int4* cmap;                   // [chunks]
    const double* vdir;
    const TrCoef* coef;
    double* Td;                   // [n][100][4] (tangent pass output)
    const double* Tb;             // [n][TRE_TB] adjoints of T and Td
    double* dump;                 // [window][TRE_CHUNK]
    int nets, nrep;
    double* rep;                  // [nrep][nets][TRE_NET], zero between frames
    double* grad;                 // gradient in the parameter layout (embedding nets first)
    int chunks, window;           // chunks of the frame, and at most as many of them at a time
    int* woff;                    // as coff, of a window (window < chunks)
};
// Chunk offsets; coff[nt - 1][n] is the number of chunks.
void tre_offsets(int n, int nt, const int* nnei, int* coff, hipStream_t s);
void tre_tangent(const TreArgs& k, hipStream_t s);    // Td
void tre_gradient(const TreArgs& k, hipStream_t s);   // embedding gradients (added)

// Fitting nets: the atoms of type t are rows [toff[t], toff[t + 1]) of every buffer.
struct TrfArgs {
    int n, nt, max_rows;          // rows; types; the largest type's rows
    int rows[MAXT + 1];           // toff on the host
    const double* theta;
    double* grad;
    int64_t fit0;                 // parameter offset of the first fitting net
    const double *T, *Td;
    double* Tb;                   // [n][TRE_TB]
    double inv_nc;
    const TrCoef* coef;
    double *D, *Dd, *Db, *Ddb;    // [n][1600] descriptor, its tangent, their adjoints
    double *a[3], *y[3], *zd[3], *yd[3];   // [n][240] per layer: tanh, output, tangents of z and y
    double *zb[3], *zdb[3];       // [n][240] adjoints of the pre-activation and its tangent
    double *yb, *ydb;             // [n][240] adjoints of layer 2's output
};
// Forward with tangents from T and Td, reverse to Tb, every fitting gradient added.
void trf_run(const TrfArgs& a, int ncu, hipStream_t s);

// Adam (Kingma and Ba): m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// theta -= lr (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps); then g = 0.
void tr_adam(int64_t n, double* theta, double* g, double* m, double* v, double lr, double b1, double b2, double eps,
             double c1, double c2, hipStream_t s);

}  // namespace dpk
