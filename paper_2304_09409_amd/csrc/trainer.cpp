// trainer.cpp -- the training path (Sec. II.B): per frame, the model's E, F and virial with the
// current parameters, the loss of eq. loss, and its parameter gradient from the forward-mode
// tangent along the loss's force/virial direction followed by reverse mode (kernels_tre.hip,
// kernels_train.hip); Adam steps and the learning-rate and prefactor schedules.
//
// Per frame, on the trainer's stream (the host waits for the geometry's error flags, while the
// network runs, and for the results at the end):
//   1. the inference pass: geometry, network and adjoint of the FP64 inference kernels, on weights
//      packed from the current parameters on the device;
//   2. the loss, cE = 2 p_E (E - E*)/N, the direction vdir = -2 p_F q (F - F*)/(3N) and
//      CV = -2 p_Xi (Xi - Xi*)/(9N) (times the frame weight);
//   3. the embedding nets' tangent, the fitting nets with tangents and their reverse pass, the
//      embedding nets' reverse pass, with every weight gradient.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "../../include/dpk.h"
#include "dpk_launch.h"
#include "dpk_train.h"

using namespace dpk;

namespace {

#define TRCHK(expr)                                                                                 \
    do {                                                                                            \
        hipError_t e_ = (expr);                                                                     \
        if (e_ != hipSuccess) return set_error(DPK_E_DEVICE, (std::string(#expr) + ": " + hipGetErrorString(e_)).c_str()); \
    } while (0)

// Device buffer that grows to the largest request (contents not kept).
struct DBuf {
    double* p = nullptr;
    size_t n = 0;
    hipError_t ensure(size_t need) {
        if (need <= n && p) return hipSuccess;
        if (p) hipFree(p);
        p = nullptr;
        n = 0;
        hipError_t e = hipMalloc((void**)&p, std::max<size_t>(need, 1) * sizeof(double));
        if (e == hipSuccess) n = need;
        return e;
    }
    ~DBuf() { if (p) hipFree(p); }
};
struct IBuf {
    int* p = nullptr;
    size_t n = 0;
    hipError_t ensure(size_t need) {
        if (need <= n && p) return hipSuccess;
        if (p) hipFree(p);
        p = nullptr;
        n = 0;
        hipError_t e = hipMalloc((void**)&p, std::max<size_t>(need, 1) * sizeof(int));
        if (e == hipSuccess) n = need;
        return e;
    }
    ~IBuf() { if (p) hipFree(p); }
};

}  // namespace

struct dpk_trainer {
    dpk_model* model = nullptr;   // private copy (description only: its parameters number the blob)
    dpk_ctx* geo = nullptr;       // FP64 context on the packed current parameters
    dpk_model_desc desc;
    int device = 0, nets = 0, nt = 0, nc = 0;
    int64_t np = 0;
    int64_t step = 0;
    bool stale = true;            // the packed weights are older than theta
    IBuf map;                     // packing maps of the four packed buffers, one after the other
    // the parameters, and what is cleared at the start: gradient, its copies, moments (one allocation)
    DBuf state;
    double *theta = nullptr, *grad = nullptr, *rep = nullptr, *mom1 = nullptr, *mom2 = nullptr;
    // frame workspace
    IBuf coff, cmap, woff;
    DBuf fl, q, vdir, part, coef, Td, Tb, dump;
    DBuf D, Dd, Db, Ddb, a[3], y[3], zd[3], yd[3], zb[3], zdb[3], yb, ydb;
    TrCoef* pin = nullptr;        // pinned copy of coef, and behind it the number of chunks
    ~dpk_trainer() {
        if (pin) hipHostFree(pin);
        if (geo) dpk_ctx_free(geo);
        if (model) dpk_model_free(model);
    }
};

namespace {

// The operand blocks of the frame's chunks, or of a window of them.
hipError_t dump_window(dpk_trainer* t, size_t chunks)
{
    return window_alloc(t->dump.n / TRE_CHUNK, chunks, hipSuccess, hipErrorOutOfMemory, [&](size_t n) {
        const hipError_t e = t->dump.ensure(n * TRE_CHUNK);
        if (e == hipErrorOutOfMemory) hipGetLastError();
        return e;
    });
}

int frame(dpk_trainer* t, int64_t natoms, const double* coord, const int32_t* atype, const double* box,
          const dpk_loss_spec* spec, double weight, double* loss, double* energy, double* force, double* virial)
{
    PackedWeights w;
    packed_weights(t->geo, &w);
    if (t->stale) {
        const int* map = t->map.p;
        for (int k = 0; k < 4; map += w.n[k++]) tr_pack(t->theta, map, w.n[k], w.p[k], w.stream);
        TRCHK(hipGetLastError());
        t->stale = false;
    }
    TrCoef* coef = (TrCoef*)t->coef.p;
    FrameNet f;
    if (natoms > 0 && natoms <= (1LL << 30)) TRCHK(t->coff.ensure((size_t)(natoms + 1) * t->nt));
    int* pin_chunks = (int*)(t->pin + 1);
    int rc = frame_network(t->geo, natoms, coord, atype, box, coef->ev, t->coff.p, pin_chunks, &f);
    if (rc) return rc;
    hipStream_t s = f.stream;
    const int n = f.n, nt = t->nt;
    const size_t nz = n, chunks = std::max(0, *pin_chunks);   // (the chunks as found, not as many as sel would allow)
    TRCHK(t->cmap.ensure(4 * chunks));
    for (DBuf* b : {&t->fl, &t->vdir}) TRCHK(b->ensure(3 * nz));
    TRCHK(t->q.ensure(nz));
    TRCHK(t->part.ensure(tr_loss_blocks(n)));
    TRCHK(t->Td.ensure(E2 * 4 * nz));
    TRCHK(t->Tb.ensure(TRE_TB * nz));
    for (DBuf* b : {&t->D, &t->Dd, &t->Db, &t->Ddb}) TRCHK(b->ensure((size_t)DD * nz));
    for (int l = 0; l < 3; ++l)
        for (DBuf* b : {&t->a[l], &t->y[l], &t->zd[l], &t->yd[l], &t->zb[l], &t->zdb[l]}) TRCHK(b->ensure((size_t)FW * nz));
    for (DBuf* b : {&t->yb, &t->ydb}) TRCHK(b->ensure((size_t)FW * nz));
    TRCHK(dump_window(t, chunks));   // (last: what the frame cannot do without comes first)
    const size_t window = std::min<size_t>(t->dump.n / TRE_CHUNK, TRE_WINDOW);
    if (window < chunks) TRCHK(t->woff.ensure((nz + 1) * nt));
    // loss and direction
    TrLossArgs la;
    std::memset(&la, 0, sizeof(la));
    la.n = n;
    la.F = f.F;
    if (spec->force) {
        TRCHK(hipMemcpyAsync(t->fl.p, spec->force, sizeof(double) * 3 * n, hipMemcpyHostToDevice, s));
        la.fl = t->fl.p;
        if (spec->atom_pref) {
            TRCHK(hipMemcpyAsync(t->q.p, spec->atom_pref, sizeof(double) * n, hipMemcpyHostToDevice, s));
            la.q = t->q.p;
        }
    }
    la.has_e = spec->energy != nullptr;
    if (spec->energy) la.el = *spec->energy;
    la.has_v = spec->virial != nullptr;
    if (spec->virial) std::memcpy(la.vl, spec->virial, sizeof(la.vl));
    la.pe = spec->pe;
    la.pf = spec->pf;
    la.pv = spec->pv;
    la.weight = weight;
    la.vdir = t->vdir.p;
    la.part = t->part.p;
    la.coef = coef;
    tr_loss(la, s);
    // training pass
    TreArgs e;
    e.e = f.emb;
    e.toff = f.toff;
    e.coff = t->coff.p;
    e.cmap = (int4*)t->cmap.p;
    e.vdir = t->vdir.p;
    e.coef = coef;
    e.Td = t->Td.p;
    e.Tb = t->Tb.p;
    e.dump = t->dump.p;
    e.chunks = (int)chunks;
    e.window = (int)window;
    e.woff = t->woff.p;
    e.nets = t->nets;
    e.nrep = tre_copies(t->nets);
    e.rep = t->rep;
    e.grad = t->grad;
    TrfArgs a;
    std::memset(&a, 0, sizeof(a));
    a.n = n;
    a.nt = nt;
    for (int64_t i = 0; i < natoms; ++i) a.rows[atype[i] + 1]++;   // (types checked by the geometry)
    for (int ty = 0; ty < nt; ++ty) {
        a.max_rows = std::max(a.max_rows, a.rows[ty + 1]);
        a.rows[ty + 1] += a.rows[ty];
    }
    a.theta = t->theta;
    a.grad = t->grad;
    a.fit0 = (int64_t)t->nets * TRE_NET;
    a.T = f.T;
    a.Td = t->Td.p;
    a.Tb = t->Tb.p;
    a.inv_nc = f.emb.inv_nc;
    a.coef = coef;
    a.D = t->D.p;
    a.Dd = t->Dd.p;
    a.Db = t->Db.p;
    a.Ddb = t->Ddb.p;
    for (int l = 0; l < 3; ++l) {
        a.a[l] = t->a[l].p;
        a.y[l] = t->y[l].p;
        a.zd[l] = t->zd[l].p;
        a.yd[l] = t->yd[l].p;
        a.zb[l] = t->zb[l].p;
        a.zdb[l] = t->zdb[l].p;
    }
    a.yb = t->yb.p;
    a.ydb = t->ydb.p;
    tre_tangent(e, s);
    trf_run(a, f.ncu, s);
    tre_gradient(e, s);
    TRCHK(hipGetLastError());
    TRCHK(hipMemcpyAsync(t->pin, coef, sizeof(TrCoef), hipMemcpyDeviceToHost, s));
    if (force) TRCHK(hipMemcpyAsync(force, f.F, sizeof(double) * 3 * n, hipMemcpyDeviceToHost, s));
    TRCHK(hipStreamSynchronize(s));
    if (loss) std::memcpy(loss, t->pin->loss, sizeof(t->pin->loss));
    if (energy) *energy = t->pin->ev[0];
    if (virial) std::memcpy(virial, t->pin->ev + 1, 9 * sizeof(double));
    return DPK_OK;
}

}  // namespace

extern "C" {

int dpk_trainer_create(const dpk_model* m, int device, dpk_trainer** out)
{
    if (!m || !out) return set_error(DPK_E_INVALID_ARG, "NULL argument");
    *out = nullptr;
    dpk_model_desc d;
    int rc = dpk_model_describe(m, &d, nullptr, nullptr, nullptr);
    if (rc) return rc;
    if (d.descriptor != DPK_SE_E2_A) return set_error(DPK_E_UNIMPLEMENTED, "training covers se_e2_a models");
    const int64_t np = dpk_model_param_count(&d);
    auto* t = new dpk_trainer;
    t->desc = d;
    t->device = device;
    t->nt = d.ntypes;
    t->nets = d.type_one_side ? d.ntypes : d.ntypes * d.ntypes;
    t->nc = 0;
    for (int ty = 0; ty < d.ntypes; ++ty) t->nc += d.sel[ty];
    t->np = np;
    // the context is packed from the numbers of the parameters, which gives the packing maps
    t->model = numbered_model(m);
    if ((rc = dpk_ctx_create(t->model, device, DPK_FP64, 0, 0, &t->geo))) {
        delete t;
        return rc;
    }
    PackedWeights w;
    packed_weights(t->geo, &w);
    const size_t nrep = (size_t)tre_copies(t->nets) * t->nets * TRE_NET, clear = 3 * (size_t)np + nrep;
    if (t->state.ensure(np + clear) != hipSuccess || t->map.ensure(w.n[0] + w.n[1] + w.n[2] + w.n[3]) != hipSuccess ||
        t->coef.ensure(sizeof(TrCoef) / sizeof(double)) != hipSuccess ||
        hipHostMalloc((void**)&t->pin, sizeof(TrCoef) + sizeof(int)) != hipSuccess) {
        hipGetLastError();
        delete t;
        return set_error(DPK_E_OOM, "hipMalloc of the trainer's parameter buffers failed");
    }
    t->theta = t->state.p;
    t->grad = t->theta + np;
    t->mom1 = t->grad + np;
    t->mom2 = t->mom1 + np;
    t->rep = t->mom2 + np;
    if (hipMemcpy(t->theta, model_params(m), sizeof(double) * np, hipMemcpyHostToDevice) != hipSuccess) {
        delete t;
        return set_error(DPK_E_DEVICE, "copy of the parameters to the device failed");
    }
    int* map = t->map.p;
    for (int k = 0; k < 4; map += w.n[k++]) tr_map(w.p[k], w.n[k], map, w.stream);
    // (cleared on the stream that the frames run on, which the null stream does not wait for or hold up)
    launch_zero(t->grad, sizeof(double) * clear, w.stream);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(w.stream) != hipSuccess) {
        delete t;
        return set_error(DPK_E_DEVICE, "clearing the gradient or building the packing maps failed");
    }
    *out = t;
    return DPK_OK;
}

void dpk_trainer_free(dpk_trainer* t)
{
    if (!t) return;
    hipSetDevice(t->device);
    hipDeviceSynchronize();
    delete t;
}

int dpk_trainer_accumulate(dpk_trainer* t, int64_t natoms, const double* coord, const int32_t* atype,
                           const double* box, const dpk_loss_spec* spec, double weight, double* loss,
                           double* energy, double* force, double* virial)
{
    if (!t || !coord || !atype || !spec) return set_error(DPK_E_INVALID_ARG, "NULL argument");
    TRCHK(hipSetDevice(t->device));
    return frame(t, natoms, coord, atype, box, spec, weight, loss, energy, force, virial);
}

int dpk_trainer_gradient(dpk_trainer* t, double* grad)
{
    if (!t || !grad) return set_error(DPK_E_INVALID_ARG, "NULL argument");
    TRCHK(hipSetDevice(t->device));
    TRCHK(hipDeviceSynchronize());
    TRCHK(hipMemcpy(grad, t->grad, sizeof(double) * t->np, hipMemcpyDeviceToHost));
    return DPK_OK;
}

int dpk_trainer_zero_grad(dpk_trainer* t)
{
    if (!t) return set_error(DPK_E_INVALID_ARG, "NULL trainer");
    TRCHK(hipSetDevice(t->device));
    TRCHK(hipDeviceSynchronize());
    PackedWeights w;
    packed_weights(t->geo, &w);
    launch_zero(t->grad, sizeof(double) * t->np, w.stream);   // (ordered with the next frame or step)
    TRCHK(hipGetLastError());
    return DPK_OK;
}

int dpk_trainer_adam_step(dpk_trainer* t, double lr, double beta1, double beta2, double eps)
{
    if (!t) return set_error(DPK_E_INVALID_ARG, "NULL trainer");
    if (!(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
        return set_error(DPK_E_INVALID_ARG, "need 0 <= beta1, beta2 < 1 and eps > 0");
    TRCHK(hipSetDevice(t->device));
    t->step += 1;
    t->stale = true;
    const double c1 = 1.0 - std::pow(beta1, (double)t->step), c2 = 1.0 - std::pow(beta2, (double)t->step);
    PackedWeights w;
    packed_weights(t->geo, &w);
    tr_adam(t->np, t->theta, t->grad, t->mom1, t->mom2, lr, beta1, beta2, eps, c1, c2, w.stream);
    TRCHK(hipGetLastError());
    TRCHK(hipDeviceSynchronize());
    return DPK_OK;
}

int dpk_trainer_params(dpk_trainer* t, double* params)
{
    if (!t || !params) return set_error(DPK_E_INVALID_ARG, "NULL argument");
    TRCHK(hipSetDevice(t->device));
    TRCHK(hipDeviceSynchronize());
    TRCHK(hipMemcpy(params, t->theta, sizeof(double) * t->np, hipMemcpyDeviceToHost));
    return DPK_OK;
}

int dpk_trainer_set_params(dpk_trainer* t, const double* params)
{
    if (!t || !params) return set_error(DPK_E_INVALID_ARG, "NULL argument");
    TRCHK(hipSetDevice(t->device));
    TRCHK(hipDeviceSynchronize());
    TRCHK(hipMemcpy(t->theta, params, sizeof(double) * t->np, hipMemcpyHostToDevice));
    t->stale = true;
    return DPK_OK;
}

double dpk_learning_rate(double lr0, double lr_stop, int64_t step, int64_t stop_steps, int64_t decay_steps)
{
    if (stop_steps <= 0 || decay_steps <= 0 || step < 0) return lr0;
    const double r = std::pow(lr_stop / lr0, (double)decay_steps / (double)stop_steps);
    return lr0 * std::pow(r, (double)(step / decay_steps));
}

double dpk_loss_prefactor(double p_start, double p_limit, double lr, double lr0)
{
    return p_limit * (1.0 - lr / lr0) + p_start * lr / lr0;
}

}  // extern "C"
