// kernels_geom.hip -- ingest, cell list and neighbour list of one frame (FP64 geometry).
//
// Compiled with FP contraction off: every coordinate difference, image shift and squared
// distance is evaluated with separately rounded multiplies and adds in a fixed order, so the
// neighbour selection (Sec. II.A: n(i), capacities padded to N_c; Sec. III.B.1: order by type,
// distance, index) is a deterministic function of the input bits.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "dpk_internal.h"
#include "dpk_launch.h"

namespace dpk {

__global__ void k_fill_zero(unsigned int* p, size_t nwords)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < nwords; i += stride) p[i] = 0u;
}

void launch_zero(void* p, size_t bytes, hipStream_t s)
{
    size_t words = (bytes + 3) / 4;
    if (!words) return;
    int blocks = (int)((words + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, s, (unsigned int*)p, words);
}

// Workspace of the allocation-free entry point: one array per device, held from the library's
// load until the process ends, shared by every call on that device. In host code `scratch` names
// a host-side stand-in; kernels get the device address that scratch_region looks up.
static __device__ __align__(256) char scratch[SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

int scratch_region(int device, void** ptr)
{
    if (device < 0 || device >= MAX_DEVICES) return -1;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        // the caller has made `device` current: this is that device's copy of the array
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return -1;
        }
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return 0;
}

// ---- atom types: validation, counts, stable partition by type (atoms are kept sorted by
// species so that each fitting GEMM and each embedding net runs over contiguous atoms; the order
// within a type is the caller order) ----
constexpr int TP_BLOCK = PREP_BLOCK;   // atoms per block of the multi-block preparation

__device__ __forceinline__ int clamp_type(int t, int ntypes) { return t < 0 ? 0 : (t >= ntypes ? ntypes - 1 : t); }

// Bounding box of an open cluster: out = {min xyz, max xyz}.
__global__ void __launch_bounds__(1024) k_bbox(int n, const double* coord, double* out)
{
    __shared__ double red[6][1024];
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
    for (int i = threadIdx.x; i < n; i += 1024)
        for (int c = 0; c < 3; ++c) {
            double x = coord[3 * (size_t)i + c];
            lo[c] = fmin(lo[c], x);
            hi[c] = fmax(hi[c], x);
        }
    for (int c = 0; c < 3; ++c) { red[c][threadIdx.x] = lo[c]; red[3 + c][threadIdx.x] = hi[c]; }
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int c = 0; c < 3; ++c) {
                red[c][threadIdx.x] = fmin(red[c][threadIdx.x], red[c][threadIdx.x + s]);
                red[3 + c][threadIdx.x] = fmax(red[3 + c][threadIdx.x], red[3 + c][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) out[threadIdx.x] = red[threadIdx.x][0];
}

// ---- fused preparation for frames of up to PS_MAX_ATOMS atoms and PS_MAX_CELLS bins --------
// One workgroup runs every preparation phase with barriers in between instead of seven dependent
// launches: type counts (ballots), the stable type partition (chunks of 1024 atoms in caller
// order, ballot ranks), wrap and bin (bin counts as LDS atomics), the bin scan, and the bin fill,
// which writes the candidate records directly. Results equal those of the multi-kernel path,
// except the order of atoms within a bin, which nothing downstream depends on (the neighbour
// list sorts its hits by a key that is unique per candidate).
constexpr int PS_THREADS = 1024;
constexpr int PS_APT = 8;                           // atoms per thread, held in registers
constexpr int PS_MAX_ATOMS = PS_THREADS * PS_APT;   // 8192
constexpr int PS_MAX_CELLS = 8192;

__device__ __forceinline__ void wrap_bin_one(const GeomParams& gp, const double* x, double* p, int* b)
{
    if (gp.periodic) {
        double s[3];
        for (int c = 0; c < 3; ++c) {
            s[c] = (x[0] * gp.hinv[c] + x[1] * gp.hinv[3 + c]) + x[2] * gp.hinv[6 + c];
            s[c] -= floor(s[c]);
            if (s[c] >= 1.0) s[c] = 0.0;
        }
        for (int c = 0; c < 3; ++c) p[c] = (s[0] * gp.h[c] + s[1] * gp.h[3 + c]) + s[2] * gp.h[6 + c];
        for (int c = 0; c < 3; ++c) {
            const int bb = (int)floor(s[c] * gp.nb[c]);
            b[c] = bb < 0 ? 0 : (bb >= gp.nb[c] ? gp.nb[c] - 1 : bb);
        }
    } else {
        for (int c = 0; c < 3; ++c) {
            p[c] = x[c];
            const int bb = (int)floor((x[c] - gp.origin[c]) / gp.binw[c]);
            b[c] = bb < 0 ? 0 : (bb >= gp.nb[c] ? gp.nb[c] - 1 : bb);
        }
    }
}

// One frame's preparation in one workgroup. Single frame (BATCH = false): counts the types itself
// and zeroes the statistics block. Frame f of a batch (BATCH = true): the per-type internal bases
// come from k_batch_scan; atoms, candidate records and bins sit at the frame's offsets.
// Ghost atoms (single frame, caller indices nlocal.. n - 1; nlocal = n without ghosts) form one
// more partition class after the types, so the owned atoms take internal positions 0.. nlocal - 1
// sorted by type; itype and the candidate records keep every atom's real type.
template <bool BATCH>
__device__ __forceinline__ void prep_frame(int f, int n, int nlocal, int atom_off, const double* coord, const int* atype,
                                           int ntypes, const GeomParams& gp, int ncell, int cell_off,
                                           const int* type_base, int* tcount, int* toff, int* perm, int* inv_perm,
                                           int* itype, int* frame_of, DevStats* st, double* pos, int* cell_of,
                                           int* cell_start, double4* cand, double* f_int, double* vir_atom)
{
    __shared__ int s_cnt[PS_MAX_CELLS];        // bin counts, then bin cursors
    __shared__ int s_w[PS_THREADS / 64][MAXT]; // per-wave type counts
    __shared__ int s_base[MAXT];               // next internal position per type
    __shared__ int s_part[PS_THREADS];         // scan partials
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (!BATCH)
        clear_stats(st, tid, PS_THREADS);
    for (int c = tid; c < ncell; c += PS_THREADS) s_cnt[c] = 0;
    if (BATCH && tid < ntypes) s_base[tid] = type_base[tid];
    __syncthreads();   // the statistics block is zero before anything raises a flag in it
    // types of this thread's atoms tid + PS_THREADS j, read once; tv is the partition class (the
    // type, or ntypes for a ghost), rv the type
    const int ncls = ntypes + (nlocal < n ? 1 : 0);
    int tv[PS_APT], rv[PS_APT];
    bool bad = false;
#pragma unroll
    for (int j = 0; j < PS_APT; ++j) {
        const int a = tid + PS_THREADS * j;
        const int t0 = a < n ? atype[atom_off + a] : 0;
        bad |= t0 < 0 || t0 >= ntypes;
        rv[j] = clamp_type(t0, ntypes);
        tv[j] = a < n ? (a < nlocal ? rv[j] : ntypes) : -1;
    }
    if (!BATCH) {
        if (__ballot(bad) != 0 && lane == 0) atomicExch(&st->err_type, 1);
        for (int k = 0; k < ncls; ++k) {
            int v = 0;
#pragma unroll
            for (int j = 0; j < PS_APT; ++j) v += tv[j] == k;
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane == 0) s_w[wid][k] = v;
        }
        __syncthreads();
        if (tid == 0) {
            int acc = 0;
            for (int k = 0; k < ncls; ++k) {
                int c = 0;
                for (int w = 0; w < PS_THREADS / 64; ++w) c += s_w[w][k];
                toff[k] = acc;
                tcount[k] = c;
                s_base[k] = acc;
                acc += c;
            }
            toff[ncls] = acc;
        }
        __syncthreads();
    }
    // stable partition by type: chunk j = atoms PS_THREADS j .. in caller order; this thread's
    // internal positions are kept for the next phase
    int qv[PS_APT];
#pragma unroll
    for (int j = 0; j < PS_APT; ++j) {
        qv[j] = -1;
        if (PS_THREADS * j >= n) continue;   // uniform
        const int a = tid + PS_THREADS * j;
        const int t = tv[j];
        unsigned long long mine = 0;
        for (int k = 0; k < (BATCH ? ntypes : ncls); ++k) {
            const unsigned long long m = __ballot(t == k);
            if (t == k) mine = m;
            if (lane == 0) s_w[wid][k] = __popcll(m);
        }
        __syncthreads();
        if (t >= 0) {
            int before = s_base[t];
            for (int w = 0; w < wid; ++w) before += s_w[w][t];
            const int q = before + __popcll(mine & lt);
            qv[j] = q;
            perm[q] = atom_off + a;
            inv_perm[atom_off + a] = q;
            itype[q] = rv[j];
            if (BATCH) frame_of[q] = f;
        }
        __syncthreads();
        if (tid < (BATCH ? ntypes : ncls)) {
            int c = 0;
            for (int w = 0; w < PS_THREADS / 64; ++w) c += s_w[w][tid];
            s_base[tid] += c;
        }
        __syncthreads();
    }
    // wrap and bin this thread's atoms (caller index atom_off + a, internal index qv[j]); zero the
    // frame's force (and, batched, virial) accumulators
    double xv[PS_APT][3];
#pragma unroll
    for (int j = 0; j < PS_APT; ++j) {
        const int a = atom_off + tid + PS_THREADS * j;
        for (int c = 0; c < 3; ++c) xv[j][c] = qv[j] >= 0 ? coord[3 * (size_t)a + c] : 0.0;
    }
    int cv[PS_APT];
#pragma unroll
    for (int j = 0; j < PS_APT; ++j) {
        cv[j] = -1;
        const int q = qv[j];
        if (q < 0) continue;
        double p[3];
        int b[3];
        wrap_bin_one(gp, xv[j], p, b);
        for (int c = 0; c < 3; ++c) {
            pos[3 * (size_t)q + c] = p[c];
            xv[j][c] = p[c];
            f_int[3 * (size_t)q + c] = 0.0;
        }
        if (BATCH)
            for (int k = 0; k < 9; ++k) vir_atom[9 * (size_t)q + k] = 0.0;
        const int cell = (b[2] * gp.nb[1] + b[1]) * gp.nb[0] + b[0];
        cell_of[q] = cell;
        cv[j] = cell;
        atomicAdd(&s_cnt[cell], 1);
    }
    __syncthreads();
    // exclusive scan of the bin counts: contiguous segments per thread, then a scan of the partials
    const int seg = (ncell + PS_THREADS - 1) / PS_THREADS;
    const int c0 = tid * seg, c1 = min(c0 + seg, ncell);
    int sum = 0;
    for (int c = c0; c < c1; ++c) sum += s_cnt[c];
    s_part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < PS_THREADS; o <<= 1) {
        const int v = tid >= o ? s_part[tid - o] : 0;
        __syncthreads();
        s_part[tid] += v;
        __syncthreads();
    }
    int run = s_part[tid] - sum;
    for (int c = c0; c < c1; ++c) {
        const int v = s_cnt[c];
        cell_start[cell_off + c] = atom_off + run;
        s_cnt[c] = run;   // cursor
        run += v;
    }
    if (tid == 0) cell_start[cell_off + ncell] = atom_off + n;
    __syncthreads();
    // bin fill: candidate records in bin order (tag: internal index, caller index, type)
#pragma unroll
    for (int j = 0; j < PS_APT; ++j) {
        const int q = qv[j];
        if (q < 0) continue;
        const int slot = atomicAdd(&s_cnt[cv[j]], 1);
        const long long tag = (long long)q | ((long long)(atom_off + tid + PS_THREADS * j) << 30) |
                              ((long long)rv[j] << 60);
        cand[atom_off + slot] = make_double4(xv[j][0], xv[j][1], xv[j][2], __longlong_as_double(tag));
    }
}

// ---- preparation of larger frames in three launches ---------------------------------------
// Blocks of TP_BLOCK atoms in caller order.
//   k_prep_count: per-block type counts (types clamped; the scatter raises the error flag) and
//                 the bin of every atom, counted into cell_count with atomics. cell_count is zero
//                 on entry: k_prep_scan clears what it read, and the host clears the array after
//                 allocating it.
//   k_prep_scan (one block): clears the statistics block, scans the block type counts over blocks
//                 and the bin counts (bin starts and fill cursors), and clears the bin counts.
//   k_prep_scatter: the stable partition by type (ballot ranks within the block plus the block's
//                 base), the wrapped position and bin in internal order (wrap_bin_one again, the
//                 same bits as in k_prep_count), zeroed force accumulators, and the candidate
//                 record of every atom at the next free slot of its bin (the order within a bin
//                 is not fixed: the neighbour list sorts its hits by a key unique per candidate).
__global__ void __launch_bounds__(TP_BLOCK) k_prep_count(int n, int nlocal, const double* coord, const int* atype,
                                                         int ntypes, GeomParams gp, int* bcount, int* cell_tmp,
                                                         int* cell_count)
{
    __shared__ int h[MAXT];
    if (threadIdx.x < MAXT) h[threadIdx.x] = 0;
    __syncthreads();
    const int i = blockIdx.x * TP_BLOCK + threadIdx.x;
    if (i < n) {
        atomicAdd(&h[i < nlocal ? clamp_type(atype[i], ntypes) : ntypes], 1);   // ghosts: one class after the types
        const double x[3] = {coord[3 * (size_t)i], coord[3 * (size_t)i + 1], coord[3 * (size_t)i + 2]};
        double p[3];
        int b[3];
        wrap_bin_one(gp, x, p, b);
        const int cell = (b[2] * gp.nb[1] + b[1]) * gp.nb[0] + b[0];
        cell_tmp[i] = cell;
        atomicAdd(&cell_count[cell], 1);
    }
    __syncthreads();
    if (threadIdx.x < MAXT) bcount[blockIdx.x * MAXT + threadIdx.x] = h[threadIdx.x];
}

// Exclusive scan of v[0..m) by one block of 1024 threads (four values per thread and pass, wave scans in
// registers, the 16 wave totals in LDS): out[i] = base + sum of v[0..i); returns the total to every thread.
// part holds 16 ints of LDS. (One value per thread and a scan through LDS, 20 barriers a pass: k_prep_scan
// of 110,592 atoms 17.6 us against 10.7.)
__device__ int block_scan_1024(int m, const int* v, int vstride, int* out, int ostride, int base, int* part)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int carry = 0;
    for (int b0 = 0; b0 < m; b0 += 4096) {
        const int i = b0 + 4 * tid;
        int x[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = i + k < m ? v[(size_t)(i + k) * vstride] : 0;
            sum += x[k];
        }
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (lane == 63) part[wave] = incl;
        __syncthreads();
        int at = base + carry + incl - sum;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) at += part[w];
            carry += part[w];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i + k < m) out[(size_t)(i + k) * ostride] = at;
            at += x[k];
        }
        __syncthreads();
    }
    return carry;
}

__global__ void __launch_bounds__(1024) k_prep_scan(int nblocks, int ntypes, const int* bcount, int* boff, int* toff,
                                                    int* tcount, int ncell, int* cell_count, int* cell_start,
                                                    int* cursor, DevStats* st)
{
    __shared__ int part[16];
    const int tid = threadIdx.x;
    clear_stats(st, tid, (int)blockDim.x);
    // types: block offsets within each type (type t's atoms follow those of types < t)
    int acc = 0;
    for (int t = 0; t < ntypes; ++t) {
        const int c = block_scan_1024(nblocks, bcount + t, MAXT, boff + t, MAXT, acc, part);
        if (tid == 0) {
            toff[t] = acc;
            tcount[t] = c;
        }
        acc += c;
    }
    if (tid == 0) toff[ntypes] = acc;
    // bins: starts and fill cursors; the counts are cleared for the next frame
    const int total = block_scan_1024(ncell, cell_count, 1, cell_start, 1, 0, part);
    for (int i = tid; i < ncell; i += 1024) {
        cursor[i] = cell_start[i];
        cell_count[i] = 0;
    }
    if (tid == 0) cell_start[ncell] = total;
}

__global__ void __launch_bounds__(TP_BLOCK) k_prep_scatter(int n, int nlocal, const double* coord, const int* atype,
                                                           int ntypes, GeomParams gp, const int* boff,
                                                           const int* cell_tmp, int* perm, int* inv_perm, int* itype,
                                                           double* pos, int* cell_of, int* cursor, double4* cand,
                                                           double* f_int, DevStats* st)
{
    __shared__ int wsum[TP_BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int i = blockIdx.x * TP_BLOCK + tid;
    const int ncls = ntypes + (nlocal < n ? 1 : 0);
    int t = -1, cls = -1;
    if (i < n) {
        const int t0 = atype[i];
        if (t0 < 0 || t0 >= ntypes) atomicExch(&st->err_type, 1);
        t = clamp_type(t0, ntypes);
        cls = i < nlocal ? t : ntypes;   // ghosts: one class after the types
    }
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int q = -1;
    for (int k = 0; k < ncls; ++k) {
        const bool f = (cls == k);
        const unsigned long long m = __ballot(f);
        if (lane == 0) wsum[wid] = __popcll(m);
        __syncthreads();
        int before = 0;
        for (int w = 0; w < wid; ++w) before += wsum[w];
        if (f) q = boff[blockIdx.x * MAXT + k] + before + __popcll(m & lt);
        __syncthreads();
    }
    if (q < 0) return;
    perm[q] = i;
    inv_perm[i] = q;
    itype[q] = t;
    const double x[3] = {coord[3 * (size_t)i], coord[3 * (size_t)i + 1], coord[3 * (size_t)i + 2]};
    double p[3];
    int b[3];
    wrap_bin_one(gp, x, p, b);
    const int cell = cell_tmp[i];
    for (int c = 0; c < 3; ++c) {
        pos[3 * (size_t)q + c] = p[c];
        f_int[3 * (size_t)q + c] = 0.0;
    }
    cell_of[q] = cell;
    const int slot = atomicAdd(&cursor[cell], 1);
    const long long tag = (long long)q | ((long long)i << 30) | ((long long)t << 60);
    cand[slot] = make_double4(p[0], p[1], p[2], __longlong_as_double(tag));
}

__global__ void __launch_bounds__(PS_THREADS) k_prep_small(int n, int nlocal, const double* coord, const int* atype,
                                                            int ntypes, GeomParams gp, int ncell, int* tcount,
                                                            int* toff, int* perm, int* inv_perm, int* itype,
                                                            DevStats* st, double* pos, int* cell_of, int* cell_start,
                                                            double4* cand, double* f_int)
{
    prep_frame<false>(0, n, nlocal, 0, coord, atype, ntypes, gp, ncell, 0, nullptr, tcount, toff, perm, inv_perm,
                      itype, nullptr, st, pos, cell_of, cell_start, cand, f_int, nullptr);
}

// ---- batched frames (serving): per-frame type counts, cross-frame type bases, per-frame prep --

__global__ void __launch_bounds__(256) k_batch_count(const int* atype, int ntypes, FrameDesc* fd)
{
    __shared__ int s_c[4][MAXT];
    __shared__ int s_bad[4];
    FrameDesc& d = fd[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int cnt[MAXT];
    for (int k = 0; k < MAXT; ++k) cnt[k] = 0;
    bool bad = false;
    for (int a = tid; a < d.natoms; a += 256) {
        const int t0 = atype[d.atom_off + a];
        bad |= t0 < 0 || t0 >= ntypes;
        const int t = clamp_type(t0, ntypes);
        for (int k = 0; k < MAXT; ++k) cnt[k] += t == k;
    }
    for (int k = 0; k < MAXT; ++k) {
        int v = cnt[k];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) s_c[wid][k] = v;
    }
    if (lane == 0) s_bad[wid] = __ballot(bad) != 0;
    __syncthreads();
    if (tid < MAXT) d.type_base[tid] = s_c[0][tid] + s_c[1][tid] + s_c[2][tid] + s_c[3][tid];
    if (tid == 0) d.bad = s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3];
}

// Per-type totals and each frame's internal base per type (atoms sorted by type over the whole
// batch, frames in order within a type); zeroes the statistics block of the batch.
__global__ void k_batch_scan(int nframes, int ntypes, FrameDesc* fd, int* tcount, int* toff, DevStats* st)
{
    clear_stats(st, threadIdx.x, (int)blockDim.x);
    __syncthreads();
    if (threadIdx.x != 0) return;
    int acc = 0, bad = 0;
    for (int t = 0; t < ntypes; ++t) {
        toff[t] = acc;
        int c = 0;
        for (int f = 0; f < nframes; ++f) {
            const int v = fd[f].type_base[t];
            fd[f].type_base[t] = acc + c;
            c += v;
        }
        tcount[t] = c;
        acc += c;
    }
    toff[ntypes] = acc;
    for (int f = 0; f < nframes; ++f) bad |= fd[f].bad;
    if (bad) st->err_type = 1;
}

__global__ void __launch_bounds__(PS_THREADS) k_prep_batch(const double* coord, const int* atype, int ntypes,
                                                            const GeomParams* gps, const FrameDesc* fd, int* perm,
                                                            int* inv_perm, int* itype, int* frame_of, double* pos,
                                                            int* cell_of, int* cell_start, double4* cand, double* f_int,
                                                            double* vir_atom)
{
    const int f = blockIdx.x;
    const FrameDesc& d = fd[f];
    prep_frame<true>(f, d.natoms, d.natoms, d.atom_off, coord, atype, ntypes, gps[f], d.ncell, d.cell_off, d.type_base,
                     nullptr, nullptr, perm, inv_perm, itype, frame_of, nullptr, pos, cell_of, cell_start, cand, f_int,
                     vir_atom);
}

// ---- neighbour list: one wave per centre atom --------------------------------------------
// Candidate records are stored in bin order (by the preparation): position and a tag holding the
// internal index, the caller index and the type (30 + 30 + 4 bits), so one 32-B load gives
// everything the candidate test and the output need.
// The wave first loads the candidate ranges of the stencil's runs at once (one lane per run of bins along
// the first axis) and scans their sizes; it then sweeps the flat candidate range, several candidates per
// lane in flight.
// Candidates within r_c are compacted into LDS as 128-bit keys that compare like
// (type, r^2, caller index j, image n0, n1, n2):
//   hi = type << 59 | bits(r^2) - bits(r_c^2 2^-128)
//   lo = j << 30 | code(n) << 9 | run
// (r^2 is a non-negative double, whose bit pattern orders like its value). They are ranked; the first
// sel[t] of each type fill that type's block of slots, the rest are counted as dropped; unfilled slots
// get index -1.
// Bound: VALU issue (about 1,450 instructions per atom of 90 neighbours, 90 % busy at 110,592 atoms); at a
// few waves per SIMD the chain of loads (ranges, candidates, the output's second look at them). One run for
// the three bins of a row instead of a range per bin, found by walking on instead of a binary search, type
// counts from the keys instead of per candidate, ranks on 32-bit words and the output written from
// registers: 12,288 water atoms 78 -> 44 us, 110,592 470 -> 290, 192 (latency alone) 21 -> 18; 32,000 fcc
// atoms, 182 neighbours, 320 -> 227 with the counters off the statistics' cache line.

__device__ __forceinline__ bool key_less(unsigned long long ah, unsigned long long al,
                                         unsigned long long bh, unsigned long long bl)
{
    return ah < bh || (ah == bh && al < bl);
}

__device__ __forceinline__ void image_shift(const GeomParams& gp, int n0, int n1, int n2, double sh[3])
{
    if (gp.periodic) {
        for (int c = 0; c < 3; ++c)
            sh[c] = ((double)n0 * gp.h[c] + (double)n1 * gp.h[3 + c]) + (double)n2 * gp.h[6 + c];
    } else {
        sh[0] = sh[1] = sh[2] = 0.0;
    }
}

constexpr int NL_UNROLL = 4;
constexpr int RANK_MAX = 256;   // hits per atom up to which the neighbour list ranks instead of sorting

// Sort key of a neighbour, 128 bits: (type, r^2, caller index, image code), and its run of the stencil. r^2 < r_c^2 as the distance of
// its bit pattern from that of r_c^2 2^-128 (smaller ones all at 0), 59 bits: the high 32 bits of the key
// then hold the type and 20 bits below the exponent, enough to tell almost any two neighbours apart.
__device__ __forceinline__ unsigned long long nl_key_base(double rc2)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(rc2);
    return b > (1ull << 59) ? b - (1ull << 59) : 0;
}

constexpr int NL_RUN_BITS = 9;
static_assert(NL_STENCIL <= 1 << NL_RUN_BITS, "run index in the key");

// One candidate per lane into the hits: those within r_c are compacted behind the count (wave-uniform) of
// hits so far. Hits past the CAP stored ones are only counted, by type: lane t holds those of type t.
template <int CAP>
__device__ __forceinline__ void nl_push(bool pass, int t, double r2, int j, int code, int run, int src, unsigned long long kbase,
                                        int ntypes, int lane, int& count, int& over, unsigned long long* khi,
                                        unsigned long long* klo, int* kq)
{
    const unsigned long long m = __ballot(pass);
    const int idx = count + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    if (pass && idx < CAP) {
        const unsigned long long rb = (unsigned long long)__double_as_longlong(r2);
        khi[idx] = ((unsigned long long)t << 59) | (rb > kbase ? rb - kbase : 0ull);
        klo[idx] = ((unsigned long long)j << 30) | (unsigned long long)((code << NL_RUN_BITS) | run);
        kq[idx] = src;
    }
    count += __popcll(m);
    if (count > CAP)
        for (int q = 0; q < ntypes; ++q) {
            const int c = __popcll(__ballot(pass && idx >= CAP && t == q));
            if (lane == q) over += c;
        }
}

// Ordering of LDS traffic between the lanes of the (single-wave) workgroup.
__device__ __forceinline__ void wave_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Ranks of count <= RANK_MAX keys in LDS, EA = ceil(count / 64) of them per lane (key lane + 64 e): a
// key's position is the number of smaller keys, counted against every stored key read once from LDS (a
// broadcast of two keys per read, no exchange chain). The high 32 bits decide unless two are equal: equal
// ranks then collide in a slot check and the ranks are recounted on the full 128-bit keys, which are
// unique.
template <int EA>
__device__ __forceinline__ void rank_keys(int count, int lane, unsigned long long* khi, unsigned long long* klo,
                                          int* kq, unsigned long long (&kh)[EA], unsigned long long (&kl)[EA],
                                          int (&kx)[EA], int (&rk)[EA])
{
    unsigned k32[EA];
#pragma unroll
    for (int e = 0; e < EA; ++e) {
        const int i = lane + 64 * e;
        const bool have = i < count;
        kh[e] = have ? khi[i] : ~0ull;
        kl[e] = have ? klo[i] : ~0ull;
        kx[e] = have ? kq[i] : 0;
        k32[e] = (unsigned)(kh[e] >> 32);
        rk[e] = 0;
    }
    if (lane < ((4 - count) & 3)) khi[count + lane] = ~0ull;   // whole groups of four (RANK_MAX is one)
    wave_barrier();
    const ulonglong2* k2 = reinterpret_cast<const ulonglong2*>(khi);
#pragma unroll 2
    for (int q = 0; q < count; q += 4) {
        const ulonglong2 h0 = k2[q >> 1], h1 = k2[(q >> 1) + 1];
        const unsigned h[4] = {(unsigned)(h0.x >> 32), (unsigned)(h0.y >> 32), (unsigned)(h1.x >> 32), (unsigned)(h1.y >> 32)};
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int e = 0; e < EA; ++e) rk[e] += h[c] < k32[e] ? 1 : 0;
    }
#pragma unroll
    for (int e = 0; e < EA; ++e)
        if (lane + 64 * e < count) kq[rk[e]] = lane + 64 * e;
    wave_barrier();
    bool clash = false;
#pragma unroll
    for (int e = 0; e < EA; ++e)
        if (lane + 64 * e < count) clash |= kq[rk[e]] != lane + 64 * e;
    if (__ballot(clash) != 0) {
#pragma unroll
        for (int e = 0; e < EA; ++e) rk[e] = 0;
        for (int q = 0; q < count; ++q) {
            const unsigned long long h = khi[q], l = klo[q];
#pragma unroll
            for (int e = 0; e < EA; ++e) rk[e] += key_less(h, l, kh[e], kl[e]) ? 1 : 0;
        }
    }
}

// Bitonic sort in LDS of count keys (padded to a power of two with keys that order last): the path
// for more than RANK_MAX atoms within r_c, rare, kept out of registers so that the buffer size does
// not set the kernel's register count.
__device__ void bitonic_keys_lds(int count, int lane, unsigned long long* khi, unsigned long long* klo, int* kq)
{
    int n2 = 64;
    while (n2 < count) n2 <<= 1;
    for (int i = count + lane; i < n2; i += 64) {
        khi[i] = ~0ull;
        klo[i] = ~0ull;
        kq[i] = 0;
    }
    wave_barrier();
    for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = lane; p < (n2 >> 1); p += 64) {
                const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));   // p with a zero bit inserted at j
                const int l = i | j;
                const bool up = (i & k) == 0;
                const unsigned long long ih = khi[i], il = klo[i], lh = khi[l], ll = klo[l];
                if (key_less(lh, ll, ih, il) == up) {
                    const int ix = kq[i];
                    khi[i] = lh; klo[i] = ll; kq[i] = kq[l];
                    khi[l] = ih; klo[l] = il; kq[l] = ix;
                }
            }
            wave_barrier();
        }
}

// The selection of one atom's list from its count hits (keys in LDS; kq the candidate each key came from;
// over: this lane's count of hits of type `lane` past the CAP stored ones): the first sel[t] of each type
// block in the order of the keys written to row a of the list (fetch(kq, run, r, j) gives the candidate's
// r_ij and caller index), padding -1, the kept counts, and the neighbours dropped by sel. What belongs to
// a type is held by the lane of its number.
template <int CAP, class Fetch>
__device__ __forceinline__ void nlist_select(int a, int lane, int count, int over, const GeomParams& gp,
                                             unsigned long long* khi, unsigned long long* klo, int* kq, int* nl_j,
                                             double* nl_r, int* nnei, DevStats* st, Fetch&& fetch)
{
    // one word shared by every atom: only the few atoms that raise the maximum touch it atomically
    if (lane == 0 && count > __atomic_load_n(&st->max_cand, __ATOMIC_RELAXED)) {
        atomicMax(&st->max_cand, count);
        if (count > CAP) atomicExch(&st->err_overflow, 1);
    }
    // An overflowed frame is flagged and its list incomplete: the type blocks hold the stored hits, so that
    // each starts where its keys do and every slot the list claims is written.
    count = min(count, CAP);
    const int nt = gp.ntypes;
    const int sel = lane < nt ? gp.sel[lane] : 0, off = lane < nt ? gp.off[lane] : 0;
    int have = 0, start = 0;   // stored hits of the lane's type, and of the types before it
    wave_barrier();
    const size_t row = (size_t)a * gp.nc;
    auto counted = [&](auto&& stored) {   // stored(t): stored hits of type t (wave-uniform)
        int acc = 0;
        for (int t = 0; t < nt; ++t) {
            const int c = stored(t);
            if (lane == t) {
                have = c;
                start = acc;
            }
            acc += c;
        }
    };
    // slot of the hit at position q of the sorted hits (every lane takes part in the shuffles: one under the
    // condition would read 0 from a lane that does not meet it)
    auto place = [&](int q, int t) {
        const int st_t = __shfl(start, t), sel_t = __shfl(sel, t), off_t = __shfl(off, t), rank = q - st_t;
        return rank < sel_t ? off_t + rank : -1;
    };
    auto write = [&](int slot, const double* r, int j) {
        nl_j[row + slot] = j;
        for (int c = 0; c < 3; ++c) nl_r[3 * (row + slot) + c] = r[c];
    };
    auto ranked = [&](auto ea) {
        constexpr int EA = decltype(ea)::value;
        unsigned long long kh[EA], kl[EA];
        int kx[EA], rk[EA], slot[EA], j[EA];
        double r[EA][3];
        rank_keys<EA>(count, lane, khi, klo, kq, kh, kl, kx, rk);
        counted([&](int t) {
            int c = 0;
#pragma unroll
            for (int e = 0; e < EA; ++e) c += __popcll(__ballot((int)(kh[e] >> 59) == t));
            return c;
        });
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            const bool in = lane + 64 * e < count;
            slot[e] = place(rk[e], in ? (int)(kh[e] >> 59) : 0);
            if (!in) slot[e] = -1;
            fetch(kx[e], in ? (int)kl[e] & ((1 << NL_RUN_BITS) - 1) : 0, r[e], j[e]);   // (no hit: candidate 0)
        }
#pragma unroll
        for (int e = 0; e < EA; ++e)
            if (slot[e] >= 0) write(slot[e], r[e], j[e]);
    };
    static_assert(RANK_MAX <= 256, "rank sort dispatch covers at most four keys per lane");
    if (count <= 64) ranked(std::integral_constant<int, 1>());
    else if (count <= 128) ranked(std::integral_constant<int, 2>());
    else if (count <= 192) ranked(std::integral_constant<int, 3>());
    else if (count <= RANK_MAX) ranked(std::integral_constant<int, 4>());
    else {
        bitonic_keys_lds(count, lane, khi, klo, kq);
        counted([&](int t) {
            int c = 0;
            for (int q0 = 0; q0 < count; q0 += 64) c += __popcll(__ballot(q0 + lane < count && (int)(khi[q0 + lane] >> 59) == t));
            return c;
        });
        for (int q0 = 0; q0 < count; q0 += 64) {
            const int q = min(q0 + lane, count - 1);
            const int slot = place(q, (int)(khi[q] >> 59));
            double r[3];
            int j;
            fetch(kq[q], (int)klo[q] & ((1 << NL_RUN_BITS) - 1), r, j);
            if (slot >= 0 && q0 + lane < count) write(slot, r, j);
        }
    }
    const int kept = min(have, sel);
    const double zero[3] = {0.0, 0.0, 0.0};
    for (int t = 0; t < nt; ++t) {
        const int k = __shfl(kept, t), e = __shfl(sel, t), o = __shfl(off, t);
        for (int s2 = k + lane; s2 < e; s2 += 64) write(o + s2, zero, -1);
    }
    if (lane < nt) nnei[(size_t)a * nt + lane] = kept;
    const int dropped = have + over - kept;
    if (__ballot(dropped > 0)) {
        int drops = dropped;
        for (int o = 32; o > 0; o >>= 1) drops += __shfl_xor(drops, o);
        if (lane == 0) atomicAdd(&drop_slots(st)[a & (NL_DROP_SLOTS - 1)], (unsigned long long)drops);
    }
}

struct NlRun {
    double sh[3];   // image shift
    int off;        // candidate index of flat position q: q + off
    int code;       // image code
};
// Periodic image of bin index t on an axis of nb bins: floor division; at least K bins leave t within one
// box length of the cell, so the image is -1, 0 or 1.
__device__ __forceinline__ int image_of(int t, int nb, int K)
{
    if (nb >= K) return t < 0 ? -1 : (t >= nb ? 1 : 0);
    return t >= 0 ? t / nb : -((nb - 1 - t) / nb);
}

// BATCH: atom a belongs to frame frame_of[a]; its geometry is gps[frame] and its bins start at
// fd[frame].cell_off of the concatenated cell_start (candidate records hold batch-wide indices). Six waves
// per SIMD: two spilled registers against 83 in use and five waves, 5 to 8 % faster.
template <int CAP, bool BATCH>
__global__ void __launch_bounds__(64, 6) k_nlist(int n, const double* pos, const int* perm, const int* inv_perm,
                                              const int* cell_of, const int* cell_start0, const double4* cand,
                                              GeomParams gp0, const GeomParams* gps, const FrameDesc* fd,
                                              const int* frame_of, int* nl_j, double* nl_r, int* nnei, DevStats* st)
{
    const int fr = BATCH ? frame_of[blockIdx.x] : 0;
    const GeomParams& gp = BATCH ? gps[fr] : gp0;
    const int* cell_start = BATCH ? cell_start0 + fd[fr].cell_off : cell_start0;
    // LDS sized per launch: keys of CAP candidates, then the stencil's runs
    extern __shared__ __attribute__((aligned(16))) unsigned long long nl_lds[];
    unsigned long long* khi = nl_lds;
    unsigned long long* klo = khi + CAP;
    const int M = gp.row_runs, w1 = 2 * gp.K[1] + 1, R = gp.runs;
    NlRun* s_run = reinterpret_cast<NlRun*>(klo + CAP);   // [R]
    int* kq = reinterpret_cast<int*>(s_run + R);          // candidate index, moved with its key
    int* s_base = kq + CAP;                               // [R + 1] flat position of each run's first candidate
    const int a = blockIdx.x, lane = threadIdx.x;
    const double pi[3] = {pos[3 * (size_t)a], pos[3 * (size_t)a + 1], pos[3 * (size_t)a + 2]};
    const int ci = cell_of[a];
    const int nb0 = gp.nb[0], nb1 = gp.nb[1], nb2 = gp.nb[2];
    // (bin coordinates: with half a unit added the products stay clear of the integers, below 2^24 bins)
    const int c12 = (int)((ci + 0.5) * gp.rnb[0]), b0 = ci - c12 * nb0;
    const int b2 = (int)((c12 + 0.5) * gp.rnb[1]), b1 = c12 - b2 * nb1;
    const int self_code = (64 << 14) | (64 << 7) | 64;
    const unsigned long long kbase = nl_key_base(gp.rc2);

    // the non-empty runs, one per lane: range, image, and their flat positions scanned across the wave
    int total = 0, nr = 0;   // wave-uniform
    for (int s0 = 0; s0 < R; s0 += 64) {
        const int k = s0 + lane, rw = (k * gp.m_row) >> 16, o2 = (rw * gp.m_w1) >> 16;
        const int tg1 = b1 + rw - o2 * w1 - gp.K[1], tg2 = b2 + o2 - gp.K[2];
        int cnt = 0, start = 0, n0 = 0, n1 = 0, n2 = 0;
        bool in = k < R;
        int x0 = b0 - gp.K[0], x1 = b0 + gp.K[0];
        if (gp.periodic) {
            n0 = image_of(x0, nb0, gp.K[0]) + k - rw * M;
            n1 = image_of(tg1, nb1, gp.K[1]);
            n2 = image_of(tg2, nb2, gp.K[2]);
        } else {
            in = in && tg1 >= 0 && tg1 < nb1 && tg2 >= 0 && tg2 < nb2;
        }
        x0 = max(x0 - n0 * nb0, 0);
        x1 = min(x1 - n0 * nb0, nb0 - 1);
        if (in && x0 <= x1) {
            const int cell = ((tg2 - n2 * nb2) * nb1 + tg1 - n1 * nb1) * nb0;
            start = cell_start[cell + x0];
            cnt = cell_start[cell + x1 + 1] - start;
        }
        int incl = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        const unsigned long long m = __ballot(cnt > 0);
        if (cnt > 0) {
            const int at = nr + __popcll(m & ((1ull << lane) - 1)), base = total + incl - cnt;
            NlRun r;
            image_shift(gp, n0, n1, n2, r.sh);
            r.off = start - base;
            r.code = ((n0 + 64) << 14) | ((n1 + 64) << 7) | (n2 + 64);
            s_run[at] = r;
            s_base[at] = base;
        }
        nr += __popcll(m);
        total += __shfl(incl, 63);
    }
    if (lane == 0) s_base[nr] = total;
    wave_barrier();

    // One flat sweep over the candidates of all runs. A lane's position grows by 64 a step, about the
    // length of a run (three bins of r_c): its run is found by walking on from the last one.
    int count = 0, over = 0;   // count: wave-uniform
    int b = 0;                 // this lane's current run
    for (int q0 = 0; q0 < total; q0 += 64 * NL_UNROLL) {
        double4 c4[NL_UNROLL];
        int run[NL_UNROLL], cq[NL_UNROLL];
#pragma unroll
        for (int u = 0; u < NL_UNROLL; ++u) {
            const int q = min(q0 + 64 * u + lane, total - 1);
            while (s_base[b + 1] <= q) ++b;
            run[u] = b;
            cq[u] = q + s_run[b].off;
            c4[u] = cand[cq[u]];
        }
#pragma unroll
        for (int u = 0; u < NL_UNROLL; ++u) {
            if (q0 + 64 * u >= total) break;   // (wave-uniform)
            const NlRun r = s_run[run[u]];
            const unsigned long long tag = (unsigned long long)__double_as_longlong(c4[u].w);
            const double d0 = (c4[u].x + r.sh[0]) - pi[0];
            const double d1 = (c4[u].y + r.sh[1]) - pi[1];
            const double d2 = (c4[u].z + r.sh[2]) - pi[2];
            const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
            const bool self = (int)(tag & 0x3fffffffull) == a && r.code == self_code;
            const bool pass = q0 + 64 * u + lane < total && !self && r2 < gp.rc2;
            nl_push<CAP>(pass, (int)(tag >> 60), r2, (int)((tag >> 30) & 0x3fffffffull), r.code, run[u], cq[u], kbase,
                         gp.ntypes, lane, count, over, khi, klo, kq);
        }
    }
    nlist_select<CAP>(a, lane, count, over, gp, khi, klo, kq, nl_j, nl_r, nnei, st,
                      [&](int q, int rn, double* r, int& j) {
                          const double4 c4 = cand[q];
                          j = (int)((__double_as_longlong(c4.w) >> 30) & 0x3fffffffll);   // caller index
                          r[0] = (c4.x + s_run[rn].sh[0]) - pi[0];
                          r[1] = (c4.y + s_run[rn].sh[1]) - pi[1];
                          r[2] = (c4.z + s_run[rn].sh[2]) - pi[2];
                      });
}

// External neighbour candidates (an MD code's own list, with or without a skin; Sec. III.B.2):
// owned atom a (internal index, caller index i = perm[a]) takes the candidates
// ext[ext_start[i] .. ext_start[i + 1]), caller indices of owned or ghost atoms in any order,
// without duplicates. Positions are used as given (open geometry: a ghost carries the image
// position its owner's domain sent), so r_ij = r_j - r_i; those within r_c are ordered by (type,
// distance, index) and selected exactly as k_nlist does. Indices outside [0, ntot) and the atom
// itself are skipped (the host entry point rejects such lists before the launch).
template <int CAP>
__global__ void __launch_bounds__(64) k_nlist_ext(int ntot, const double* pos, const int* perm, const int* inv_perm,
                                                  const int* itype, const int* ext_start, const int* ext,
                                                  GeomParams gp, int* nl_j, double* nl_r, int* nnei, DevStats* st)
{
    extern __shared__ __attribute__((aligned(16))) unsigned long long nl_lds[];
    unsigned long long* khi = nl_lds;
    unsigned long long* klo = khi + CAP;
    int* kq = reinterpret_cast<int*>(klo + CAP);   // internal index of the candidate, moved with its key
    const int a = blockIdx.x, lane = threadIdx.x;
    const int ci = perm[a];
    const double pi[3] = {pos[3 * (size_t)a], pos[3 * (size_t)a + 1], pos[3 * (size_t)a + 2]};
    const int b0 = ext_start[ci], b1 = ext_start[ci + 1];
    const unsigned long long kbase = nl_key_base(gp.rc2);
    int count = 0, over = 0;   // count: wave-uniform
    for (int q0 = b0; q0 < b1; q0 += 64) {
        const int q = q0 + lane;
        bool pass = false;
        double r2 = 0.0;
        int tj = 0, j = -1, jq = 0;
        if (q < b1) {
            j = ext[q];
            if (j >= 0 && j < ntot && j != ci) {
                jq = inv_perm[j];
                tj = itype[jq];
                const double d0 = pos[3 * (size_t)jq] - pi[0];
                const double d1 = pos[3 * (size_t)jq + 1] - pi[1];
                const double d2 = pos[3 * (size_t)jq + 2] - pi[2];
                r2 = d0 * d0 + d1 * d1 + d2 * d2;
                pass = r2 < gp.rc2;
            }
        }
        // (no image, no run: 0)
        nl_push<CAP>(pass, tj, r2, j, 0, 0, jq, kbase, gp.ntypes, lane, count, over, khi, klo, kq);
    }
    nlist_select<CAP>(a, lane, count, over, gp, khi, klo, kq, nl_j, nl_r, nnei, st,
                      [&](int q, int, double* r, int& jj) {
                          jj = perm[q];
                          for (int c = 0; c < 3; ++c) r[c] = pos[3 * (size_t)q + c] - pi[c];
                      });
}

// ---- reductions and output ----------------------------------------------------------------

// Compensated (Neumaier) running sum: the error of a long sum stays about one rounding of the
// result instead of growing with the number of terms (this file is built without FMA contraction,
// which the compensation relies on).
struct NeumaierSum {
    double s = 0.0, c = 0.0;
    __device__ void add(double x) {
        const double t = s + x;
        c += fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s;
        s = t;
    }
    __device__ double value() const { return s + c; }
};

// Single frame: E and the virial from the embedding backward's block partials [E, virial[9]], in a fixed
// order with compensated sums: thread t < 1020 sums component t % 10 of the partials t / 10, t / 10 + 102,
// ..., then 170 threads six of those sums each and ten threads their component's 17. Also the frame's
// count of neighbours dropped by sel from its per-atom counters (one wave, lane = its lane index). A chain
// of dependent additions per thread, so many threads: 250 took 24 us for the 110,592-atom box, 1020 take 7.
__device__ void sum_drop_slots(DevStats* st, int lane)
{
    unsigned long long v = 0;
    for (int i = lane; i < NL_DROP_SLOTS; i += 64) v += drop_slots(st)[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) st->nbr_dropped = v;
}

constexpr int FIN_T = 1024, FIN_R = 102, FIN_G = 17;   // threads; partial sums per component; groups of them
__global__ void __launch_bounds__(FIN_T) k_finalize(int nb, const double* part, double* energy, double* virial,
                                                    DevStats* st)
{
    __shared__ double red[10 * FIN_R], grp[10 * FIN_G];
    const int t = threadIdx.x;
    if (t < 10 * FIN_R) {
        NeumaierSum v;
        constexpr int U = 4;
        for (int i = t; i < 10 * nb; i += U * 10 * FIN_R) {
            double x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = i + u * 10 * FIN_R < 10 * nb ? part[i + u * 10 * FIN_R] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) v.add(x[u]);
        }
        red[t] = v.value();
    }
    __syncthreads();
    if (t < 10 * FIN_G) {
        NeumaierSum v;
        for (int k = 0; k < FIN_R / FIN_G; ++k) v.add(red[t + 10 * FIN_G * k]);
        grp[t] = v.value();
    }
    if (t >= FIN_T - 64) sum_drop_slots(st, t - (FIN_T - 64));   // the last wave, beside the sums
    __syncthreads();
    if (t < 10) {
        NeumaierSum x;
        for (int k = 0; k < FIN_G; ++k) x.add(grp[t + 10 * k]);
        if (t == 0) *energy = x.value();
        else virial[t - 1] = x.value();
    }
}

// Batched frames: per frame (one block each) E = sum E_i and the virial = sum over the frame's
// atoms of their per-atom virial, both in a fixed order, and the frame's forces (and E_i) in its
// caller order. Output of frame f at out + out_off: E, virial[9], F[3n], E_i[n].
__global__ void __launch_bounds__(256) k_finalize_batch(const FrameDesc* fd, const int* inv_perm, const double* ei,
                                                        const double* vir_atom, const double* f_int, double* out,
                                                        DevStats* st)
{
    __shared__ double red[10][256];
    const FrameDesc& d = fd[blockIdx.x];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < 64) sum_drop_slots(st, tid);   // one count for the batch
    double* o = out + d.out_off;
    double acc[10];
    for (int k = 0; k < 10; ++k) acc[k] = 0.0;
    for (int a = tid; a < d.natoms; a += 256) {
        const int q = inv_perm[d.atom_off + a];
        acc[0] += ei[q];
        for (int k = 0; k < 9; ++k) acc[1 + k] += vir_atom[9 * (size_t)q + k];
        for (int c = 0; c < 3; ++c) o[10 + 3 * (size_t)a + c] = f_int[3 * ((size_t)d.atom_off + a) + c];
        if (d.want_ei) o[10 + 3 * (size_t)d.natoms + a] = ei[q];
    }
    for (int k = 0; k < 10; ++k) red[k][tid] = acc[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w)
            for (int k = 0; k < 10; ++k) red[k][tid] += red[k][tid + w];
        __syncthreads();
    }
    if (tid < 10) o[tid] = red[tid][0];
}

// Debug: neighbour list (caller numbering already), rows in caller order.
__global__ void k_debug_nlist(int n, int ncentre, int nc, const int* perm, const int* nl_j, int* out)
{
    int a = blockIdx.x;
    int i = perm[a];
    // atoms past the centres (ghost atoms) have no list
    for (int s = threadIdx.x; s < nc; s += blockDim.x) out[(size_t)i * nc + s] = a < ncentre ? nl_j[(size_t)a * nc + s] : -1;
}

// ---- launchers --------------------------------------------------------------------------

void launch_prep_large(int n, const double* coord, const int* atype, int ntypes, const GeomParams& gp, int* tcount,
                       int* toff, int* bcount, int* boff, int* perm, int* inv_perm, int* itype, DevStats* st,
                       double* pos, int* cell_of, int* cell_count, int* cell_start, int* cursor, int* cell_tmp,
                       double4* cand, double* f_int, hipStream_t s, int nlocal)
{
    if (nlocal < 0) nlocal = n;
    const int nb = (n + TP_BLOCK - 1) / TP_BLOCK;
    const int ncell = gp.nb[0] * gp.nb[1] * gp.nb[2];
    const int ncls = ntypes + (nlocal < n ? 1 : 0);
    hipLaunchKernelGGL(k_prep_count, dim3(nb), dim3(TP_BLOCK), 0, s, n, nlocal, coord, atype, ntypes, gp, bcount,
                       cell_tmp, cell_count);
    hipLaunchKernelGGL(k_prep_scan, dim3(1), dim3(1024), 0, s, nb, ncls, bcount, boff, toff, tcount, ncell,
                       cell_count, cell_start, cursor, st);
    hipLaunchKernelGGL(k_prep_scatter, dim3(nb), dim3(TP_BLOCK), 0, s, n, nlocal, coord, atype, ntypes, gp, boff,
                       cell_tmp, perm, inv_perm, itype, pos, cell_of, cursor, cand, f_int, st);
}

bool launch_prep_small(int n, const double* coord, const int* atype, int ntypes, const GeomParams& gp, int* tcount,
                       int* toff, int* perm, int* inv_perm, int* itype, DevStats* st, double* pos, int* cell_of,
                       int* cell_start, double4* cand, double* f_int, hipStream_t s, int nlocal)
{
    if (nlocal < 0) nlocal = n;
    const int ncell = gp.nb[0] * gp.nb[1] * gp.nb[2];
    if (n > PS_MAX_ATOMS || ncell > PS_MAX_CELLS) return false;
    hipLaunchKernelGGL(k_prep_small, dim3(1), dim3(PS_THREADS), 0, s, n, nlocal, coord, atype, ntypes, gp, ncell,
                       tcount, toff, perm, inv_perm, itype, st, pos, cell_of, cell_start, cand, f_int);
    return true;
}

void launch_batch_prep(int nframes, int ntypes, const double* coord, const int* atype, const GeomParams* gps,
                       FrameDesc* fd, int* tcount, int* toff, int* perm, int* inv_perm, int* itype, int* frame_of,
                       DevStats* st, double* pos, int* cell_of, int* cell_start, double4* cand, double* f_int,
                       double* vir_atom, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_count, dim3(nframes), dim3(256), 0, s, atype, ntypes, fd);
    hipLaunchKernelGGL(k_batch_scan, dim3(1), dim3(64), 0, s, nframes, ntypes, fd, tcount, toff, st);
    hipLaunchKernelGGL(k_prep_batch, dim3(nframes), dim3(PS_THREADS), 0, s, coord, atype, ntypes, gps, fd, perm,
                       inv_perm, itype, frame_of, pos, cell_of, cell_start, cand, f_int, vir_atom);
}

void launch_finalize(int nb, const double* part, double* energy, double* virial, DevStats* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(FIN_T), 0, s, nb, part, energy, virial, st);
}

void launch_finalize_batch(int nframes, const FrameDesc* fd, const int* inv_perm, const double* ei,
                           const double* vir_atom, const double* f_int, double* out, DevStats* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize_batch, dim3(nframes), dim3(256), 0, s, fd, inv_perm, ei, vir_atom, f_int, out, st);
}

int prep_small_max_atoms() { return PS_MAX_ATOMS; }
int prep_small_max_cells() { return PS_MAX_CELLS; }

void launch_bbox(int n, const double* coord, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_bbox, dim3(1), dim3(1024), 0, s, n, coord, out);
}

void launch_nlist(int n, const double* pos, const int* perm, const int* inv_perm, const int* cell_of,
                  const int* cell_start, const double4* cand, const GeomParams& gp, int* nl_j, double* nl_r,
                  int* nnei, DevStats* st, hipStream_t s, const GeomParams* gps, const FrameDesc* fd,
                  const int* frame_of, int max_runs, int max_cap)
{
    // candidate buffer sized from the expected count within r_c (the synchronous entry point reruns
    // a frame that overflowed with the largest buffer); LDS = 20 B per candidate slot + 36 B per
    // run, so small stencils leave room for more resident waves. A batch passes the most runs and
    // the largest buffer of its frames.
    const bool batch = gps != nullptr;
    const int R = batch ? max_runs : gp.runs;
    const int want = batch ? max_cap : gp.cap;
    const int cap = want <= 256 ? 256 : (want <= 512 ? 512 : NL_CAP);
    const size_t lds = (size_t)cap * 20 + (size_t)R * (sizeof(NlRun) + 4) + 4;
#define DPK_NL(C, B)                                                                                              \
    hipLaunchKernelGGL((k_nlist<C, B>), dim3(n), dim3(64), lds, s, n, pos, perm, inv_perm, cell_of, cell_start,   \
                       cand, gp, gps, fd, frame_of, nl_j, nl_r, nnei, st)
    if (batch) {
        if (cap == 256) DPK_NL(256, true);
        else if (cap == 512) DPK_NL(512, true);
        else DPK_NL(NL_CAP, true);
    } else {
        if (cap == 256) DPK_NL(256, false);
        else if (cap == 512) DPK_NL(512, false);
        else DPK_NL(NL_CAP, false);
    }
#undef DPK_NL
}

// Model deviation of the forces (Sec. II.C): over the nm models of an ensemble (ensemble averages
// with weight 1/nm), eps_i = sqrt(< |F_i - <F_i>|^2 >); with nu >= 0 the relative form
// eps_i / (|<F_i>| + nu). F holds model k's forces (caller order) at F + k * stride doubles.
__global__ void k_force_devi(int n, int nm, const double* F, int64_t stride, double nu, double* eps)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0;
    for (int k = 0; k < nm; ++k) {
        const double* f = F + k * stride + 3 * (size_t)i;
        m0 += f[0];
        m1 += f[1];
        m2 += f[2];
    }
    const double inv = 1.0 / nm;
    m0 *= inv;
    m1 *= inv;
    m2 *= inv;
    double v = 0.0;
    for (int k = 0; k < nm; ++k) {
        const double* f = F + k * stride + 3 * (size_t)i;
        const double d0 = f[0] - m0, d1 = f[1] - m1, d2 = f[2] - m2;
        v += d0 * d0 + d1 * d1 + d2 * d2;
    }
    double e = sqrt(v * inv);
    if (nu >= 0.0) e /= sqrt(m0 * m0 + m1 * m1 + m2 * m2) + nu;
    eps[i] = e;
}

void launch_force_devi(int n, int nm, const double* F, int64_t stride, double nu, double* eps, hipStream_t s)
{
    hipLaunchKernelGGL(k_force_devi, dim3((n + 255) / 256), dim3(256), 0, s, n, nm, F, stride, nu, eps);
}

void launch_nlist_ext(int nlocal, int ntot, const double* pos, const int* perm, const int* inv_perm, const int* itype,
                      const int* ext_start, const int* ext, const GeomParams& gp, int* nl_j, double* nl_r, int* nnei,
                      DevStats* st, hipStream_t s)
{
    const size_t lds = (size_t)NL_CAP * 20;
    hipLaunchKernelGGL((k_nlist_ext<NL_CAP>), dim3(nlocal), dim3(64), lds, s, ntot, pos, perm, inv_perm, itype,
                       ext_start, ext, gp, nl_j, nl_r, nnei, st);
}

void launch_debug_nlist(int n, int ncentre, int nc, const int* perm, const int* nl_j, int* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_debug_nlist, dim3(n), dim3(64), 0, s, n, ncentre, nc, perm, nl_j, out);
}

}  // namespace dpk
