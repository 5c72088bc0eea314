// Host runtime of the MHD library: handle lifetime, device buffers, argument
// checking and the enqueueing of the kernels behind the C ABI of mhd.h.
//
// Buffers.  Each handle owns two device allocations of 8 fields each.  Every
// operator reads the current copy of its inputs and writes the other copy
// of the fields it changes (never in place: neighbour pencils of one lane are
// another lane's output), then the per-field "current" index flips.  Handles
// of small FP32 grids have a third copy of the faces (mid_aside).
//
// Time step on the device.  Kernels read dt and the relaxation speed from a
// small device block; the host path writes it with a one-thread kernel
// (never hipMemsetAsync, so a HIP graph can capture a step), the device path
// writes it from the CFL reduction.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>

#include "../../include/mhd.h"
#include "mhd_kernels.h"
#include "runtime_common.h"

using namespace mhd;

static thread_local std::string g_last_error = "no error";

int mhd_fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}
#define fail mhd_fail

struct mhd_ctx {
    int n[3];
    size_t N;
    double gamma;
    int prec;
    size_t esize;
    hipStream_t stream;
    int device;
    void* buf[2];
    bool own_buf;           // buf[] allocated here (false: the caller's, never freed here)
    int cur[8];
    // a third place for the faces, which the one-launch middle of small grids
    // writes (mid_aside; null: no such grid), and whether they are there now
    // instead of in buf[cur]
    void* aside;
    bool in_aside;
    double* scal;           // device SCAL_COUNT doubles
    int* flag;              // device FLAG_COUNT ints
    double* partial;        // reduction partials (max of cfl and diag needs)
    int* partial_bad;
    int nblk_cfl, nblk_diag;
    double* pinned;         // host pinned scratch (16 doubles), also written by kernels
    bool have_c;
    double c_host;
    bool scal_known;        // host knows what dt / c the device block holds
    // fused CFL: the last fluid operator of a step leaves the FP64 maximum
    // signal speed of the new state in cfl_acc; acc_valid while the state
    // is still the one it describes.  acc_capture: the graph capture that
    // recorded that launch (0: it was enqueued to run); captured: some call
    // that changes the state was ever recorded instead of run
    unsigned long long* cfl_acc;
    bool acc_valid;
    unsigned long long acc_capture;
    bool captured;
    // reverse-half pairs M_d F_d: one fused launch each (true) or the two
    // operators in turn; same result bit for bit
    int rev_mode;           // 0 built-in choice, 1 fused, 2 the two operators
    // the middle of a step, M_z M_z F_z: one launch (1), or M_z and the fused
    // reverse pair (2); 0 the built-in choice
    int mid_mode;
    int limiter;            // slope limiter of the operators (MHD_LIMITER_*)
    int freeze;             // freezing speed of the fluid operator (MHD_FREEZE_*)
    double scal_dt, scal_c;
    bool failed;
    LaunchTuning tune;
};

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

#define HIP_TRY MHD_HIP_TRY

static int check_handle(const mhd_ctx* h)
{
    if (!h) return fail(MHD_EINVAL, "null handle");
    if (h->failed) return fail(MHD_ESTATE, "handle failed earlier (HIP error); destroy it");
    return MHD_OK;
}

template <typename T>
static T* field_ptr(mhd_ctx* h, int f, int which)
{
    return reinterpret_cast<T*>(h->buf[which]) + (size_t)f * h->N;
}

template <typename T>
static T* aside_ptr(mhd_ctx* h, int f)
{
    return reinterpret_cast<T*>(h->aside) + (size_t)(f - 5) * h->N;
}

template <typename T>
static T* current_ptr(mhd_ctx* h, int f)
{
    return f >= 5 && h->in_aside ? aside_ptr<T>(h, f) : field_ptr<T>(h, f, h->cur[f]);
}

template <typename T>
static void current_fields(mhd_ctx* h, const T* f[8])
{
    for (int q = 0; q < 8; ++q) f[q] = current_ptr<T>(h, q);
}

// Built-in march chunk of a pencil of nd cells: the divisor (>= 8) with the
// least estimated time.  A lane walks chunk + warm positions (rounded up to
// the unrolled group); the launch gives each of the 256 CUs at most m
// workgroups (one wave per SIMD each), `resident` of them at a time, in
// ceil(m / resident) rounds.  A position costs about m issue slots per SIMD
// plus half a slot of latency per round (fluid march, cache-resident: 0.63,
// 1.1, 2.1 us per position at m = 1, 2, 4).  So a chunk that leaves the last
// round nearly empty, or one whose warm-up outweighs the lanes it adds,
// loses.  Against the earlier rule (the longest chunk with lanes for every
// wave slot), us along y: 160^3 fluid 42.5 from 52.2, magnetic 26.5 from
// 29.7, pair 65 from 102, middle 98 from 119; 192^3 magnetic 41.5 from 48,
// pair 124 from 143, middle 163 from 224; 256^3 fluid 198 from 218 (z 173
// from 206), magnetic 131 from 136; 512^3 fluid 1435 from 1537.
// even: rather than one workgroup per CU two of half as many positions where
// the estimate is the same, for the single operators (128^3 magnetic 16.0 us
// at 16 cells, 17.5 at 32; 128x100x128 z 14.5 / 17.0; 160x68x144 y, 17 and 34
// cells: fluid 24.5 / 28.5); other ties keep the longer (160x88x148: magnetic
// 17.1 us at 22 cells, 18.0 at 11), and the pairs' differ within 7% either way.
static int march_chunk(int nd, long npencil, int warm, int unroll, int resident, bool even)
{
    int best = nd;
    long best_m = 0;
    double least = 0.0;
    for (int ch = nd; ch >= 8; --ch) {
        if (nd % ch) continue;
        const long wgs = (npencil * (nd / ch) + 255) / 256;
        const long m = (wgs + 255) / 256, rounds = (m + resident - 1) / resident;
        const int pos = (ch + warm + unroll - 1) / unroll * unroll;
        const double cost = pos * ((double)m + 0.5 * (double)rounds);
        if (ch == nd || cost < least || (even && cost == least && best_m == 1)) { best = ch; best_m = m; least = cost; }
    }
    return best;
}

static void default_tuning(mhd_ctx* h)
{
    h->tune.chunk[0] = h->tune.pair_chunk[0] = h->tune.triple_chunk[0] = 0;
    h->tune.wide = 0;
    h->tune.row_group = 0;
    for (int d = 0; d < 3; ++d) h->tune.set_chunk[d] = h->tune.set_pair[d] = h->tune.set_triple[d] = false;
    // warm-up positions, unrolled group and waves per SIMD of the marches
    // (the fluid march's for both single operators)
    const bool f32 = h->prec == MHD_F32;
    for (int d = 1; d < 3; ++d) {
        const long npencil = (long)h->n[0] * h->n[3 - d];
        h->tune.chunk[d] = march_chunk(h->n[d], npencil, 6, f32 ? 4 : 2, f32 ? 3 : 2, true);
        h->tune.pair_chunk[d] = march_chunk(h->n[d], npencil, 13, f32 ? 4 : 2, f32 ? 2 : 1, false);
        h->tune.triple_chunk[d] = march_chunk(h->n[d], npencil, 19, f32 ? 6 : 2, 1, false);
    }
}

// built-in choice of fused reverse pairs: FP32 with van Leer's or minmod
// (measured faster at 256^3); not with MC or superbee, whose fused march
// kernels spill registers (2-3% and 34% slower than the two operators), nor
// in FP64 (the fused FP64 march runs 1 wave per SIMD)
static bool default_rev_fused(int prec, int limiter)
{
    return prec == MHD_F32 && (limiter == MHD_LIMITER_VANLEER || limiter == MHD_LIMITER_MINMOD);
}

static int sync_stream(mhd_ctx* h)
{
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return MHD_OK;
}

// ---------------------------------------------------------------------------
// lifetime
// ---------------------------------------------------------------------------

// a caller's state buffer: device memory of this device, 256-byte aligned,
// at least `bytes` long inside its allocation
static int check_user_buffer(const void* p, size_t bytes, int device, const char* name)
{
    if (reinterpret_cast<uintptr_t>(p) % 256)
        return fail(MHD_EINVAL, "%s: a state buffer must be 256-byte aligned", name);
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return fail(MHD_EINVAL, "%s: not memory known to HIP", name);
    }
    if (a.type != hipMemoryTypeDevice || a.isManaged)
        return fail(MHD_EINVAL, "%s: not device memory", name);
    if (a.device != device)
        return fail(MHD_EINVAL, "%s: memory of device %d, handle on device %d", name, a.device, device);
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(MHD_EINVAL, "%s: allocation range unknown", name);
    }
    if (static_cast<const char*>(p) + bytes > static_cast<const char*>(base) + size)
        return fail(MHD_EINVAL, "%s: allocation shorter than 8*nx*ny*nz elements", name);
    return MHD_OK;
}

extern "C" mhd_ctx* mhd_create_ex(int nx, int ny, int nz, double gamma, int prec, void* hip_stream,
                                   void* dev_buf_a, void* dev_buf_b)
{
    const int n[3] = { nx, ny, nz };
    for (int d = 0; d < 3; ++d)
        if (n[d] < 8 || n[d] % 4) {
            fail(MHD_EINVAL, "grid dimension %d = %d: must be >= 8 and a multiple of 4", d, n[d]);
            return nullptr;
        }
    if (nx > 1024 || ny > 4096 || nz > 4096 || (long long)nx * ny * nz >= (1LL << 31)) {
        fail(MHD_EINVAL, "grid above the limit (nx <= 1024, ny, nz <= 4096, < 2^31 cells)");
        return nullptr;
    }
    if (!(gamma > 1.0) || !isfinite(gamma)) {
        fail(MHD_EINVAL, "gamma must be > 1 (got %g)", gamma);
        return nullptr;
    }
    if (prec != MHD_F32 && prec != MHD_F64) {
        fail(MHD_EINVAL, "precision must be MHD_F32 or MHD_F64 (got %d)", prec);
        return nullptr;
    }
    if ((dev_buf_a == nullptr) != (dev_buf_b == nullptr)) {
        fail(MHD_EINVAL, "give both state buffers or neither");
        return nullptr;
    }
    mhd_ctx* h = new mhd_ctx();
    memset(h, 0, sizeof *h);
    h->n[0] = nx; h->n[1] = ny; h->n[2] = nz;
    h->N = (size_t)nx * ny * nz;
    h->gamma = gamma;
    h->prec = prec;
    h->esize = prec == MHD_F64 ? sizeof(double) : sizeof(float);
    h->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&h->device) != hipSuccess) {
        fail(MHD_EDEVICE, "no HIP device");
        delete h;
        return nullptr;
    }
    const size_t bytes = 8 * h->N * h->esize;
    h->nblk_cfl = cfl_blocks(h->N);
    h->nblk_diag = diag_blocks(h->N);
    const int npart = std::max(h->nblk_cfl, 10 * h->nblk_diag);
    if (dev_buf_a) {
        const char* a = static_cast<const char*>(dev_buf_a);
        const char* b = static_cast<const char*>(dev_buf_b);
        if (check_user_buffer(dev_buf_a, bytes, h->device, "dev_buf_a") ||
            check_user_buffer(dev_buf_b, bytes, h->device, "dev_buf_b")) {
            delete h;
            return nullptr;
        }
        if (a < b + bytes && b < a + bytes) {
            fail(MHD_EINVAL, "the two state buffers overlap");
            delete h;
            return nullptr;
        }
        h->buf[0] = dev_buf_a;
        h->buf[1] = dev_buf_b;
        h->own_buf = false;
    } else {
        h->own_buf = true;
        if (hipMalloc(&h->buf[0], bytes) != hipSuccess || hipMalloc(&h->buf[1], bytes) != hipSuccess) {
            (void)hipGetLastError();
            fail(MHD_ENOMEM, "device allocation of 2 x %zu bytes failed", bytes);
            mhd_destroy(h);
            return nullptr;
        }
    }
    bool ok = hipMalloc(&h->scal, SCAL_COUNT * sizeof(double)) == hipSuccess &&
              hipMalloc(&h->flag, FLAG_COUNT * sizeof(int)) == hipSuccess &&
              hipMalloc(&h->partial, npart * sizeof(double)) == hipSuccess &&
              hipMalloc(&h->partial_bad, h->nblk_cfl * sizeof(int)) == hipSuccess &&
              hipMalloc(&h->cfl_acc, (CFL_ACC_SLOTS + 1) * sizeof(unsigned long long)) == hipSuccess &&
              hipHostMalloc(&h->pinned, 16 * sizeof(double), hipHostMallocDefault) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        fail(MHD_ENOMEM, "device allocation of the handle's scratch failed");
        mhd_destroy(h);
        return nullptr;
    }
    ok = hipMemsetAsync(h->buf[0], 0, bytes, h->stream) == hipSuccess &&
         hipMemsetAsync(h->buf[1], 0, bytes, h->stream) == hipSuccess &&
         hipMemsetAsync(h->scal, 0, SCAL_COUNT * sizeof(double), h->stream) == hipSuccess &&
         hipMemsetAsync(h->flag, 0, FLAG_COUNT * sizeof(int), h->stream) == hipSuccess &&
         hipMemsetAsync(h->cfl_acc, 0, (CFL_ACC_SLOTS + 1) * sizeof(unsigned long long), h->stream) == hipSuccess &&
         hipStreamSynchronize(h->stream) == hipSuccess;
    if (!ok) {
        fail(MHD_EDEVICE, "device initialisation failed");
        mhd_destroy(h);
        return nullptr;
    }
    default_tuning(h);
    h->rev_mode = 0;
    h->acc_valid = false;
    // (12 bytes a cell below 128^3 cells; without it the middle is two launches)
    if (prec == MHD_F32 && h->N < MID_CELLS && sweep_uses_tiles<float>(h->n, 3, 2, h->tune) &&
        hipMalloc(&h->aside, 3 * h->N * h->esize) != hipSuccess) {
        (void)hipGetLastError();
        h->aside = nullptr;
    }
    return h;
}

extern "C" mhd_ctx* mhd_create(int nx, int ny, int nz, double gamma)
{
    return mhd_create_ex(nx, ny, nz, gamma, MHD_F32, nullptr, nullptr, nullptr);
}

extern "C" void mhd_destroy(mhd_ctx* h)
{
    if (!h) return;
    (void)hipStreamSynchronize(h->stream);
    if (h->own_buf) {
        if (h->buf[0]) (void)hipFree(h->buf[0]);
        if (h->buf[1]) (void)hipFree(h->buf[1]);
    }
    if (h->aside) (void)hipFree(h->aside);
    if (h->scal) (void)hipFree(h->scal);
    if (h->flag) (void)hipFree(h->flag);
    if (h->partial) (void)hipFree(h->partial);
    if (h->partial_bad) (void)hipFree(h->partial_bad);
    if (h->cfl_acc) (void)hipFree(h->cfl_acc);
    if (h->pinned) (void)hipHostFree(h->pinned);
    delete h;
}

extern "C" int mhd_info(const mhd_ctx* h, int dims[3], int* prec)
{
    if (!h) return fail(MHD_EINVAL, "null handle");
    if (dims) { dims[0] = h->n[0]; dims[1] = h->n[1]; dims[2] = h->n[2]; }
    if (prec) *prec = h->prec;
    return MHD_OK;
}

// ---------------------------------------------------------------------------
// state transfer
// ---------------------------------------------------------------------------

// a call that changes the state begins: what cfl_acc holds is void
static void state_changes(mhd_ctx* h)
{
    h->acc_valid = false;
    if (mhd_capture_id(h->stream)) h->captured = true;
}

// the last launch enqueued leaves the maximum of the new state in cfl_acc
static void maximum_follows(mhd_ctx* h)
{
    h->acc_valid = true;
    h->acc_capture = mhd_capture_id(h->stream);
}

// cfl_acc will hold the maximum of the state that the next launch finds.
// Within one capture it is what the launch recorded before leaves; a capture
// takes nothing from before it, as each replay finds another state; and once
// anything has been captured the host does not know what was replayed since.
static bool maximum_holds(const mhd_ctx* h)
{
    if (!h->acc_valid) return false;
    const unsigned long long id = mhd_capture_id(h->stream);
    return id ? id == h->acc_capture : !h->captured;
}

static int reset_after_set(mhd_ctx* h)
{
    state_changes(h);
    for (int q = 0; q < 8; ++q) h->cur[q] = 0;
    h->in_aside = false;
    h->have_c = false;
    h->c_host = 0.0;
    h->scal_known = false;
    HIP_TRY(h, launch_reset_scalars(h->scal, h->flag, h->stream));
    return MHD_OK;
}

extern "C" int mhd_set_state(mhd_ctx* h, const double* host, size_t n)
{
    int r = check_handle(h);
    if (r) return r;
    if (!host) return fail(MHD_EINVAL, "null host pointer");
    if (n != 8 * h->N) return fail(MHD_EINVAL, "state size %zu != 8*nx*ny*nz = %zu", n, 8 * h->N);
    HIP_TRY(h, hipSetDevice(h->device));
    if ((r = reset_after_set(h))) return r;
    if (h->prec == MHD_F64) {
        HIP_TRY(h, hipMemcpyAsync(h->buf[0], host, 8 * h->N * sizeof(double), hipMemcpyHostToDevice,
                                  h->stream));
    } else {
        double* stage = nullptr;
        if (hipMalloc(&stage, h->N * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            return fail(MHD_ENOMEM, "staging allocation failed");
        }
        for (int q = 0; q < 8 && !r; ++q) {
            if (hipMemcpyAsync(stage, host + (size_t)q * h->N, h->N * sizeof(double),
                               hipMemcpyHostToDevice, h->stream) != hipSuccess ||
                launch_convert_in<float>(stage, field_ptr<float>(h, q, 0), h->N, h->stream) !=
                    hipSuccess)
                r = 1;
        }
        const hipError_t e = hipStreamSynchronize(h->stream);
        (void)hipFree(stage);
        if (r || e != hipSuccess) {
            h->failed = true;
            return fail(MHD_EDEVICE, "state upload failed");
        }
    }
    return sync_stream(h);
}

extern "C" int mhd_get_state(mhd_ctx* h, double* host, size_t n)
{
    int r = check_handle(h);
    if (r) return r;
    if (!host) return fail(MHD_EINVAL, "null host pointer");
    if (n != 8 * h->N) return fail(MHD_EINVAL, "state size %zu != 8*nx*ny*nz = %zu", n, 8 * h->N);
    HIP_TRY(h, hipSetDevice(h->device));
    if (h->prec == MHD_F64) {
        for (int q = 0; q < 8; ++q)
            HIP_TRY(h, hipMemcpyAsync(host + (size_t)q * h->N, current_ptr<double>(h, q),
                                      h->N * sizeof(double), hipMemcpyDeviceToHost, h->stream));
        return sync_stream(h);
    }
    double* stage = nullptr;
    if (hipMalloc(&stage, h->N * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(MHD_ENOMEM, "staging allocation failed");
    }
    for (int q = 0; q < 8 && !r; ++q) {
        if (launch_convert_out<float>(current_ptr<float>(h, q), stage, h->N, h->stream) !=
                hipSuccess ||
            hipMemcpyAsync(host + (size_t)q * h->N, stage, h->N * sizeof(double),
                           hipMemcpyDeviceToHost, h->stream) != hipSuccess)
            r = 1;
    }
    const hipError_t e = hipStreamSynchronize(h->stream);
    (void)hipFree(stage);
    if (r || e != hipSuccess) {
        h->failed = true;
        return fail(MHD_EDEVICE, "state download failed");
    }
    return MHD_OK;
}

extern "C" int mhd_set_state_device(mhd_ctx* h, const void* src, size_t n, int prec)
{
    int r = check_handle(h);
    if (r) return r;
    if (!src) return fail(MHD_EINVAL, "null device pointer");
    if (n != 8 * h->N) return fail(MHD_EINVAL, "state size %zu != 8*nx*ny*nz = %zu", n, 8 * h->N);
    if (prec != MHD_F32 && prec != MHD_F64) return fail(MHD_EINVAL, "bad precision %d", prec);
    HIP_TRY(h, hipSetDevice(h->device));
    if ((r = reset_after_set(h))) return r;
    const size_t n8 = 8 * h->N;
    hipError_t e;
    if (prec == h->prec)
        e = hipMemcpyAsync(h->buf[0], src, n8 * h->esize, hipMemcpyDeviceToDevice, h->stream);
    else if (prec == MHD_F64)
        e = launch_cast<double, float>((const double*)src, (float*)h->buf[0], n8, h->stream);
    else
        e = launch_cast<float, double>((const float*)src, (double*)h->buf[0], n8, h->stream);
    HIP_TRY(h, e);
    return MHD_OK;
}

extern "C" int mhd_get_state_device(mhd_ctx* h, void* dst, size_t n, int prec)
{
    int r = check_handle(h);
    if (r) return r;
    if (!dst) return fail(MHD_EINVAL, "null device pointer");
    if (n != 8 * h->N) return fail(MHD_EINVAL, "state size %zu != 8*nx*ny*nz = %zu", n, 8 * h->N);
    if (prec != MHD_F32 && prec != MHD_F64) return fail(MHD_EINVAL, "bad precision %d", prec);
    HIP_TRY(h, hipSetDevice(h->device));
    const size_t es = prec == MHD_F64 ? sizeof(double) : sizeof(float);
    // one copy (or conversion) for each run of fields that lie one after another
    auto at = [&](int q) {
        return h->prec == MHD_F64 ? (char*)current_ptr<double>(h, q) : (char*)current_ptr<float>(h, q);
    };
    for (int q = 0, m; q < 8; q += m) {
        for (m = 1; q + m < 8 && at(q + m) == at(q) + m * h->N * h->esize; ++m) {}
        char* d = (char*)dst + (size_t)q * h->N * es;
        hipError_t e;
        if (prec == h->prec)
            e = hipMemcpyAsync(d, at(q), m * h->N * es, hipMemcpyDeviceToDevice, h->stream);
        else if (prec == MHD_F64)
            e = launch_cast<float, double>((const float*)at(q), (double*)d, m * h->N, h->stream);
        else
            e = launch_cast<double, float>((const double*)at(q), (float*)d, m * h->N, h->stream);
        HIP_TRY(h, e);
    }
    return MHD_OK;
}

// ---------------------------------------------------------------------------
// CFL and relaxation speed
// ---------------------------------------------------------------------------

// The CFL of the current state: from the maximum that the last launch of the
// step before left (the same FP64 expression, the same maximum) where that
// describes the state, else a reduction of its own.  step: the CFL of a
// device-dt step (record in the flag block, time advanced, accumulator left
// clear); otherwise dt, vmax and the record go to report and a valid
// accumulator stays valid.
template <typename T>
static hipError_t enqueue_cfl(mhd_ctx* h, double cfl, bool step, double* report)
{
    if (maximum_holds(h))
        return launch_cfl_from_acc(h->cfl_acc, h->n[0], cfl, h->scal, h->flag, step, report, !step, h->stream);
    const T* f[8];
    current_fields<T>(h, f);
    return launch_cfl<T>(f, h->n[0], h->n[1], h->n[2], h->gamma, cfl, h->partial, h->partial_bad,
                         h->nblk_cfl, h->scal, h->flag, step, report, step ? h->cfl_acc : nullptr, h->stream);
}

static hipError_t enqueue_cfl(mhd_ctx* h, double cfl, bool step, double* report)
{
    return h->prec == MHD_F64 ? enqueue_cfl<double>(h, cfl, step, report) : enqueue_cfl<float>(h, cfl, step, report);
}

extern "C" int mhd_cfl_dt(mhd_ctx* h, double cfl, double* dt_out)
{
    int r = check_handle(h);
    if (r) return r;
    if (!dt_out) return fail(MHD_EINVAL, "null dt pointer");
    if (!(cfl > 0.0) || !isfinite(cfl)) return fail(MHD_EINVAL, "cfl must be > 0 (got %g)", cfl);
    HIP_TRY(h, hipSetDevice(h->device));
    h->scal_known = false;
    HIP_TRY(h, enqueue_cfl(h, cfl, false, h->pinned));
    if ((r = sync_stream(h))) return r;
    if (h->pinned[2] != 0.0 && h->acc_valid) {
        // the maximum carries a record, maybe one of an earlier state that a
        // skipped step passed on: the state itself decides
        h->acc_valid = false;
        HIP_TRY(h, enqueue_cfl(h, cfl, false, h->pinned));
        if ((r = sync_stream(h))) return r;
    }
    const int bad = (int)h->pinned[2];
    if (bad == 1) {
        *dt_out = 0.0;
        return fail(MHD_ENONPHYS, "non-physical state: rho <= 0, p < 0 or non-finite value");
    }
    if (bad) {
        *dt_out = 0.0;
        return fail(MHD_EINVAL, "largest signal speed is zero: no CFL time step");
    }
    *dt_out = h->pinned[0];
    h->c_host = h->pinned[1];
    h->have_c = true;
    return MHD_OK;
}

extern "C" int mhd_set_relaxation_speed(mhd_ctx* h, double c)
{
    int r = check_handle(h);
    if (r) return r;
    if (!(c > 0.0) || !isfinite(c)) return fail(MHD_EINVAL, "relaxation speed must be > 0");
    h->c_host = c;
    h->have_c = true;
    return MHD_OK;
}

extern "C" int mhd_get_relaxation_speed(const mhd_ctx* hc, double* c)
{
    if (!hc || !c) return fail(MHD_EINVAL, "null argument");
    mhd_ctx* h = const_cast<mhd_ctx*>(hc);
    int r = check_handle(h);
    if (r) return r;
    if (!h->have_c) return fail(MHD_ESTATE, "relaxation speed not set (call mhd_cfl_dt)");
    if (h->c_host < 0.0) {      // set by a device-side CFL: read it back
        HIP_TRY(h, hipSetDevice(h->device));
        HIP_TRY(h, hipMemcpyAsync(h->pinned, h->scal + SCAL_C, sizeof(double),
                                  hipMemcpyDeviceToHost, h->stream));
        if ((r = sync_stream(h))) return r;
        h->c_host = h->pinned[0];
    }
    *c = h->c_host;
    return MHD_OK;
}

// ---------------------------------------------------------------------------
// operators
// ---------------------------------------------------------------------------

static bool mid_aside(const mhd_ctx* h);

// op 0 = fluid, 1 = magnetic, 2 = magnetic then fluid in one launch, 3 =
// magnetic twice then fluid in one launch; flag (nullable): skip-and-copy
// switch
template <typename T>
static hipError_t enqueue_op(mhd_ctx* h, int op, int d, const int* flag, unsigned long long* acc)
{
    // the faces of a middle that stands for two launches stay where those two
    // would leave them, or aside where that is what it reads
    const bool twice = op == 3 && mid_aside(h);
    SweepParams<T> P;
    for (int q = 0; q < 8; ++q) {
        P.in[q] = current_ptr<T>(h, q);
        P.out[q] = q < 5 || !twice ? field_ptr<T>(h, q, 1 - h->cur[q])
                   : h->in_aside   ? field_ptr<T>(h, q, h->cur[q])
                                   : aside_ptr<T>(h, q);
    }
    P.nx = h->n[0]; P.ny = h->n[1]; P.nz = h->n[2];
    P.gamma = (T)h->gamma;
    P.scal = h->scal;
    P.flag = flag;
    P.cfl_acc = acc;
    P.gamma64 = h->gamma;
    P.limiter = h->limiter;
    P.freeze = h->freeze;
    hipError_t e = op == 0 ? launch_fluid<T>(P, d, h->tune, h->stream)
                 : op == 1 ? launch_magnetic<T>(P, d, h->tune, h->stream)
                 : op == 2 ? launch_magfluid<T>(P, d, h->tune, h->stream)
                           : launch_magmagfluid<T>(P, d, h->tune, h->stream);
    if (e == hipSuccess) {
        if (op != 1)
            for (int q = 0; q < 5; ++q) h->cur[q] = 1 - h->cur[q];
        if (op != 0) {
            if (!twice)
                for (int q = 5; q < 8; ++q) h->cur[q] = 1 - h->cur[q];
            h->in_aside = twice && !h->in_aside;
        }
    }
    return e;
}

// acc (nullable; fluid along x, alone or fused): fused CFL accumulator
static hipError_t op(mhd_ctx* h, int o, int d, const int* flag, unsigned long long* acc = nullptr)
{
    return h->prec == MHD_F64 ? enqueue_op<double>(h, o, d, flag, acc) : enqueue_op<float>(h, o, d, flag, acc);
}

static int check_dt(double dt)
{
    if (!(dt > 0.0) || !isfinite(dt)) return fail(MHD_EINVAL, "dt must be > 0 and finite (got %g)", dt);
    return MHD_OK;
}

// checks of a host-dt call; step: the opening launch of a full step, which
// sets the scalars in any case (and advances the time, and clears the fused
// CFL's accumulator)
static int prepare_host_dt(mhd_ctx* h, double dt, bool need_c, bool step = false)
{
    int r = check_handle(h);
    if (r) return r;
    if ((r = check_dt(dt))) return r;
    // the per-cell and per-pencil freezing speeds come from the state
    if (h->freeze != MHD_FREEZE_STEP) need_c = false;
    if (need_c && !h->have_c)
        return fail(MHD_ESTATE, "relaxation speed not set: call mhd_cfl_dt or mhd_set_relaxation_speed");
    HIP_TRY(h, hipSetDevice(h->device));
    // c_host < 0: the speed was set by a device-side CFL and stays there
    const double c = h->have_c ? h->c_host : 0.0;
    if (step)
        HIP_TRY(h, launch_begin_step(h->scal, dt, c, h->cfl_acc, h->stream));
    else if (h->scal_known && h->scal_dt == dt && (c <= 0.0 || h->scal_c == c))
        return MHD_OK;
    else
        HIP_TRY(h, launch_set_scalars(h->scal, dt, c, h->flag, 0, h->stream));
    h->scal_known = c > 0.0;
    h->scal_dt = dt;
    h->scal_c = c;
    return MHD_OK;
}

extern "C" int mhd_fluid(mhd_ctx* h, int dim, double dt)
{
    if (dim < 0 || dim > 2) return fail(MHD_EINVAL, "dim must be 0, 1 or 2 (got %d)", dim);
    int r = prepare_host_dt(h, dt, true);
    if (r) return r;
    state_changes(h);
    HIP_TRY(h, op(h, 0, dim, nullptr));
    return MHD_OK;
}

extern "C" int mhd_magnetic(mhd_ctx* h, int dim, double dt)
{
    if (dim < 0 || dim > 2) return fail(MHD_EINVAL, "dim must be 0, 1 or 2 (got %d)", dim);
    int r = prepare_host_dt(h, dt, false);
    if (r) return r;
    state_changes(h);
    HIP_TRY(h, op(h, 1, dim, nullptr));
    return MHD_OK;
}

// the reverse pairs run as one fused launch each (the fused kernels take
// the step's freezing speed only)
static bool pairs_fused(const mhd_ctx* h)
{
    if (h->freeze != MHD_FREEZE_STEP) return false;
    return h->rev_mode == 1 || (h->rev_mode == 0 && default_rev_fused(h->prec, h->limiter));
}

// the built-in choice runs operator o along axis d with the tile kernels
static bool tiles(const mhd_ctx* h, int o, int d)
{
    return h->prec == MHD_F64 ? sweep_uses_tiles<double>(h->n, o, d, h->tune)
                              : sweep_uses_tiles<float>(h->n, o, d, h->tune);
}

// the reverse pair along axis d runs as one launch: as pairs_fused says for
// the marches, and, where the choice is the library's, wherever the tile
// kernels run it (none of them spills, whatever the limiter and the tier; FP64
// 64^3: 16.5 us against 11.6 + 8.3 for the two operators), and along x in FP64,
// whose row kernel holds the pair at the 2 waves per SIMD of F_x alone (with
// the CFL, against the two operators: 96^3 48.0 us / 54.8, 160^3 193.3 /
// 194.9, 256^3 714 / 746; superbee's drops to 1 wave with the CFL, and so do
// the forms with 64-bit offsets)
static bool pair_fused(const mhd_ctx* h, int d)
{
    if (pairs_fused(h)) return true;
    if (h->rev_mode != 0 || h->freeze != MHD_FREEZE_STEP) return false;
    if (d == 0)
        return h->prec == MHD_F64 && h->limiter != MHD_LIMITER_SUPERBEE && !h->tune.wide &&
               (unsigned long long)h->N * sizeof(double) <= (1ull << 32);
    return tiles(h, 2, d);
}

static bool mid_one_launch(const mhd_ctx* h);

extern "C" int mhd_sweep(mhd_ctx* h, int dim, double dt)
{
    if (dim < 0 || dim > 7) return fail(MHD_EINVAL, "sweep code must be 0..7 (got %d)", dim);
    int r = prepare_host_dt(h, dt, true);
    if (r) return r;
    state_changes(h);
    if (dim == 7) {
        // the middle of a step: M_z, then the reverse z pair
        if (mid_one_launch(h)) {
            HIP_TRY(h, op(h, 3, 2, nullptr));
        } else {
            HIP_TRY(h, op(h, 1, 2, nullptr));
            if (pair_fused(h, 2)) {
                HIP_TRY(h, op(h, 2, 2, nullptr));
            } else {
                HIP_TRY(h, op(h, 1, 2, nullptr));
                HIP_TRY(h, op(h, 0, 2, nullptr));
            }
        }
        return MHD_OK;
    }
    if (dim == 6) {
        // the reverse x pair with the fused CFL of its result
        unsigned long long* acc = h->cfl_acc;
        HIP_TRY(h, launch_clear_acc(acc, h->stream));
        if (pair_fused(h, 0)) {
            HIP_TRY(h, op(h, 2, 0, nullptr, acc));
        } else {
            HIP_TRY(h, op(h, 1, 0, nullptr));
            HIP_TRY(h, op(h, 0, 0, nullptr, acc));
        }
        maximum_follows(h);
        return MHD_OK;
    }
    const int d = dim % 3;
    if (dim < 3) {
        HIP_TRY(h, op(h, 0, d, nullptr));
        HIP_TRY(h, op(h, 1, d, nullptr));
    } else if (pair_fused(h, d)) {
        HIP_TRY(h, op(h, 2, d, nullptr));
    } else {
        HIP_TRY(h, op(h, 1, d, nullptr));
        HIP_TRY(h, op(h, 0, d, nullptr));
    }
    return MHD_OK;
}

// M_z M_z F_z of a step in one launch: FP32 (the FP64 windows would not fit
// the register file), fused reverse pairs, van Leer's limiter, the step's
// freezing speed.  Built in: from 128^3 cells up (measured 4.5% faster per
// step at 256^3 and 5% at 512^3, equal at 96^3-128^3 and 1-2% slower below,
// where launch latency dominates and the 19-cell warm-up of the one wave per
// SIMD it runs is long against the pencils)
static bool mid_fused(const mhd_ctx* h)
{
    if (!pairs_fused(h) || h->limiter != MHD_LIMITER_VANLEER || h->prec != MHD_F32) return false;
    if (h->mid_mode == 0) return h->N >= MID_CELLS;
    return h->mid_mode == 1;
}

// the same with the tile kernels counted: where the library chooses and they
// run the z axis, the middle is one launch on smaller grids too (16^3: 7.4 us
// against 4.7 + 6.6 for M_z and the pair).  A step on such a grid has always
// left every field in the buffer it started in, which a caller's captured
// step, replayed on its own buffers, relies on; one launch in place of two
// would leave the faces in the other one.  So it writes them to a third place,
// from where the next launch that writes them goes on as after the two.  A
// chunk that the caller set for M_z or the z pair asks for those two.
static bool mid_aside(const mhd_ctx* h)
{
    return h->aside && h->mid_mode == 0 && !h->tune.set_chunk[2] && !h->tune.set_pair[2] && pairs_fused(h) && h->limiter == MHD_LIMITER_VANLEER && tiles(h, 3, 2);
}
static bool mid_one_launch(const mhd_ctx* h)
{
    return mid_fused(h) || mid_aside(h);
}

// the 12 operators of a full step: x, y, z forward (fluid, magnetic), then
// z, y, x reverse (magnetic, fluid), each reverse pair in one launch when
// pair_fused (9 launches), and M_z with the z pair in one when mid_one_launch
// (8 launches).  acc (nullable): the last operator (F_x) also accumulates
// the CFL maximum of the state it leaves.
static int enqueue_step_ops(mhd_ctx* h, const int* flag, unsigned long long* acc)
{
    const bool mid = mid_one_launch(h);
    for (int d = 0; d < 3; ++d) {
        HIP_TRY(h, op(h, 0, d, flag));
        if (d == 2 && mid) {
            HIP_TRY(h, op(h, 3, 2, flag));
            break;
        }
        HIP_TRY(h, op(h, 1, d, flag));
    }
    for (int d = mid ? 1 : 2; d >= 0; --d) {
        if (pair_fused(h, d)) {
            HIP_TRY(h, op(h, 2, d, flag, d == 0 ? acc : nullptr));
        } else {
            HIP_TRY(h, op(h, 1, d, flag));
            HIP_TRY(h, op(h, 0, d, flag, d == 0 ? acc : nullptr));
        }
    }
    return MHD_OK;
}

extern "C" int mhd_set_limiter(mhd_ctx* h, int limiter)
{
    int r = check_handle(h);
    if (r) return r;
    if (limiter < MHD_LIMITER_VANLEER || limiter > MHD_LIMITER_SUPERBEE)
        return fail(MHD_EINVAL, "limiter must be 0..3 (got %d)", limiter);
    if (limiter != MHD_LIMITER_VANLEER && h->freeze != MHD_FREEZE_STEP)
        return fail(MHD_EINVAL, "the freezing-speed variants come with van Leer's limiter only");
    h->limiter = limiter;
    return MHD_OK;
}

extern "C" int mhd_set_freezing_speed(mhd_ctx* h, int mode)
{
    int r = check_handle(h);
    if (r) return r;
    if (mode < MHD_FREEZE_STEP || mode > MHD_FREEZE_PENCIL)
        return fail(MHD_EINVAL, "freezing-speed mode must be 0..2 (got %d)", mode);
    if (mode != MHD_FREEZE_STEP && h->limiter != MHD_LIMITER_VANLEER)
        return fail(MHD_EINVAL, "the freezing-speed variants come with van Leer's limiter only");
    h->freeze = mode;
    return MHD_OK;
}

extern "C" int mhd_get_freezing_speed(const mhd_ctx* h, int* mode)
{
    int r = check_handle(h);
    if (r) return r;
    if (!mode) return fail(MHD_EINVAL, "null output");
    *mode = h->freeze;
    return MHD_OK;
}

extern "C" int mhd_get_limiter(const mhd_ctx* h, int* limiter)
{
    int r = check_handle(h);
    if (r) return r;
    if (!limiter) return fail(MHD_EINVAL, "null output");
    *limiter = h->limiter;
    return MHD_OK;
}

extern "C" int mhd_step(mhd_ctx* h, double dt)
{
    int r = prepare_host_dt(h, dt, true, true);
    if (r) return r;
    state_changes(h);
    if ((r = enqueue_step_ops(h, nullptr, h->cfl_acc))) return r;
    maximum_follows(h);
    return MHD_OK;
}

extern "C" int mhd_step_auto(mhd_ctx* h, double cfl)
{
    int r = check_handle(h);
    if (r) return r;
    if (!(cfl > 0.0) || !isfinite(cfl)) return fail(MHD_EINVAL, "cfl must be > 0 (got %g)", cfl);
    HIP_TRY(h, hipSetDevice(h->device));
    h->scal_known = false;
    HIP_TRY(h, enqueue_cfl(h, cfl, true, nullptr));
    state_changes(h);
    if ((r = enqueue_step_ops(h, h->flag + FLAG_NONPHYS, h->cfl_acc))) return r;
    maximum_follows(h);
    // the device CFL also set the relaxation speed; it stays on the device
    // (c_host < 0 marks that) until read back
    h->have_c = true;
    h->c_host = -1.0;
    return MHD_OK;
}

extern "C" int mhd_status(mhd_ctx* h, long long* steps_out)
{
    int r = check_handle(h);
    if (r) return r;
    HIP_TRY(h, hipSetDevice(h->device));
    HIP_TRY(h, hipMemcpyAsync(h->pinned, h->flag, FLAG_COUNT * sizeof(int), hipMemcpyDeviceToHost,
                              h->stream));
    HIP_TRY(h, hipMemcpyAsync(h->pinned + 4, h->scal, SCAL_COUNT * sizeof(double),
                              hipMemcpyDeviceToHost, h->stream));
    if ((r = sync_stream(h))) return r;
    int fl[FLAG_COUNT];
    memcpy(fl, h->pinned, sizeof fl);
    if (steps_out) *steps_out = fl[FLAG_STEPS];
    if (fl[FLAG_NONPHYS]) {
        h->acc_valid = false;       // skipped steps left the record in it, not a maximum
        HIP_TRY(h, hipMemsetAsync(h->flag + FLAG_NONPHYS, 0, sizeof(int), h->stream));
        if ((r = sync_stream(h))) return r;
        return fl[FLAG_NONPHYS] == 1
                   ? fail(MHD_ENONPHYS, "non-physical state found by the device CFL; steps skipped")
                   : fail(MHD_EINVAL, "largest signal speed is zero; steps skipped");
    }
    return MHD_OK;
}

extern "C" int mhd_time(mhd_ctx* h, double* t)
{
    int r = check_handle(h);
    if (r) return r;
    if (!t) return fail(MHD_EINVAL, "null pointer");
    HIP_TRY(h, hipSetDevice(h->device));
    HIP_TRY(h, hipMemcpyAsync(h->pinned, h->scal + SCAL_TIME, sizeof(double), hipMemcpyDeviceToHost,
                              h->stream));
    if ((r = sync_stream(h))) return r;
    *t = h->pinned[0];
    return MHD_OK;
}

// ---------------------------------------------------------------------------
// diagnostics and restriction
// ---------------------------------------------------------------------------

template <typename T>
static hipError_t enqueue_diag(mhd_ctx* h)
{
    const T* f[8];
    current_fields<T>(h, f);
    return launch_diag<T>(f, h->n[0], h->n[1], h->n[2], h->partial, h->nblk_diag, h->pinned, h->stream);
}

extern "C" int mhd_diag(mhd_ctx* h, double out[9])
{
    int r = check_handle(h);
    if (r) return r;
    if (!out) return fail(MHD_EINVAL, "null output");
    HIP_TRY(h, hipSetDevice(h->device));
    HIP_TRY(h, h->prec == MHD_F64 ? enqueue_diag<double>(h) : enqueue_diag<float>(h));
    if ((r = sync_stream(h))) return r;
    memcpy(out, h->pinned, 9 * sizeof(double));
    return MHD_OK;
}

template <typename T>
static hipError_t enqueue_restrict(mhd_ctx* fine, mhd_ctx* coarse, int r)
{
    const T* f[8];
    T* c[8];
    current_fields<T>(fine, f);
    for (int q = 0; q < 8; ++q) c[q] = field_ptr<T>(coarse, q, 0);
    return launch_restrict<T>(f, c, fine->n[0], fine->n[1], fine->n[2], r, coarse->stream);
}

extern "C" int mhd_restrict(mhd_ctx* fine, mhd_ctx* coarse)
{
    int r = check_handle(fine);
    if (r) return r;
    if ((r = check_handle(coarse))) return r;
    if (fine == coarse) return fail(MHD_EINVAL, "fine and coarse handles must differ");
    if (fine->prec != coarse->prec) return fail(MHD_EINVAL, "precision tiers differ");
    if (fine->device != coarse->device) return fail(MHD_EINVAL, "handles on different devices");
    if (fine->n[0] % coarse->n[0]) return fail(MHD_EINVAL, "coarse nx does not divide fine nx");
    const int f = fine->n[0] / coarse->n[0];
    for (int d = 0; d < 3; ++d)
        if (coarse->n[d] * f != fine->n[d])
            return fail(MHD_EINVAL, "fine/coarse sizes are not one integer factor on every axis");
    HIP_TRY(fine, hipSetDevice(fine->device));
    HIP_TRY(fine, hipStreamSynchronize(fine->stream));
    if ((r = reset_after_set(coarse))) return r;
    HIP_TRY(coarse, fine->prec == MHD_F64 ? enqueue_restrict<double>(fine, coarse, f)
                                          : enqueue_restrict<float>(fine, coarse, f));
    return MHD_OK;
}

extern "C" int mhd_set_launch(mhd_ctx* h, int key, int value)
{
    int r = check_handle(h);
    if (r) return r;
    if (key == MHD_TUNE_REVERSE) {
        if (value < 0 || value > 2)
            return fail(MHD_EINVAL, "reverse-half choice must be 0, 1 or 2 (got %d)", value);
        h->rev_mode = value;
        return MHD_OK;
    }
    if (key == MHD_TUNE_WIDE_OFFSETS) {
        if (value < 0 || value > 1) return fail(MHD_EINVAL, "wide-offset switch must be 0 or 1 (got %d)", value);
        h->tune.wide = value;
        return MHD_OK;
    }
    if (key == MHD_TUNE_MIDDLE) {
        if (value < 0 || value > 2)
            return fail(MHD_EINVAL, "middle-of-step choice must be 0, 1 or 2 (got %d)", value);
        h->mid_mode = value;
        return MHD_OK;
    }
    if (key == MHD_TUNE_ROW_GROUP) {
        if (value < 0) return fail(MHD_EINVAL, "row group must be >= 0 (got %d)", value);
        h->tune.row_group = value;
        return MHD_OK;
    }
    const bool pair = key == MHD_TUNE_PAIR_CHUNK_Y || key == MHD_TUNE_PAIR_CHUNK_Z;
    const bool triple = key == MHD_TUNE_MIDDLE_CHUNK;
    if (key != MHD_TUNE_CHUNK_Y && key != MHD_TUNE_CHUNK_Z && !pair && !triple)
        return fail(MHD_EINVAL, "unknown launch key %d", key);
    const int d = triple ? 2 : pair ? key - MHD_TUNE_PAIR_CHUNK_Y + 1 : key;   // axis 1 (y) or 2 (z)
    bool* set = triple ? &h->tune.set_triple[d] : pair ? &h->tune.set_pair[d] : &h->tune.set_chunk[d];
    int* slot = triple ? &h->tune.triple_chunk[d] : pair ? &h->tune.pair_chunk[d] : &h->tune.chunk[d];
    if (value == 0) {
        const LaunchTuning keep = h->tune;
        default_tuning(h);
        const int v = *slot;
        h->tune = keep;
        *slot = v;
        *set = false;
        return MHD_OK;
    }
    if (value < 8 || h->n[d] % value)
        return fail(MHD_EINVAL, "chunk %d must be >= 8 and divide the axis length %d", value, h->n[d]);
    *slot = value;
    *set = true;
    return MHD_OK;
}

extern "C" int mhd_get_launch(const mhd_ctx* h, int key, int* value)
{
    if (!h || !value) return fail(MHD_EINVAL, "null argument");
    if (key == MHD_TUNE_REVERSE) {
        *value = pairs_fused(h) ? 1 : 2;
        return MHD_OK;
    }
    if (key == MHD_TUNE_WIDE_OFFSETS) {
        *value = h->tune.wide;
        return MHD_OK;
    }
    if (key == MHD_TUNE_MIDDLE) {
        *value = mid_fused(h) ? 1 : 2;
        return MHD_OK;
    }
    if (key == MHD_TUNE_MIDDLE_CHUNK) {
        *value = h->tune.triple_chunk[2];
        return MHD_OK;
    }
    if (key == MHD_TUNE_ROW_GROUP) {
        const int rpw = x_rows_per_wg(h->n[0]);
        const int st = row_group_tiles(h->n[1], rpw, h->tune.row_group);
        *value = (st <= 0 || st * rpw >= h->n[1]) ? h->n[1] : st * rpw;
        return MHD_OK;
    }
    if (key == MHD_TUNE_PAIR_CHUNK_Y || key == MHD_TUNE_PAIR_CHUNK_Z) {
        *value = h->tune.pair_chunk[key - MHD_TUNE_PAIR_CHUNK_Y + 1];
        return MHD_OK;
    }
    if (key != MHD_TUNE_CHUNK_Y && key != MHD_TUNE_CHUNK_Z)
        return fail(MHD_EINVAL, "unknown launch key %d", key);
    *value = h->tune.chunk[key];
    return MHD_OK;
}

// The operators flip the fluid fields and the faces each as a group, and
// after a step the two need not share a buffer: the fused middle of a step
// writes b once for two magnetic operators.
void mhd_internal_state(mhd_ctx* h, void** fluid, void** faces, void** first)
{
    *fluid = h->buf[h->cur[0]];
    *faces = h->buf[h->cur[5]];
    *first = h->buf[0];
}
int mhd_internal_prec(const mhd_ctx* h) { return h->prec; }
void mhd_internal_dims(const mhd_ctx* h, int n[3]) { n[0] = h->n[0]; n[1] = h->n[1]; n[2] = h->n[2]; }
hipStream_t mhd_internal_stream(const mhd_ctx* h) { return h->stream; }
void mhd_internal_state_changed(mhd_ctx* h)
{
    for (int q = 0; q < 8; ++q) h->cur[q] = 0;
    h->in_aside = false;
    h->acc_valid = false;
}

double mhd_internal_gamma(const mhd_ctx* h) { return h->gamma; }

extern "C" int mhd_stream_copy(const void* src, void* dst, size_t bytes, void* stream)
{
    if (!src || !dst) return fail(MHD_EINVAL, "null device pointer");
    if (bytes % 16 || reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(dst) % 16)
        return fail(MHD_EINVAL, "the copy moves 16-byte words: size and both pointers must be multiples of 16");
    const char* a = static_cast<const char*>(src);
    const char* b = static_cast<const char*>(dst);
    if (a < b + bytes && b < a + bytes) return fail(MHD_EINVAL, "source and destination overlap");
    if (bytes == 0) return MHD_OK;
    const hipError_t e = launch_stream_copy(src, dst, bytes, (hipStream_t)stream);
    if (e != hipSuccess) return fail(MHD_EDEVICE, "stream copy: %s", hipGetErrorString(e));
    return MHD_OK;
}

extern "C" const char* mhd_last_error(void)
{
    return g_last_error.c_str();
}
