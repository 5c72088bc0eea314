// Host-side helpers shared by the single-grid and batched runtimes.
#pragma once
#include <hip/hip_runtime.h>

// Record a thread-local error message (mhd_last_error) and return code.
int mhd_fail(int code, const char* fmt, ...);

#define MHD_HIP_TRY(h, expr)                                                           \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess) {                                                        \
            (h)->failed = true;                                                        \
            return mhd_fail(MHD_EDEVICE, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                            __FILE__, __LINE__);                                       \
        }                                                                              \
    } while (0)

// The graph capture that records what is enqueued on the stream, 0 for none
// (the legacy default stream takes part in none).
inline unsigned long long mhd_capture_id(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (!s || hipStreamGetCaptureInfo(s, &status, &id) != hipSuccess) return 0;
    return status == hipStreamCaptureStatusActive ? id : 0;
}

// Internal accessors of a single-grid handle (used by the closure runtime).
struct mhd_ctx;
// the buffers ([8][cell]) that hold the fluid fields (0 - 4) and the faces (5 - 7), and the first one
void mhd_internal_state(mhd_ctx* h, void** fluid, void** faces, void** first);
int mhd_internal_prec(const mhd_ctx* h);
void mhd_internal_dims(const mhd_ctx* h, int n[3]);
hipStream_t mhd_internal_stream(const mhd_ctx* h);
double mhd_internal_gamma(const mhd_ctx* h);
void mhd_internal_state_changed(mhd_ctx* h);   // a state made outside the operators is in the first buffer
