// Learned-closure kernels: BF16 MFMA convolutions and helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mhd {

enum {
    EPI_BIAS_RELU = 0,   // y = relu(acc + bias) -> bf16 (32 output channels)
    EPI_BIAS_F32 = 1,    // y = acc + bias -> fp32
    EPI_MASK = 2,        // y = acc * (mask > 0) -> bf16 (32 output channels)
    EPI_F32 = 3,         // y = acc -> fp32
    EPI_CLOSURE = 4      // y = (acc + bias) gate -> fp32, and its channel sums (32 -> 8 channels)
};

struct ConvArgs {
    int n[3];
    const uint16_t* x;      // bf16 [cell][cin]
    const uint16_t* wp;     // packed weights
    const float* bias;      // [cout] (bias epilogues)
    const float* gate;      // [cell] or null (EPI_CLOSURE)
    double* sums;           // [closure_sum_blocks][8] (EPI_CLOSURE)
    const uint16_t* mask;   // bf16 [cell][cout] (EPI_MASK)
    float* yf;              // fp32 [cell][cout]
    uint16_t* yb;           // bf16 [cell][cout]
};

struct WgradArgs {
    int n[3];
    const uint16_t* x;      // bf16 [cell][cin]
    const uint16_t* dy;     // bf16 [cell][cout]
    float* partial;         // [workgroups][27][cin][cout]
    double* bias_partial;   // [workgroups][cout]
};
constexpr int WGRAD_MAX_WG = 512;   // persistent workgroups of wgrad (bounds the partial sums)
// a layer of a reduction of partial sums
struct WgradLayer {
    const float* partial;
    const double* bias_partial;
    float* dw;              // [27][cin][cout]
    float* dbias;           // [cout]
    int count, cout;        // 27 cin cout (a multiple of 64)
};

// packed size (bf16 elements) of a layer's weights
inline size_t packed_weight_elems(int cin, int cout)
{
    return (size_t)((27 * cin + 31) / 32) * ((cout + 15) / 16) * 64 * 8;
}

hipError_t launch_pack_weights(const float* w, int cin, int cout, int flip, uint16_t* wp, hipStream_t s);
hipError_t launch_conv3d(const ConvArgs& A, int cin, int cout, int epi, hipStream_t s);
int wgrad_blocks(const int n[3]);                       // workgroups of a wgrad launch
hipError_t launch_conv3d_wgrad(const WgradArgs& A, int cin, int cout, hipStream_t s);
// grads of the layers, and (loss_partial not null) the loss over N cells from
// the sums of launch_project_loss
hipError_t launch_wgrad_reduce(const WgradLayer* layers, int nlayer, int nwg, const double* loss_partial, size_t N,
                               double* loss, hipStream_t s);
hipError_t launch_channel_last(const uint16_t* src, size_t N, int c, uint16_t* dst, hipStream_t s);

// per-channel input normalisation, output and target scales of the closure
struct ClosureScales {
    float in_mean[8], in_std[8], out_scale[8], target_scale[8];
};
// a state of 8 fields of N cells: field f at fluid + f N (f < 5) or faces + f N
struct ClosureState {
    const float* fluid;
    const float* faces;
};
constexpr int LOSS_BLOCKS = 1024, LOSS_SUMS = 6;    // workgroups and sums of launch_project_loss

hipError_t launch_normalize(const ClosureState& u, size_t N, const ClosureScales& sc, uint16_t* x, hipStream_t s);
int closure_sum_blocks(const int n[3]);             // workgroups that write EPI_CLOSURE channel sums
int loss_blocks(size_t N);                          // workgroups that write loss sums
hipError_t launch_project(const float* o, const double* sums, int nsums, const int n[3], const ClosureScales& sc,
                          float* delta, int* clear, hipStream_t s);
hipError_t launch_project_loss(const float* o, const double* sums, int nsums, const int n[3], const ClosureScales& sc,
                               const float* target, float* g, double* partial, hipStream_t s);
hipError_t launch_project_T(const float* g, const double* partial, const float* gate, const int n[3],
                            const ClosureScales& sc, uint16_t* go, hipStream_t s);
constexpr int GUARD_LEVELS = 4;     // theta = 1, 1/2, 1/4, 1/8
hipError_t launch_guard_levels(const ClosureState& u, const float* delta, const int n[3], float gamma, int* bad,
                               hipStream_t s);
hipError_t launch_apply_level(const ClosureState& u, const float* delta, size_t N, const int* bad, int* counts,
                              float* out, hipStream_t s);
constexpr int STATS_BLOCKS = 256;
hipError_t launch_residual(const float* ref, const float* plain, size_t n, float* out, hipStream_t s);
hipError_t launch_stats(const float* u, const float* t, const int n[3], double* partial, double* out, hipStream_t s);
struct GateScales {
    float inv_r[8];     // 1 / (training-set mean roughness) per field
};
// the gate g (g0: scratch) and the network input x of a state
hipError_t launch_gate(const ClosureState& u, const int n[3], const GateScales& gs, const ClosureScales& sc, float* g0,
                       float* g, uint16_t* x, hipStream_t s);
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       int step, hipStream_t s);

}  // namespace mhd
