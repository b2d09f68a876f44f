// Host-side launchers of the learned-initialiser kernels (lbml_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "lbml.h"

namespace lbml {

constexpr int kIn = 4;       // inputs: a, T/T_c, R, nu_g/nu_l (standardised)
constexpr int kInPad = 32;   // first-layer depth padded to one matrix-core step
constexpr int kHidden = 256;
constexpr int kOut = 128;    // log-density samples across the interface
constexpr double kSmooth = 1e-4;  // weight of the profile fit's smoothness term

// Device state of a training loop: the step being run (cur), the next one, the running powers b1^t and b2^t of Adam's bias
// correction (FP64, multiplied once per step as the host does), and the current
// step's learning rate and FP32 bias corrections.
struct TrainSched {
    int cur, next;
    double p1, p2;
    float lr, c1, c2;
    int bad_rows;
};

hipError_t gemm(const __bf16* A, long long sam, long long sak, const __bf16* B, long long sbk, long long sbn,
                float* C, int ldc, int M, int N, int K, hipStream_t s);

// One pass of a batch through the network.  Layers 0 .. 3: w[i] [out][in, padded] and wt[i]
// [in][out] (i > 0) bf16 weights, bias[i].  These and the bf16 outputs below are in fragment
// order (frag_at in lbml_kernels.hip).  Row m of the batch is row m of x, base (may be
// NULL), target and y, or row idx[sc->next][m] of them.  Forward: y = network(x) + base.
// Training: the first four rows of xT [16][B], hT[i] [256][B], dzT[i] [out][B] and the loss sums
// loss_part [B / mlp_rows(B)]; with sc also the step's learning rate and bias corrections.
struct MlpArgs {
    const float *x, *base, *target;
    const int* idx;
    TrainSched* sc;
    const float* lr;
    double b1, b2;
    const float* norm;  // feature means, then inverse standard deviations
    const __bf16 *w[4], *wt[4];
    const float* bias[4];
    float* y;
    __bf16 *xT, *hT[3], *dzT[4];
    float* loss_part;
    int B;
};
// B a multiple of 16 (forward) or 32 (training).  mlp_rows(B): rows per workgroup.
int mlp_rows(int B);
hipError_t launch_mlp_pass(const MlpArgs& a, bool train, hipStream_t s);

// Gradients of all parameters from a training pass (inT[0] = xT, inT[i] = hT[i-1]) and the mean
// loss; update: Adam on the parameters with the schedule's current values, their bf16 copies,
// loss_out[sc->cur] (if not NULL) and the step count.
struct GradArgs {
    const __bf16 *dzT[4], *inT[4];
    const float* loss_part;
    float *grad, *loss, *loss_out;
    float *theta, *m, *v;
    __bf16 *w[4], *wt[4];
    int w_off[4];
    TrainSched* sc;
    float b1, b2, eps;
    int B, parts;  // parts = B / mlp_rows(B)
};
hipError_t launch_mlp_grads(const GradArgs& g, bool update, hipStream_t s);
hipError_t launch_adam(float* p, float* m, float* v, const float* g, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t s);
hipError_t launch_check_rows(const int* idx, long long n, int rows, int* flag, hipStream_t s);
hipError_t launch_to_bf16(const float* src, __bf16* dst, __bf16* dst_t, int rows, int cols, int pad, hipStream_t s);
hipError_t launch_fill(void* p, size_t bytes, hipStream_t s);
hipError_t launch_profiles_extract(const lbml_fit* p, int n, hipStream_t s);
hipError_t launch_profile_extract(const float* rho, int nx, int ny, double cx, double cy, double R, double* part,
                                  float* logrho, hipStream_t s);
// The same fit with its row partials in the library's static device scratch (ny up to
// static_profile_rows()); hipErrorInvalidValue for a larger ny.
hipError_t launch_profile_extract_static(const float* rho, int nx, int ny, double cx, double cy, double R,
                                         float* logrho, hipStream_t s);
int static_profile_rows();
hipError_t launch_profile_to_rho0(const float* logrho, double R, double cx, double cy, int nx, int ny, float* rho0,
                                  hipStream_t s);
hipError_t launch_profiles_to_rho0_mass(const lbml_placement* p, int n, hipStream_t s);
hipError_t launch_profile_levels(const float* L, const float* x, int B, double* lev, hipStream_t s);
hipError_t launch_profile_anchor(float* L, const float* x, const double* target, int B, hipStream_t s);

}  // namespace lbml
