// Internal interface of the layer-wise calibration kernels (kq_calib.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace kq {

// Work split and workspace layout of one calibration problem: R activation
// rows, o output features, d input features, nfac factor sets of split a.
struct CalibPlan {
    int64_t R = 0, o = 0, d = 0, nb = 0, nfac = 0;
    int a = 4;
    bool big = true;                      // 256 x 256 tiles of the backward products, else 128 x 128
    bool fold = false;                    // the backward products' block sums go onto the quantizer's, no gpa and gpw
    int64_t ntn = 0;                      // column tiles of the d axis
    int64_t act_mt = 0, act_ks = 0, act_kchunk = 0;  // activation side: row tiles, K parts and their length
    int64_t w_mt = 0, w_ks = 0, w_kchunk = 0;        // weight side
    int64_t nsum = 0;                     // room for the partial sums of the residual's squares
    int64_t Rp = 0, op = 0;               // R and o rounded up to the 32-deep K stage
    // byte offsets into the workspace (each 256-byte aligned)
    // of X and W: codes, scales, dequantized bf16, clipped-element words, the quantizer's
    // per-strip sums over clipped elements (strips_*) and sums of squares (nsq*)
    size_t cA = 0, sA = 0, qA = 0, mA = 0, dA = 0, cW = 0, sW = 0, qW = 0, mW = 0, dW = 0;
    int64_t strips_a = 0, strips_w = 0, nsqa = 0, nsqw = 0;
    size_t rh = 0, rl = 0;                // the residual's two bf16 terms [Rp, op]
    size_t gpa = 0, gpw = 0, sqa = 0, sqw = 0, sr = 0;
    size_t grad = 0, am = 0, av = 0, lam = 0;
    size_t total = 0;                     // what a caller's workspace holds
};

CalibPlan calib_plan(int64_t R, int64_t o, int64_t d, int a, int64_t nfac);

// Yneg[r][n] = -sum_c X[r][c] W[n][c] (bf16 matrix cores, exact products, fp32 accumulation).
hipError_t launch_calib_reference(const uint16_t* X, int64_t R, int64_t d, const uint16_t* W, int64_t o,
                                  float* Yneg, hipStream_t st);

struct CalibStepArgs {
    const uint16_t* X;      // [R, d] bf16
    const uint16_t* W;      // [o, d] bf16
    const float* lu;        // [nfac, 5, 3]
    const float* lambdas;   // device [2]: lambda_A, lambda_W
    float* grad;            // [nfac, 5, 3]
    double* losses;         // device [4]: L_out, L_A, L_W, L
    float* lu_out;          // parameters updated in place when adam_t > 0 (== lu)
    float* adam_m;          // [nfac * 15]
    float* adam_v;          // [nfac * 15]
    int adam_t;             // 1-based Adam step; 0 = no update
    float lr;
    unsigned char* ws;      // workspace laid out by the plan
};

// Backward and update part of a step; the quantizer's outputs, the residual's terms and
// the nsr partial sums of its squares must already be in the workspace.
hipError_t launch_calib_backward(const CalibPlan& pl, const CalibStepArgs& s, int64_t nsr, hipStream_t st);

// Small helpers of the calibration loop.
hipError_t launch_calib_init(float* adam_m, float* adam_v, int64_t n, float* lambdas, hipStream_t st);
hipError_t launch_calib_set_lambdas(const double* losses, float* lambdas, hipStream_t st);

}  // namespace kq
