// Internal declarations of the learned-proposal MLP.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pump {

constexpr int kComp = 16;               // mixture components
constexpr int kDState = 6;              // state dimension
constexpr int kMaxBoxes = 64;           // boxes in the condition vector
constexpr int kIn = 12 + 6 * kMaxBoxes; // 396 condition values
constexpr int kInPad = 416;             // padded to a multiple of 32
constexpr int kHidden = 256;
constexpr int kOut = kComp * (1 + 2 * kDState);  // 208 outputs
constexpr int kOutPad = 224;
constexpr int kLayers = 5;              // 4 hidden + output
constexpr float kLogStdMin = -4.0f, kLogStdMax = 2.0f;

constexpr int kBiasTotal = 4 * kHidden + kOut;   // bias entries of all layers

// Shapes of layer l: real and padded (multiples of 32).
__host__ __device__ constexpr int mlp_in(int l) { return l == 0 ? kIn : kHidden; }
__host__ __device__ constexpr int mlp_in_p(int l) { return l == 0 ? kInPad : kHidden; }
__host__ __device__ constexpr int mlp_out(int l) { return l == kLayers - 1 ? kOut : kHidden; }
__host__ __device__ constexpr int mlp_out_p(int l) { return l == kLayers - 1 ? kOutPad : kHidden; }

// Network state and buffers the kernels read and write.
struct MlpDev {
    int off_W[kLayers], off_b[kLayers];    // into params and grads
    float *params, *m1, *m2, *grads;       // [n_params]
    uint16_t *Wb[kLayers], *WbT[kLayers];  // BF16 weights [out_p][in_p] and [in_p][out_p], in fragment order
    // a training step, batch rows contiguous (Bp of them)
    uint16_t* HT[kLayers];                 // layer inputs [in_p][Bp], in fragment order
    uint16_t* GT[kLayers];                 // output gradients [out_p][Bp], likewise
    float* bpart;                          // bias gradients [Bp / 16][kBiasTotal]
    float* lpart;                          // losses [Bp / 16]
    int n_params;
};

// out[m * ld + n] (n < n_out, m < rows) = the network's outputs for the
// condition rows X [B][kIn].
void launch_mlp_forward(hipStream_t s, const MlpDev& d, const float* X, int B, float* out, int ld,
                        int n_out, int rows);
// Loss and gradients of a batch, in two launches: the rows through the network
// and back (layer inputs, output gradients, bias and loss partials), then the
// gradients (into grads) and the mean loss (*loss, memory the device can
// write).
void launch_mlp_grad(hipStream_t s, const MlpDev& d, const float* X, const float* Z, int B, int Bp,
                     float* loss);
// One Adam step (t counts from 1) on grads, and the BF16 weights it changes.
void launch_adam(hipStream_t s, const MlpDev& d, float lr, int t);
// BF16 weights from the parameters, padding zeroed.
void launch_refresh_bf16(hipStream_t s, const MlpDev& d);
void launch_condition(hipStream_t s, const float* x_init, const float* goal, const float* boxes,
                      const int32_t* n_obs, int q, int max_boxes_in, float* cond);
void launch_sample(hipStream_t s, const float* Y, int ldy, int q, int n, const float* u,
                   const float* eps, float* out);

}  // namespace pump
