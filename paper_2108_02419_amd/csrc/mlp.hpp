// mlp.hpp -- sizes, packed parameter layout and kernel arguments of the
// surrogate network.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "race_common.hpp"

namespace bbe {

constexpr int kIn = 160;    // 20 slots x 8 features
constexpr int kHid = 256;
constexpr int kOut = 20;
constexpr int kOutP = 32;   // output rows padded to two 16-wide blocks

// Packed float32 parameters: W1 [256][160], b1, W2 [256][256], b2,
// W3 [256][256], b3, W4 [20][256], b4.
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kHid * kIn;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid * kHid;
constexpr int kOffW4 = kOffB3 + kHid;
constexpr int kOffB4 = kOffW4 + kOut * kHid;
constexpr int kNParams = kOffB4 + kOut;
static_assert(kNParams == 177940, "parameter count");

// a thread's four parameters lie in one layer
static_assert(kOffB1 % 4 == 0 && kOffW2 % 4 == 0 && kOffB2 % 4 == 0 && kOffW3 % 4 == 0 &&
                  kOffB3 % 4 == 0 && kOffW4 % 4 == 0 && kOffB4 % 4 == 0 && kNParams % 4 == 0,
              "layers in whole groups of four parameters");

// Forward pass (and, for training, the gradients of the pre-activations).
// Fragment order: see mlp_kernels.hip.
struct MlpArgs {
    const uint16_t* x;        // [B][160] bf16
    const int32_t* n_valid;   // [B]
    int B;
    // bf16 weights in fragment order: [256][160], [256][256] x2, [32][256],
    // and for training the transposes [256][32], [256][256] x2
    const uint16_t *w1, *w2, *w3, *w4, *w4t, *w3t, *w2t;
    const float *b1, *b2, *b3, *b4;
    uint16_t *h1, *h2, *h3;   // [B][256] bf16 or null (inference)
    float* probs;             // [B][20] or null
    float* entropy;           // [B] or null
    float* logits;            // [B][32] or null
    // training
    const float* target;      // [B][20]
    float inv_batch;
    float* loss_part;         // [workgroups]
    uint16_t *xf, *hf1, *hf2, *hf3;       // inputs of the layers, fragment order over the batch
    uint16_t *df1, *df2, *df3, *df4;      // gradients of the pre-activations, the same
};

struct LayerGrad {
    const uint16_t* dz;  // gradients of the outputs, fragment order over the batch
    const uint16_t* h;   // inputs of the layer, the same
    int K;
    int n_rows;          // outputs of the layer
    float* gw;           // [n_rows][K]
    float* gb;           // [n_rows]
    int woff;            // offset of gw in the packed parameter vector
};

// Rows of the batch per weight-gradient work item.
constexpr int kWgRows = 256;

struct WgradTile {
    int layer, n0, k0, pad;
};

struct MlpWgradArgs {
    int B;
    int n_parts;  // mlp_wgrad_parts(B)
    LayerGrad layers[4];
    const WgradTile* tiles;
    // partial weight gradients, one packed parameter vector per chunk of
    // kWgRows rows (used when B > kWgRows); summed in chunk order
    float* part;
    const float* loss_part;  // [n_loss], summed into loss
    int n_loss;
    float* loss;
};

// Chunks (= partial gradients) of a batch.
constexpr int mlp_wgrad_parts(int B) { return (B + kWgRows - 1) / kWgRows; }

struct MlpAdamArgs {
    float* params;
    float *m, *v;
    // the gradient: a vector, or n_parts partials to sum into grad_out; both
    // null: refresh the bf16 copies only
    const float* grad;
    const float* part;
    int n_parts;
    float* grad_out;
    float lr, beta1, beta2, eps, inv_bc1, inv_bc2;
    uint16_t *w1, *w2, *w3, *w4, *w2t, *w3t, *w4t;
};

struct EncodeArgs {
    const float* comp;   // [B][20][5]
    const int32_t* n;    // [B]
    const float* pos;    // [B][20]
    const float* prev;   // [B][20]
    int B;
    float track_len, c75, c15, c750;  // 7.5 dt, 15 dt, 75 dt
    uint16_t* x;         // [B][160]
    int32_t* slot;       // [B][20] or null
    const double* probs_in;  // [B][20] competitor order, or null
    float* target;           // [B][20] slot order (with probs_in)
};

hipError_t launch_mlp_fwd(const MlpArgs& a, hipStream_t s);
hipError_t launch_mlp_train(const MlpArgs& a, hipStream_t s);
int mlp_train_groups(int B);  // workgroups of launch_mlp_train
hipError_t launch_mlp_wreduce(const float* part, int n_parts, float* grad, hipStream_t s);
hipError_t launch_mlp_wgrad(const MlpWgradArgs& a, int n_tiles, hipStream_t s);
hipError_t launch_mlp_adam(const MlpAdamArgs& a, hipStream_t s);
hipError_t launch_encode(const EncodeArgs& a, hipStream_t s);

}  // namespace bbe
