// Warm-start network shapes, parameter layout and device state (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>

namespace vrm {

constexpr int kMlpSlots = 32;    // LP columns seen by the network
constexpr int kMlpIn = 128;      // 2 * 32 offsets, 32 masks, q - 2, padding
constexpr int kMlpHid = 128;
constexpr int kMlpOut = 64;      // 32 basis logits, 32 fractions
// FP32 parameter vector: W1[in][hid], b1, W2[hid][hid], b2, W3[hid][out], b3
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kMlpIn * kMlpHid;
constexpr int kOffW2 = kOffB1 + kMlpHid;
constexpr int kOffB2 = kOffW2 + kMlpHid * kMlpHid;
constexpr int kOffW3 = kOffB2 + kMlpHid;
constexpr int kOffB3 = kOffW3 + kMlpHid * kMlpOut;
constexpr int kMlpParams = kOffB3 + kMlpOut;

struct MlpState {
    int max_rows;
    int loaded;
    int step;
    float* w;        // FP32 master parameters
    float* am;       // AdamW moments
    float* av;
    uint16_t* wbf;   // BF16 copy of w
    uint16_t* wt;    // BF16 weights transposed to [n][k] (inference)
    // training: transposed BF16 operands of the weight gradients, [rows / 32][feature][32]
    uint16_t* xt;    // inputs
    uint16_t* h1t;   // activations
    uint16_t* h2t;
    uint16_t* dyt;   // d loss / d outputs
    uint16_t* dz2t;  // d loss / d pre-activations
    uint16_t* dz1t;
    float* bias_part;    // per workgroup: column sums of the last three in FP32,
    double* loss_part;   // the loss
};

}  // namespace vrm
