// Internal declarations of the surrogate kernels (sur_kernels.hip) used by the
// C ABI in sur_api.hip.  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace sur {

typedef __bf16 bf16;

hipError_t conv(const bf16* in, int cin, const bf16* w, const float* bias, const void* res, const bf16* mask,
                void* out, int out_f32, int relu_in, int dil, int N, int H, int W, hipStream_t s);
// Layers handled by one launch.
constexpr int kMaxLayers = 8;
struct AdjointLayers {
    int n;
    const bf16* w[kMaxLayers];
    bf16* wt[kMaxLayers];
    int cin[kMaxLayers];
};
hipError_t adjoint_weights(const AdjointLayers& L, hipStream_t s);
hipError_t wgrad(const bf16* dy, const bf16* in, int cin, int relu_in, int dil, int N, int H, int W, float* part,
                 int groups, float* out, hipStream_t s);
hipError_t bgrad(const bf16* dy, long long npix, float* part, int groups, float* out, hipStream_t s);
hipError_t adam(float* p, const float* g, float* m1, float* m2, bf16* pb, long long n, float lr, float b1, float b2,
                float eps, int t, hipStream_t s);
// Weight and bias gradients of a layer as `groups` partial sums (32 * 9 * cin
// weights, then 32 biases), every one of them written.
hipError_t layer_grads(const bf16* dy, const bf16* in, int cin, int relu_in, int dil, int N, int H, int W, float* part,
                       int groups, hipStream_t s);
struct AdamLayer {
    const float* part;
    float *W, *b, *mW1, *mW2, *mb1, *mb2;
    bf16* Wb;
    int cin, groups;
};
struct AdamLayers {
    int n, blocks[kMaxLayers];
    AdamLayer l[kMaxLayers];
};
constexpr int kLossParts = 512;  // partial sums of the squared error
// Adam on every layer from the partial sums of its gradients; loss = the sum of
// the kLossParts values of lpart.
hipError_t adam_layers(AdamLayers& L, float lr, float b1, float b2, float eps, int t, const float* lpart, float* loss,
                       hipStream_t s);
// The five FP32 state fields of a frame: phi, ux, uy, T, p.
struct State5 {
    const float* v[5];
};
// Scalings of a frame (mirrors sur_scales of the C ABI).
struct Scales {
    float u, dT, t_a, t_b, P, c4, c5;
    float inc[5];
};

hipError_t mse(const float* delta, const float* target, long long npix, int nout, float scale, bf16* grad,
               float* part, int groups, hipStream_t s);
hipError_t pack(const State5& f, long long npix, int w, const Scales& sc, bf16* x, hipStream_t s);
hipError_t pack_target(const State5& f0, const State5& f1, long long npix, const Scales& sc, float* t, hipStream_t s);
hipError_t advance(const float* delta, long long npix, const Scales& sc, const State5& f, hipStream_t s);
// The output layer (dilation <= 16) compared with the target of 5 channels:
// gradient as mse with nout = 5, partial sums of the squared error in lpart.
hipError_t conv_mse(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int N, int H, int W,
                    const float* target, float scale, bf16* grad, float* lpart, hipStream_t s);
// The first layer on one frame packed from its state as it is staged
// (dilation <= 16; bitwise pack followed by conv with cin = 8).
hipError_t conv_packed(const State5& f, const Scales& sc, const bf16* w, const float* bias, bf16* out, int dil, int H,
                       int W, hipStream_t s);
hipError_t conv_advance(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int H, int W,
                        const Scales& sc, const State5& f, hipStream_t s);
constexpr int kVolPartsApi = 512;  // partials of conv_advance_volume (the column kernel's kVolParts)
// conv_advance (dilation <= 16) that also sums the light-phase volume of the
// updated phi into *vout; vpart holds kVolParts partials and a zero counter.
hipError_t conv_advance_volume(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int H, int W,
                               const Scales& sc, const State5& f, double* vpart, double* vout, hipStream_t s);
hipError_t frame_sums(const State5& a, const State5* b, long long npix, int w, const Scales& sc, double* part,
                      int groups, double* out, hipStream_t s);

// Largest partial-sum count of the allocation-free judge, and the devices it
// keeps an address for.
constexpr int kJudgeMaxGroups = 1024;
constexpr int kMaxDevices = 64;
// Device address of the current device's judge scratch (kJudgeMaxGroups * 8
// doubles), looked up on the first call on each device.
hipError_t judge_scratch_ptr(double** out);

}  // namespace sur
