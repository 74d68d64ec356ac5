// Launchers of the learned-preconditioner kernels (cnn.hip).  Rows: row = cb * Ns + s, 32 channels; the order of the
// bf16 arrays (rows, sites, weights) in memory is described there.
#pragma once
#include "eofa_int.h"

namespace eofa {

// 4 layers; layer l maps CNN_CIN[l] -> CNN_COUT[l] live channels (padded to 32)
constexpr int CNN_LAYERS = 4;
constexpr int CNN_CIN[CNN_LAYERS] = {24, 32, 32, 32};
constexpr int CNN_COUT[CNN_LAYERS] = {32, 32, 32, 24};
constexpr int CNN_WSZ = 81 * 32 * 32;         // weights per layer (padded), [tap][n][k]
constexpr int CNN_LSZ = CNN_WSZ + 32;         // + bias
constexpr int CNN_NPARAM = CNN_LAYERS * CNN_LSZ;

hipError_t cnn_conv_fwd(const unsigned short* X, const unsigned short* W, const float* bias, void* Y, bool out_f32,
                        const Geom& g, int Ns, int relu, hipStream_t st);
// XT, dYT: bf16 sites; part: cnn_wgrad_chunks x 81 x 1024 floats
int cnn_wgrad_chunks(const Geom& g, int Ns);
hipError_t cnn_wgrad(const unsigned short* dYT, const unsigned short* XT, float* part, float* gw, const Geom& g, int Ns,
                     int cin, int cout, hipStream_t st);
// of the rows' output gradient dY (times act > 0 when act is given): BF16 rows (rows_out may be null), the
// copy in site order and the bias gradient gb; part: scratch of CNN_PREP_PART doubles
constexpr int CNN_PREP_PART = 1024 * 32;
hipError_t cnn_dy_prep(const float* dY, const unsigned short* act, unsigned short* rows_out, unsigned short* dYT,
                       double* part, float* gb, int cout, int rows, int Ns, hipStream_t st);
hipError_t cnn_rows_to_site(const unsigned short* in, unsigned short* out, int rows, int Ns, hipStream_t st);
// bf16 weights of a layer for the forward (wb) and the backward-data convolution (wt)
hipError_t cnn_w_pack(const float* w, unsigned short* wb, unsigned short* wt, hipStream_t st);
hipError_t cnn_adam(float* p, const float* g, float* m, float* v, size_t n, float lr, float b1, float b2, float eps,
                    float c1, float c2, float gscale, hipStream_t st);
hipError_t cnn_half_to_rows(const cd* h, unsigned short* X, const Geom& g, int Ns, const double* scale, int inv,
                            hipStream_t st);
hipError_t cnn_half_to_rows_f32(const cd* h, float* T, const Geom& g, int Ns, const double* scale, hipStream_t st);
hipError_t cnn_rows_to_half(const float* Y, cd* h, const Geom& g, int Ns, const double* scale, hipStream_t st);
hipError_t cnn_mse(const float* Y, const float* T, float* dY, size_t n, float w, const Red& red, hipStream_t st);

}  // namespace eofa
