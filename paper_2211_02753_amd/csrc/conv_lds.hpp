// 3x3 convolutions between 32 and 64 channels, a band of rows at a time in
// LDS.  Each function launches its pass and returns true, or returns false
// when the layer's rows do not fit its LDS buffer (wide images).  Tensors as
// in the C interface; every pointer 16-byte aligned.
#pragma once

#include "common.hpp"

namespace tdp {

bool conv_fwd_32_64(const uint16_t* x, const uint16_t* w, const float* bias, int B, int H, int W, int relu,
                    uint16_t* y, hipStream_t s);
bool conv_dgrad_64_32(const uint16_t* dy, const uint16_t* w, const uint16_t* mask, int B, int H, int W, uint16_t* dx,
                      hipStream_t s);
// Adds to dw and db (float32, cleared by the caller; db may be null).
bool conv_wgrad_32_64(const uint16_t* x, const uint16_t* dy, int B, int H, int W, float* dw, float* db, hipStream_t s);

}  // namespace tdp
