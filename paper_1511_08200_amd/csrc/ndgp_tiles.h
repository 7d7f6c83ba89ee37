// ndgp_tiles.h -- what the one-launch levels (ndgp_tiles.hip) need to know of the
// field they relax.  Not part of the public ABI.
#pragma once

#include "ndgp_corr.h"

namespace ndgp {

template <int V>
struct Int {
    static constexpr int value = V;
};

// the FP64 field itself
struct TileField {
    using T = double;
    using Pair = double2;
    static constexpr bool two = false;
    __device__ __forceinline__ static double fma_(double a, double b, double c) {
        return fma(a, b, c);
    }
    __device__ __forceinline__ static double relax(const double v[19], const double *, double s,
                                                   double al, double w, unsigned &ev) {
        return dev::relax_cell(v, s, al, w, ev);
    }
    __device__ __forceinline__ static double apply(const double v[19], const double *, double al) {
        return dev::apply_L(dev::stencil_terms(v), al);
    }
};

// the FP32 correction of the mixed-precision solve, about a static FP32 field
struct TileCorrection {
    using T = float;
    using Pair = float2;
    static constexpr bool two = true;
    __device__ __forceinline__ static float fma_(float a, float b, float c) {
        return fmaf(a, b, c);
    }
    __device__ __forceinline__ static float relax(const float v[19], const float vb[19], float r,
                                                  float al, double w, unsigned &ev) {
        return dev::relax_corr_cell(vb, v, r, al, w, ev);
    }
    __device__ __forceinline__ static float apply(const float v[19], const float vb[19], float al) {
        return dev::corr_terms(vb, v, al).A;
    }
};

} // namespace ndgp
