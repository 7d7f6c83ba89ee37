// ndgp_corr.h -- the cell update of the mixed-precision solve's FP32 correction
// equation (derived at the head of ndgp_mixed.hip).  Not part of the public ABI.
#pragma once

#include "ndgp_device.h"

namespace ndgp {
namespace dev {

struct CorrTerms {
    float A;    // L[phi + e] - L[phi] at the cell
    float lapw; // lap of w = phi + e
    float seew; // sum over edges of (w_edge - w_centre)
};

__device__ __forceinline__ CorrTerms corr_terms(const float vp[19], const float ve[19], float al) {
    const float up = vp[0], ue = ve[0];
    const float pxp = vp[1] - up, pxm = vp[2] - up, pyp = vp[3] - up, pym = vp[4] - up;
    const float pzp = vp[5] - up, pzm = vp[6] - up;
    const float exp_ = ve[1] - ue, exm = ve[2] - ue, eyp = ve[3] - ue, eym = ve[4] - ue;
    const float ezp = ve[5] - ue, ezm = ve[6] - ue;
    const float Dpx = pxp + pxm, Dpy = pyp + pym, Dpz = pzp + pzm;
    const float Dex = exp_ + exm, Dey = eyp + eym, Dez = ezp + ezm;
    const float Dwx = Dpx + Dex, Dwy = Dpy + Dey, Dwz = Dpz + Dez;
    const float pair = fmaf(Dwx, Dey, Dex * Dpy) + fmaf(Dwx, Dez, Dex * Dpz) +
                       fmaf(Dwy, Dez, Dey * Dpz);
    // corner (s, t) of plane a-b: C = (v_st - v_s) - (v_t - v_centre), the
    // first difference exact for neighbouring values (Sterbenz), for phi and
    // for e; the sum of the corner differences of w is the edge sum less
    // 4 lap w (every face neighbour sits in four corners)
    float cs = 0.f, sw = 0.f;
    auto corner = [&](int q, int s_face, float pb, float eb) {
        const float Cp = (vp[q] - vp[s_face]) - pb, Ce = (ve[q] - ve[s_face]) - eb;
        const float Cw = Cp + Ce;
        sw += Cw;
        cs = fmaf(Cw + Cp, Ce, cs);
    };
    corner(7, 1, pyp, eyp);
    corner(8, 1, pym, eym);
    corner(9, 2, pyp, eyp);
    corner(10, 2, pym, eym);
    corner(11, 1, pzp, ezp);
    corner(12, 1, pzm, ezm);
    corner(13, 2, pzp, ezp);
    corner(14, 2, pzm, ezm);
    corner(15, 3, pzp, ezp);
    corner(16, 3, pzm, ezm);
    corner(17, 4, pzp, ezp);
    corner(18, 4, pzm, ezm);
    CorrTerms t;
    t.A = fmaf(2.f * al, pair - 0.25f * cs, (Dex + Dey) + Dez);
    t.lapw = (Dwx + Dwy) + Dwz;
    t.seew = fmaf(4.f, t.lapw, sw);
    return t;
}

// New correction at the cell: w times the way to the root of its own quadratic (same
// algebra and cases as relax_cell, with phi + e in place of phi), discriminant and root
// in FP64.
__device__ __forceinline__ float relax_corr_cell(const float vp[19], const float ve[19], float r,
                                                 float al, double w, unsigned &fallbacks) {
    const CorrTerms t = corr_terms(vp, ve, al);
    const double ad = (double)al;
    const double rT = (double)t.A - (double)r;
    const double B = fma(ad, fma(2.0, (double)t.lapw, 0.5 * (double)t.seew), 3.0);
    const double D = fma(B, B, -18.0 * ad * rT);
    if (D < 0.0) {
        ++fallbacks;
        return (float)fma(fmin(w, 1.0), B / (18.0 * ad), (double)ve[0]);
    }
    if (B > 0.0) return (float)fma(w * rT, fast_rcp(B + fast_sqrt(D)), (double)ve[0]);
    fallbacks += kPastVertexEvent;
    return (float)fma(fmin(w, 1.0), (B - fast_sqrt(D)) / (18.0 * ad), (double)ve[0]);
}

} // namespace dev
} // namespace ndgp
