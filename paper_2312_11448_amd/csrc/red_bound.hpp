// Per-box constants of the deposit-free end of an escaping packet's walk
// (red_core.hpp) and the bound on the walk's roundings that its count rests
// on. No device code: the host sets the constants up.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#ifdef __HIPCC__
#define MCLYA_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MCLYA_HOST_DEVICE inline
#endif

namespace mclya {

// A later deposit is at most w (cg exp(-xup^2) + cv / xup^2), xup the largest
// frequency still to come.
enum : int32_t { kRedOff = 0, kRedStill = 1, kRedFlow = 2 };   // not used, no flow, flow
struct alignas(64) RedBox {
    float cg, cv;
    float ub[3];          // <U>
    float udev;           // max |U_c - <U>|, rounded up
    float round_x;        // bound on the two binary32 roundings of x at one face, |x| <= x_eff
    float round_jump;     // ... on those of the jump's difference and of the segment's length
    float slack;          // roundings of the count itself: X and k.U at the flow's size
    float binade;         // largest power of two <= x_eff
    int32_t mode;
};
static_assert(sizeof(RedBox) == 64, "RedBox layout");

// The constants of red_only and red_count for a box with largest kappa kmax,
// drift delta, threshold x_eff and largest flow deviation udev from the mean
// flow u. The bounds: a segment is at most 1.75 cells long; the thermal
// profile at x is exp(-x^2)/sqrt(pi); the Voigt correction -(2a/pi) F'(x) is at
// most damp 0.85 / x^2 for |x| >= 1; 2 % for the binary32 evaluation. One
// face rounds x twice (the drift, the jump), by at most half an ulp of x_eff's
// binade each, and the jump's difference of projections once; a segment's
// length by 2^-24 of itself.
// With a flow, red_count's decisions are unsure within the sum of those
// roundings over the walk that is left, so it pays where that sum is well
// below a cell's drift: at most a quarter of delta (at delta = 0.019, the
// paper's cells, it is under 3 % of it, and some 2 % of the packets are
// unsure; below delta = 0.006 most would be).
inline RedBox red_constants(double kmax, double delta, double x_eff, const double u[3], double udev, bool vel,
                            double damp)
{
    RedBox r;
    std::memset(&r, 0, sizeof r);
    r.cg = (float)(std::max(kmax, 0.0) * delta * 1.75 * 0.5641895835477563 * 1.02);
    r.cv = (float)(std::max(kmax, 0.0) * delta * 1.75 * damp * 0.85 * 1.02);
    for (int a = 0; a < 3; ++a) r.ub[a] = (float)u[a];
    auto half_ulp = [](double v) { return std::ldexp(1.0, std::ilogb(std::max(v, 1e-30)) - 24); };
    // X = x + k.U and the projections k.<U> and k.U are as large as the flow:
    // a handful of roundings at that size
    const double moving = 8.0 * half_ulp(std::fabs(u[0]) + std::fabs(u[1]) + std::fabs(u[2]) + udev + x_eff);
    r.udev = (float)(udev * 1.0001 + std::max(1e-4, moving));
    r.slack = (float)std::max(2e-6, moving);
    r.round_x = (float)(1.02 * 2.0 * half_ulp(x_eff));
    r.round_jump = (float)(1.02 * (half_ulp(2.0 * udev + 1e-6) + delta * 1.75 * 0x1p-24));
    r.binade = (float)std::ldexp(1.0, std::ilogb(std::max(x_eff, 1e-30)));
    const bool still = !vel || (udev == 0.0 && u[0] == 0.0 && u[1] == 0.0 && u[2] == 0.0);
    const double most = 1.7321 * 2.0 * (x_eff + udev) / delta + 4.0;
    const double sum = ((double)r.round_x + (double)r.round_jump) * most + (double)r.slack;
    const bool fine = std::isfinite(r.cg) && std::isfinite(r.cv) && std::isfinite(x_eff) && delta > 0.0;
    r.mode = !fine ? kRedOff : still ? kRedStill : sum <= 0.25 * delta ? kRedFlow : kRedOff;
    return r;
}

// Bound on the sum of the stepping walk's roundings of x over a walk `far`
// cells long (at most sqrt 3 faces a cell and three more). While |x| is below
// the binade of x_eff in every cell, which the first `near` cells are, the
// roundings of x are half as large; those of the jump and of the length are not.
MCLYA_HOST_DEVICE float red_eps(const RedBox &R, float far, float near)
{
    const float faces = fmaf(1.7321f, far, 4.0f);
    return fmaf(R.round_x, fmaf(-0.86605f, fminf(near, far), faces), fmaf(R.round_jump, faces, R.slack));
}

}  // namespace mclya
