// The end of an escaping packet's walk. Once a packet has drifted so far into
// the red wing that no cell of its box can take a unit of its weight, the rest
// of its walk only counts cells until it passes -x_eff: no deposit, no
// opacity, no change of weight. About 40 % of all crossings are of this kind
// (a packet emitted red of the core walks some 200 cells more with a residue
// of its weight), so they are not stepped through:
//   - without a flow the frequency falls steadily and only the ray's geometry
//     is needed (red_exact<false>: no records, no profile);
//   - with a flow the comoving frequency X = x + k.U falls steadily, the gas
//     frequency of a cell is X - k.U, and |k.(U - <U>)| <= udev in every cell.
//     So no cell that the ray leaves while X - k.<U> - udev > -x_eff can end
//     the walk, and the faces crossed up to there are counted from the ray
//     alone (red_count); the few cells after it are looked at one by one.
// The count is the integer the stepping walk arrives at. That walk rounds x in
// binary32 at every face, so red_count carries a bound on the sum of those
// roundings and gives a packet back (kUnsure) when a decision is closer than
// it, or when two faces are too close to order; such a packet is stepped with
// the walk's own rounding (red_exact<true>), as is one that could reach the
// crossing cap.
#pragma once

#include "walk_core.hpp"

namespace mclya {

// Whether every later deposit of a packet rounds to zero. A segment through a
// cell sweeps at most delta * 1.75 (RedBox) at a density no larger than the
// profile at xup = X - k.<U> + udev, the largest frequency any later cell can
// show it (the profile rises towards the core, so for xup < -1 its value there
// bounds them all); w times the resulting depth below 0.48 rounds to 0 in
// absorbed_share. The bound's constants hold 2 % for the binary32 evaluation
// of the profile.
__device__ __forceinline__ bool red_only(const RedBox &R, float x, float ku, float kx, float ky, float kz, uint32_t w)
{
    const float xup = x + ku - fmaf(kx, R.ub[0], fmaf(ky, R.ub[1], kz * R.ub[2])) + R.udev;
    const float x2 = xup * xup;
    const float depth = fmaf(R.cg, __expf(-x2), R.cv * __builtin_amdgcn_rcpf(x2));
    return R.mode != kRedOff && xup < -1.0f && (float)w * depth < 0.48f;
}

// How a packet's walk ends, and the crossings it made getting there.
struct RedEnd {
    uint32_t n;
    int fate;            // kEscaped, kCapped, or kUnsure
    uint32_t wing;       // Voigt: the far wing's share of its weight
};
enum : int { kUnsure = 5 };

// Coordinate i moved by one cell, or by n (periodic).
__device__ __forceinline__ int32_t moved(int32_t i, int32_t cells, bool up)
{
    const int32_t j = i + (up ? 1 : -1);
    return j == cells ? 0 : (j < 0 ? cells - 1 : j);
}

__device__ __forceinline__ int32_t moved_by(int32_t i, uint32_t n, int32_t cells, bool up)
{
    const int32_t m = (int32_t)(n % (uint32_t)cells);
    const int32_t j = up ? i + m : i - m;
    return j >= cells ? j - cells : (j < 0 ? j + cells : j);
}

// The rest of the walk of a packet standing inside its cell, face by face,
// with the roundings of the walk (segment, finish_entry) but no deposits. The
// ray's faces do not depend on the cells, so with a flow they are taken
// kAhead at a time and their cells' records read together.
template <bool FLOW, bool VOIGT>
__device__ __forceinline__ RedEnd red_exact(Lane &L, const void *__restrict__ rec, uint32_t max_cross, const Line &ln)
{
    constexpr int kAhead = FLOW ? 8 : 1;
    RedEnd e{0u, kEscaped, 0u};
    float stop = -L.xeff;
    bool done = false;
    while (!done) {
        float s[kAhead];
        Rec r[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const Face f = next_face(L.tmx, L.tmy, L.tmz);
            s[j] = (float)(f.tn - L.t);
            L.t = f.tn;
            L.tmx = f.bx ? L.tmx + L.tdx : L.tmx;
            L.tmy = f.by ? L.tmy + L.tdy : L.tmy;
            L.tmz = f.bz ? L.tmz + L.tdz : L.tmz;
            if (FLOW) {
                L.ix = f.bx ? moved(L.ix, L.nx, L.kx > 0.0f) : L.ix;
                L.iy = f.by ? moved(L.iy, L.ny, L.ky > 0.0f) : L.iy;
                L.iz = f.bz ? moved(L.iz, L.nz, L.kz > 0.0f) : L.iz;
                r[j] = load_rec<true>(rec, cell_of(L));
            }
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (done) break;
            if (L.x <= -L.xeff) {
                stop = L.x;
                done = true;
                break;
            }
            if (L.ncross + e.n >= max_cross) {
                e.fate = kCapped;
                return e;
            }
            const float xo = fmaf(-L.delta, s[j], L.x);
            ++e.n;
            L.x = xo;
            if (xo <= -L.xeff) {
                done = true;
                break;
            }
            if (FLOW) finish_entry<true>(L, r[j]);
        }
    }
    if (VOIGT) e.wing = wing_share(L.w, stop, ln);
    return e;
}

// The same with a flow, without the steps in between: L as red_exact takes it
// (its x may still be the frequency before the jump into its cell, with ku of
// the cell it left: only their sum is used). Works on its own copy of the
// geometry.
template <bool VOIGT>
__device__ __forceinline__ RedEnd red_count(const Lane &L, const RedBox &R, const void *__restrict__ rec,
                                            uint32_t max_cross, const Line &ln)
{
    constexpr double kTie = 1e-9;        // faces closer than this are not ordered here
    RedEnd e{0u, kUnsure, 0u};
    const double X = (double)L.x + (double)L.ku;
    const float kub = fmaf(L.kx, R.ub[0], fmaf(L.ky, R.ub[1], L.kz * R.ub[2]));
    const double rd = 1.0 / (double)L.delta;
    const double t0 = L.t;
    // crossings left at most (every ray crosses at most sqrt 3 faces per unit
    // length), and with them the bound on the sum of the walk's roundings
    const double xc = X - (double)kub;
    const float far = fmaxf((float)((xc + (double)R.udev + (double)L.xeff) * rd), 0.0f);
    const float near = fmaxf((float)((xc - (double)R.udev + (double)R.binade) * rd), 0.0f);
    const float most = fmaf(1.7321f, far, 4.0f);
    const float eps = red_eps(R, far, near);
    const double safe = t0 + (xc - (double)R.udev + (double)L.xeff - 2.0 * (double)eps) * rd;
    double tmx = L.tmx, tmy = L.tmy, tmz = L.tmz, t = t0;
    int32_t ix = L.ix, iy = L.iy, iz = L.iz;
    bool unsure = false;
    // along each axis, the faces at or before `safe`
    auto skip = [&](double &tm, double td, int32_t &i, int32_t cells, bool up) {
        if (tm <= safe) {
            const double j = floor((safe - tm) / td);
            const double last = fma(j, td, tm);
            tm = last + td;
            unsure |= safe - last < kTie || tm - safe < kTie;
            t = fmax(t, last);
            const uint32_t n = (uint32_t)j + 1u;
            e.n += n;
            i = moved_by(i, n, cells, up);
        }
    };
    skip(tmx, L.tdx, ix, L.nx, L.kx > 0.0f);
    skip(tmy, L.tdy, iy, L.ny, L.ky > 0.0f);
    skip(tmz, L.tdz, iz, L.nz, L.kz > 0.0f);
    if (unsure) return e;
    const uint32_t limit = e.n + (uint32_t)most + 4u;
    auto read = [&]() {
        return load_rec<true>(rec, L.coff + (uint32_t)ix + (uint32_t)L.nx * ((uint32_t)iy + (uint32_t)L.ny * (uint32_t)iz));
    };
    // then cell by cell, kAhead cells' records read together
    constexpr int kAhead = 4;
    bool done = false, jumped = false;
    float stop = -L.xeff;
    Rec r = read();
    while (!done) {
        Rec nr[kAhead];
        float in[kAhead], out[kAhead];       // X + x_eff on entering and leaving the cell
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const Face f = next_face(tmx, tmy, tmz);
            unsure |= fmin(f.bx ? tmy : tmx, f.bz ? tmy : tmz) - f.tn < kTie;
            in[j] = (float)fma(-(double)L.delta, t - t0, X);
            out[j] = (float)fma(-(double)L.delta, f.tn - t0, X);
            t = f.tn;
            tmx = f.bx ? tmx + L.tdx : tmx;
            tmy = f.by ? tmy + L.tdy : tmy;
            tmz = f.bz ? tmz + L.tdz : tmz;
            ix = f.bx ? moved(ix, L.nx, L.kx > 0.0f) : ix;
            iy = f.by ? moved(iy, L.ny, L.ky > 0.0f) : iy;
            iz = f.bz ? moved(iz, L.nz, L.kz > 0.0f) : iz;
            nr[j] = read();
        }
        if (unsure || e.n > limit) return e;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (done) break;
            const float ku = ray_velocity(L.kx, L.ky, L.kz, r);
            r = nr[j];
            const float xi = in[j] - ku + L.xeff, xo = out[j] - ku + L.xeff;
            if (fabsf(xi) <= eps) return e;
            if (xi < 0.0f) {                 // redshifted out by the jump into this cell
                stop = xi - L.xeff;
                jumped = true;
                done = true;
                break;
            }
            ++e.n;
            if (fabsf(xo) <= eps) return e;
            if (xo < 0.0f) {                 // escapes inside this cell
                done = true;
                break;
            }
        }
    }
    if (VOIGT) {
        e.wing = wing_share(L.w, stop, ln);
        if (jumped) {
            // the stopping frequency is known to eps: the wing's share has to
            // be the same over that range
            const float d = eps + 1e-4f;
            if (wing_share(L.w, stop - d, ln) != e.wing || wing_share(L.w, stop + d, ln) != e.wing) return e;
        }
    }
    // (the cap is the stepping walk's to decide)
    if (e.n <= max_cross && L.ncross <= max_cross - e.n) e.fate = kEscaped;
    return e;
}

}  // namespace mclya
