// The red list of a tiled batch: packets whose remaining deposits all round to
// zero (red_core.hpp), written out by the tiles and the tail walk and counted
// to their escape here, one per thread.
//
// What bounds it: with a flow, the cells looked at one by one before the
// escape (about 20 a packet at the paper's cell size, a 16-byte record each
// from a random place); without one, the arithmetic of the face steps. It
// replaces some 200 full steps a packet, at 58 % of the lanes, in the tiles.
#include "red_core.hpp"

namespace mclya {
namespace {

constexpr int kRedBlock = 256;

// Box of a global cell (boxes sorted by cell offset).
__device__ __forceinline__ int box_of_cell(const WalkBox *boxes, int n_boxes, uint32_t c)
{
    int lo = 0, hi = n_boxes - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (boxes[mid].cell_off <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ void load_red(Lane &L, const PState &o, const WalkBox &B)
{
    load_state(L, o, B);
    const uint32_t local = o.pos - B.cell_off;
    const uint32_t rest = local / (uint32_t)B.nx;
    L.ix = (int32_t)(local - rest * (uint32_t)B.nx);
    L.iz = (int32_t)(rest / (uint32_t)B.ny);
    L.iy = (int32_t)(rest - (uint32_t)L.iz * (uint32_t)B.ny);
    L.c = o.pos;
}

// The packets that red_count gives back (a few per cent) go to a list of
// their own and are stepped by a second launch (STEP), so that one of them
// does not hold a wave of others.
template <bool VEL, bool VOIGT, bool STEP>
__global__ __launch_bounds__(kRedBlock) void red_list_kernel(RedParams P)
{
    const uint64_t done = STEP ? 0 : P.counters[kRedDoneSlot];
    const uint64_t n = STEP ? P.counters[kRedUnsureSlot] : P.counters[kRedCountSlot];
    Acc acc{-1, 0, 0, 0, 0, 0};
    const uint64_t stride = (uint64_t)gridDim.x * kRedBlock;
    for (uint64_t base = done + (uint64_t)blockIdx.x * kRedBlock; base < n; base += stride) {
        uint64_t i = base + threadIdx.x;
        const bool have = i < n;
        PState o;
        int box = acc.box;
        if (have) {
            if (STEP) i = P.unsure[i];
            o = P.state[i];
            box = P.n_boxes == 1 ? 0 : box_of_cell(P.boxes, P.n_boxes, o.pos);
        }
        const bool change = have && box != acc.box;
        if (__ballot(change && acc.box >= 0)) flush(acc, change, P.tot);
        bool unsure = false;
        if (have) {
            acc.box = box;
            const WalkBox B = P.boxes[box];
            const RedBox R = P.red[box];
            const Line ln = line_of(B);
            Lane L;
            load_red(L, o, B);
            RedEnd e;
            if (STEP) {
                finish_entry<true>(L, load_rec<true>(P.rec, L.c));
                e = red_exact<true, VOIGT>(L, P.rec, P.max_cross, ln);
            } else if (!VEL || R.mode == kRedStill) {
                e = red_exact<false, VOIGT>(L, P.rec, P.max_cross, ln);
            } else {
                e = red_count<VOIGT>(L, R, P.rec, P.max_cross, ln);
                unsure = e.fate == kUnsure;
            }
            if (!unsure) {
                acc.cross += e.n;
#ifdef MCLYA_COUNT_ENDS
                // (build.py --count-ends, for bench.py --count-ends: the
                // crossings counted here, in the total that tally returns as
                // scatterings)
                atomicAdd(&P.tot[box].pad[0], (unsigned long long)e.n);
#endif
                acc.esc += e.fate == kEscaped ? L.w : 0u;
                acc.capn += e.fate == kCapped ? 1u : 0u;
                acc.capw += e.fate == kCapped ? L.w : 0u;
                acc.wing += e.wing;
            }
        }
        if (VEL && !STEP) {
            const uint64_t m = __ballot(unsure);
            if (m) {
                unsigned long long at = 0;
                if (__lane_id() == (uint32_t)(__ffsll((unsigned long long)m) - 1))
                    at = atomicAdd(&P.counters[kRedUnsureSlot], (unsigned long long)__popcll(m));
                at = __shfl(at, __ffsll((unsigned long long)m) - 1, 64);
                if (unsure)
                    P.unsure[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = (uint32_t)i;
            }
        }
    }
    flush(acc, true, P.tot);
}

__global__ void red_mark_kernel(unsigned long long *counters)
{
    counters[kRedDoneSlot] = counters[kRedCountSlot];
    counters[kRedUnsureSlot] = 0;
}

template <bool VOIGT>
hipError_t launch(const RedParams &p, dim3 g, bool vel, hipStream_t s)
{
    const dim3 b(kRedBlock);
    if (!vel) {
        hipLaunchKernelGGL((red_list_kernel<false, VOIGT, false>), g, b, 0, s, p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((red_list_kernel<true, VOIGT, false>), g, b, 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((red_list_kernel<true, VOIGT, true>), g, b, 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_red_list(const RedParams &p, int grid, bool vel, bool voigt, hipStream_t s)
{
    return voigt ? launch<true>(p, dim3((unsigned)grid), vel, s) : launch<false>(p, dim3((unsigned)grid), vel, s);
}

hipError_t launch_red_mark(unsigned long long *counters, hipStream_t s)
{
    hipLaunchKernelGGL(red_mark_kernel, dim3(1), dim3(1), 0, s, counters);
    return hipGetLastError();
}

}  // namespace mclya
