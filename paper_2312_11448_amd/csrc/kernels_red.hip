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
constexpr uint32_t kRedChunk = 1024;     // packets of a workgroup's turn

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

// Each workgroup takes chunks of the list. The packets that red_count gives
// back (a few per cent) are collected and stepped together afterwards, so that
// one of them does not hold a wave of others.
template <bool VEL, bool VOIGT>
__global__ __launch_bounds__(kRedBlock) void red_list_kernel(RedParams P)
{
    __shared__ uint32_t s_unsure[kRedChunk];
    __shared__ uint32_t s_n;
    const uint64_t n = P.counters[kRedCountSlot], done = P.counters[kRedDoneSlot];
    Acc acc{-1, 0, 0, 0, 0, 0};
    // one packet of the list (or none: i >= n); second = stepped
    auto take = [&](bool have, uint64_t i, bool second) {
        PState o;
        int box = acc.box;
        if (have) {
            o = P.state[i];
            box = P.n_boxes == 1 ? 0 : box_of_cell(P.boxes, P.n_boxes, o.pos);
        }
        const bool change = have && box != acc.box;
        if (__ballot(change && acc.box >= 0)) flush(acc, change, P.tot);
        if (!have) return;
        acc.box = box;
        const WalkBox B = P.boxes[box];
        const RedBox R = P.red[box];
        const Line ln = line_of(B);
        Lane L;
        load_red(L, o, B);
        RedEnd e;
        if (!VEL || R.mode == kRedStill) {
            e = red_exact<false, VOIGT>(L, P.rec, P.max_cross, ln);
        } else if (!second) {
            e = red_count<VOIGT>(L, R, P.rec, P.max_cross, ln);
            if (e.fate == kUnsure) {
                s_unsure[atomicAdd(&s_n, 1u)] = (uint32_t)(i - done);
                return;
            }
        } else {
            finish_entry<true>(L, load_rec<true>(P.rec, L.c));
            e = red_exact<true, VOIGT>(L, P.rec, P.max_cross, ln);
        }
        acc.cross += e.n;
        acc.esc += e.fate == kEscaped ? L.w : 0u;
        acc.capn += e.fate == kCapped ? 1u : 0u;
        acc.capw += e.fate == kCapped ? L.w : 0u;
        acc.wing += e.wing;
    };
    for (uint64_t base = done + (uint64_t)blockIdx.x * kRedChunk; base < n; base += (uint64_t)gridDim.x * kRedChunk) {
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < kRedChunk; k += kRedBlock) take(base + k < n, base + k, false);
        if (VEL) {
            __syncthreads();
            const uint32_t m = s_n;
            for (uint32_t k0 = 0; k0 < m; k0 += kRedBlock) {
                const uint32_t k = k0 + threadIdx.x;
                take(k < m, k < m ? done + s_unsure[k] : 0, true);
            }
        }
        __syncthreads();
    }
    flush(acc, true, P.tot);
}

__global__ void red_mark_kernel(unsigned long long *counters)
{
    counters[kRedDoneSlot] = counters[kRedCountSlot];
}

}  // namespace

hipError_t launch_red_list(const RedParams &p, int grid, bool vel, bool voigt, hipStream_t s)
{
    const dim3 g((unsigned)grid), b(kRedBlock);
    if (voigt) {
        if (vel) hipLaunchKernelGGL((red_list_kernel<true, true>), g, b, 0, s, p);
        else hipLaunchKernelGGL((red_list_kernel<false, true>), g, b, 0, s, p);
    } else {
        if (vel) hipLaunchKernelGGL((red_list_kernel<true, false>), g, b, 0, s, p);
        else hipLaunchKernelGGL((red_list_kernel<false, false>), g, b, 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_red_mark(unsigned long long *counters, hipStream_t s)
{
    hipLaunchKernelGGL(red_mark_kernel, dim3(1), dim3(1), 0, s, counters);
    return hipGetLastError();
}

}  // namespace mclya
