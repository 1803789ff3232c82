// How the persistent walk is launched, from its options and the packets. No
// device code.
#pragma once

#include <algorithm>
#include <cstdint>

namespace mclya {

// MC_LYA_OPT_BLOCK, _WAVES_PER_CU, _CHUNK and _QUEUES
struct WalkOptions {
    int block = 256, waves_per_cu = 32, chunk = 256, nqueues = 8;
    bool operator==(const WalkOptions &o) const
    {
        return block == o.block && waves_per_cu == o.waves_per_cu && chunk == o.chunk && nqueues == o.nqueues;
    }
};

struct WalkLaunch {
    bool box;             // a lone box's records in LDS (walk_box_kernel)
    int block, grid, chunk, nqueues;
};

// Where one of the options is set to something else than its default, all of
// them act as they are; at the defaults a lone box whose records fit the LDS
// (lone_fits) has a kernel of its own, and the chunk follows the packets.
// resident: workgroups a compute unit holds at once; waves_cap: at most this
// many waves a compute unit (0: the option's).
inline WalkLaunch plan_persistent(const WalkOptions &o, uint64_t count, int num_cu, int resident, int waves_cap,
                                  bool lone_fits)
{
    const bool free = o == WalkOptions{};
    const uint64_t need = (count + 63) / 64;             // waves, with a packet a lane
    WalkLaunch l;
    l.box = free && lone_fits;
    if (l.box) {
        const int per = (int)std::min<uint64_t>(16, (need + num_cu - 1) / num_cu);
        l.block = 64 * per;
        l.grid = (int)std::min<uint64_t>((uint64_t)num_cu, (need + per - 1) / per);
        l.chunk = 64;
        l.nqueues = 1;
        return l;
    }
    const int waves_per_block = o.block / 64;
    const int waves = waves_cap > 0 ? std::min(o.waves_per_cu, waves_cap) : o.waves_per_cu;
    // never more workgroups than can be resident at once, nor waves than packets
    l.block = o.block;
    l.grid = num_cu * std::max(1, std::min(waves / waves_per_block, resident));
    if ((uint64_t)l.grid * waves_per_block > need)
        l.grid = (int)std::max<uint64_t>(1, (need + waves_per_block - 1) / waves_per_block);
    // Few packets: a chunk for each of four waves a compute unit, one per
    // SIMD (whole chunks would leave most of the chip without; one for
    // every resident wave leaves none to refill the lanes that finish
    // first), from 128 packets a chunk on for each of eight. Transports with
    // 256 a chunk, with one for all 3072 waves, with this, us: 28 518 packets
    // (23^3, flow) 632, 416, 416; 62 046 (Voigt, flow) 970, 785, 783; 139 172
    // (30^3, Voigt, flow) 683, 751, 708; 156 927 (Voigt, flow) 616, 712, 626;
    // 262 296 (four of 40^3) 2165, 1700, 1864; from 524 288 on 256.
    const uint64_t per4 = count / (4 * (uint64_t)num_cu), per8 = per4 / 2;
    const uint64_t each = std::max({(uint64_t)64, std::min<uint64_t>(per4, 128), per8});
    l.chunk = free ? (int)std::min<uint64_t>((uint64_t)o.chunk, each) : o.chunk;
    l.nqueues = o.nqueues;
    return l;
}

}  // namespace mclya
