"""The persistent walk's launch, from its options and the packets (CPU): an
option that is set acts as it is, also for a lone box whose records fit the
LDS; at the defaults every packet has a lane, no chunk is empty and no launch
is larger than the chip.
"""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "walk_plan.hpp"
extern "C" void plan(int block, int waves, int chunk, int queues, unsigned long long count, int resident, int cap,
                     int lone, int *out)
{
    const mclya::WalkOptions o{block, waves, chunk, queues};
    const mclya::WalkLaunch l = mclya::plan_persistent(o, count, 256, resident, cap, lone != 0);
    out[0] = l.box;
    out[1] = l.block;
    out[2] = l.grid;
    out[3] = l.chunk;
    out[4] = l.nqueues;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    lib = d / "plan.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2312_11448_amd", "csrc"), "-o", str(lib), str(d / "plan.cpp")], check=True)
    f = C.CDLL(str(lib)).plan

    def call(block, waves, chunk, queues, count, resident=3, cap=0, lone=0):
        out = (C.c_int * 5)()
        f(block, waves, chunk, queues, C.c_ulonglong(count), resident, cap, lone, out)
        return dict(zip(("box", "block", "grid", "chunk", "queues"), out))
    return call


@pytest.mark.parametrize("lone", [0, 1])
@pytest.mark.parametrize("count", [1, 5_000, 100_000, 3_000_000])
@pytest.mark.parametrize("opts", [(64, 32, 256, 8), (256, 8, 256, 8), (256, 32, 7, 8), (256, 32, 4096, 8),
                                  (256, 32, 256, 1)])
def test_a_set_option_acts(plan, opts, count, lone):
    block, waves, chunk, queues = opts
    l = plan(*opts, count, resident=8, lone=lone)
    assert not l["box"] and l["block"] == block and l["chunk"] == chunk and l["queues"] == queues
    assert l["grid"] * block // 64 <= max(256 * waves, block // 64)


@pytest.mark.parametrize("lone", [0, 1])
@pytest.mark.parametrize("cap", [0, 4])
@pytest.mark.parametrize("count", [1, 63, 64, 65, 16_384, 16_385, 65_537, 262_143, 262_144, 10 ** 7, 1 << 40])
def test_the_defaults_follow_the_packets(plan, count, cap, lone):
    l = plan(256, 32, 256, 8, count, cap=cap, lone=lone)
    waves = l["grid"] * l["block"] // 64
    assert l["box"] == lone and 1 <= l["grid"] and 64 <= l["block"] <= 1024
    assert waves <= (16 if lone else (cap or 12)) * 256
    assert 64 <= l["chunk"] <= 256
    assert waves <= max((count + 63) // 64 + l["block"] // 64 - 1, 1)     # no workgroup without packets
    if lone:
        assert l["chunk"] == 64 and l["queues"] == 1
    else:
        assert l["queues"] == 8 and (l["chunk"] == 256) == (count >= 524_288)
