"""The split of short-block attention over workgroups (csrc/attn_plan.h), compiled for the host: batches whose contexts differ are split by
the work there is, so that no workgroup is left walking a long context while the other CUs are idle."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2604_05417_amd", "csrc")
N_CU = 256
SRC = '''#include "attn_plan.h"
extern "C" void plan(const int* len, int nseg, int H, int KH, int hd, int m, int n_cu, int force, int* o) {
    const msd::AttnPlan p = msd::plan_attn(len, nseg, H, KH, hd, m, n_cu, force);
    o[0] = p.hp; o[1] = p.spw; o[2] = p.nrec; o[3] = p.grid;
    for (int s = 0; s <= nseg; ++s) o[4 + s] = p.items.first[s];
}'''


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "p.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "p.so"), str(d / "p.cpp")], check=True)
    f = C.CDLL(str(d / "p.so")).plan

    def call(lens, H, KH, hd, m, force=0):
        o = (C.c_int * 40)()
        f((C.c_int * len(lens))(*lens), len(lens), H, KH, hd, m, N_CU, force, o)
        return dict(hp=o[0], spw=o[1], nrec=o[2], grid=o[3], first=list(o[4: 5 + len(lens)]), subs=[(n + 31) // 32 for n in lens])
    return call


SHAPES = [(32, 32, 128), (32, 8, 64), (12, 12, 64)]
MIXES = [[8000] + [64] * 31, [8000] * 4 + [64] * 28, [8000] + [64] * 7, [8000, 64, 64], [64 + 256 * i for i in range(32)], [4000] * 16 + [64] * 16,
         [32000] + [64] * 31, [1000 * (i + 1) for i in range(8)], [2048] * 32, [2048 - 60 * i for i in range(8)], [333, 330, 327], [16] * 32, [8000]]


@pytest.mark.parametrize("H,KH,hd", SHAPES)
@pytest.mark.parametrize("m", [1, 2, 8, 16])
@pytest.mark.parametrize("i", range(len(MIXES)))
def test_span_of_a_workgroup_follows_the_work(plan, H, KH, hd, m, i):
    lens = MIXES[i]
    p = plan(lens, H, KH, hd, m)
    assert (H // KH) % p["hp"] == 0 and (p["hp"] == 1 or p["hp"] * m <= 16)
    assert p["spw"] % 4 == 0 and p["nrec"] == -(-max(p["subs"]) // p["spw"])
    # items without gaps: a sequence of k records has k per K/V head
    assert p["first"][0] == 0 and [b - a for a, b in zip(p["first"], p["first"][1:])] == [KH * -(-n // p["spw"]) for n in p["subs"]]
    assert 0 <= p["grid"] // (H // KH // p["hp"]) - p["first"][-1] < 8
    # The longest walk of a workgroup: no more than twice an even share of the work for every CU, or what the longest context alone would be
    # split into, or 128 KiB of K and V (a context that is not worth splitting), or what a CU by itself walks (35 GB/s) while the full chip
    # (25 GB/s per CU) goes through everything and merges (5.5 us).
    share = sum(p["subs"]) * (H // p["hp"]) / N_CU
    alone = plan([max(lens)], H, KH, hd, m)["spw"]
    walk, kib = min(p["spw"], max(p["subs"])), 32 * hd * 4 / 1024
    assert walk <= max(2 * share, alone, 128 / kib) or walk * kib / 34.2 <= share * kib / 24.4 + 5.5, (walk, share, alone)
    # records are merged at a cost that grows with them: never more than the merge reads at once
    assert p["nrec"] <= 16
