"""The batch launch's LDS: a plan that the host accepts must fit a workgroup,
the kernel's static LDS included.  The host's rule and frame sizes are compiled
here with the system compiler; nothing is launched."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1403_4560_amd", "csrc")
LDS = 160 << 10  # bytes of a gfx950 workgroup
PROGRAM = r"""
#define __host__
#define __device__
#include "ea_types.hpp"
#include <cstdio>
using namespace ea;
int main()
{
    for (int jk = 0; jk < 2; ++jk)
        for (int L = 2; L <= LDS_MAX_L; L += 2)
            for (int nT = 1; nT <= MAX_T; ++nT)
                for (int group = 0; group < 2; ++group)
                    for (int P = 1; P <= 8; P *= 2) {
                        const size_t lds = !group ? lds_offsets(L, nT, jk, jk == 0 && L == 8).total
                                           : jk   ? group_bits_lds_offsets(L, nT).total
                                                  : group_lds_offsets(L, nT).total;
                        std::printf("%d %d %d %d %d %zu %d %zu\n", jk, L, nT, group, P, lds,
                                    (int)batch_teams_fit(P, 64, lds, jk, 160 << 10), SPREAD_BYTES);
                    }
}
"""


def test_accepted_plans_fit_a_workgroup(tmp_path):
    src, exe = tmp_path / "fit.cpp", tmp_path / "fit"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    rows = [tuple(int(x) for x in line.split()) for line in subprocess.check_output([str(exe)], text=True).splitlines()]
    assert len(rows) == 2 * 8 * 64 * 2 * 4
    accepted = 0
    for jk, L, nT, group, P, lds, ok, static in rows:
        need = P * (-(-lds // 16) * 16) + (static if jk else 0)
        assert ok == (need <= LDS), (jk, L, nT, group, P)
        accepted += ok
    assert 0 < accepted < len(rows)
    # eight frames alone fit here, with the spreading tables they do not
    edge = {(nT, P): (8 * lds <= LDS, ok) for jk, L, nT, group, P, lds, ok, _ in rows if jk and group and L == 8}
    assert all(edge[nT, 8] == (True, 0) and edge[nT, 4][1] for nT in (21, 22, 23, 24))
