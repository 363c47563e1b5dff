"""How the gradient products of an update are cut and launched, from the header that decides it (no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CUS, GIB = 256, 1 << 30


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """(n_sel, rows, d, V, bytes for partial sums) -> (slices, vocabulary blocks of a slice, whether dW has a launch of its own)."""
    at = tmp_path_factory.mktemp("plan")
    (at / "p.cpp").write_text("""
#include <cstdio>
#include "umas_plan.h"
int main() {
  long long n, rows, d, V, room;
  while (std::scanf("%lld %lld %lld %lld %lld", &n, &rows, &d, &V, &room) == 5) {
    const umas::GradPlan p = umas::plan_gradients(n, rows, static_cast<int>(d), static_cast<int>(V), static_cast<size_t>(room));
    std::printf("%d %d %d\\n", p.dh.slices, p.dh.voc_blks, p.dw_apart ? 1 : 0);
  }
}""")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", f"-I{HERE}/../paper_2605_26646_amd/csrc", "-o", at / "p", at / "p.cpp"], check=True)

    def ask(cases):
        out = subprocess.run([at / "p"], input="\n".join(" ".join(map(str, c)) for c in cases), check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return ask


# column tiles of which whole rounds leave compute units idle (86 to 95 in two slices, 129 to 191 in one) among others, and little room
def test_dh_alone_is_cut_into_whole_rounds_and_else_as_beside_dw(plan):
    cases = [(rows, rows, tiles * 256 - off, V, room) for rows in (65, 128, 200, 256) for tiles in (4, 8, 16, 60, 85, 86, 90, 95, 96, 127, 128, 129, 160, 191, 192, 255, 256, 300)
             for off in (0, 248) for V in (300, 5000, 15000, 60000, 151936) for room in (0, 20 << 20, 60 << 20, GIB)]
    kinds = set()
    for (n, _, d, V, room), (slices, blks, apart) in zip(cases, plan(cases)):
        tiles, tiles_v = -(-d // 256), -(-V // 256)

        def cut(want):
            want = min(want, room // (tiles * 256 * 256 * 4), tiles_v)
            per = -(-tiles_v // want) if want >= 2 else tiles_v
            return -(-tiles_v // per), per
        beside, alone = cut((CUS + tiles - 1) // tiles), cut(CUS // tiles)
        assert slices * blks >= tiles_v > (slices - 1) * blks and (slices == 1 or slices * tiles * 256 * 256 * 4 <= room)
        assert (slices, blks) == (alone if apart else beside), (n, d, V, room)
        assert not apart or alone[0] * tiles >= 192
        kinds.add((apart, alone == beside))
    assert len(kinds) == 4


def test_rows_that_have_a_launch_for_dw(plan):
    cases = [(n, n, 3584, 152064, GIB) for n in (1, 64, 65, 256, 257, 700)] + [(200, 200, 2048, V, GIB) for V in ((1 << 17) - 1, 1 << 17)]
    cases += [(128, 128, 4096, V, GIB) for V in (81919, 81920)] + [(128, 128, 4104, 90000, GIB), (129, 129, 4104, 90000, GIB)]
    assert [p[2] for p in plan(cases)] == [0, 0, 1, 1, 0, 0, 0, 1, 0, 1, 0, 1]
