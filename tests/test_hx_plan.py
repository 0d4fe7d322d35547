"""How the c128 products are cut into workgroups (hx_plan.h, host code),
compiled alone with the host compiler (CPU only)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_10557_amd", "csrc")

# one line per "rows2 N ws" of stdin (ws < 0: the workspace of hx_workspace for
# -ws columns)
MAIN = r"""
#include "hx_plan.h"
#include <cstdio>
using namespace chase;
int main() {
  long long rows2, N, ws;
  while (std::scanf("%lld %lld %lld", &rows2, &N, &ws) == 3) {
    const size_t bytes = ws < 0 ? hx_workspace(rows2, -ws) : (size_t)ws;
    const HxPlan p = hx_plan(rows2, N, bytes);
    std::printf("%lld %zu %d %d %d %d %d %d %d %lld %lld %d %zu\n", (long long)hx_group(rows2), bytes, p.shape, p.TM, p.TN, p.wq, p.wr, p.KB, p.teams,
                (long long)p.lq, (long long)p.unit, p.lr, hx_plan_bytes(p));
  }
}
"""
KEYS = "group ws shape TM TN wq wr KB teams lq unit lr need".split()


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("hx_plan")
    (d / "main.cpp").write_text(MAIN)
    cc = shutil.which("g++") or shutil.which("c++")
    assert cc, "no C++ compiler"
    subprocess.run([cc, "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def run(cases):
        text = "\n".join("%d %d %d" % c for c in cases) + "\n"
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [dict(zip(KEYS, map(int, line.split()))) for line in out.splitlines()]

    return run


def _sizes():
    return [(2 * m, n) for m in (3, 40, 500, 850, 900, 1000, 1050, 1200, 1250, 1450, 1700, 2000, 2011, 2100, 4000, 9000)
            for n in (1, 16, 100, 256, 417, 544, 576, 640, 800, 967, 1024)]


def test_every_product_runs_as_with_unlimited_workspace(plans):
    # the handle's workspace is hx_workspace of its widest product: no width
    # up to there may be cut differently for want of room
    sizes = _sizes()
    have = plans([(r, n, -1024) for r, n in sizes])
    free = plans([(r, n, 1 << 40) for r, n in sizes])
    for (r, n), p, q in zip(sizes, have, free):
        assert {k: p[k] for k in KEYS[2:]} == {k: q[k] for k in KEYS[2:]}, (r, n)
        assert p["need"] <= p["ws"] <= 128 << 20


@pytest.mark.parametrize("m,k", [(1000, 400), (1050, 272), (1200, 417), (1200, 480), (1250, 320), (1450, 288), (1450, 320)])
def test_wide_products_at_m_near_1000_use_the_chip(plans, m, k):
    # with 64 KB of workspace a row these ran on whole strips, 100 to 250 of
    # the 512 workgroups
    p = plans([(2 * m, 2 * k, -1024)])[0]
    assert p["shape"] >= 0 or p["teams"] * p["TN"] > 448, p


@pytest.mark.parametrize("ws", [0, 1 << 20, 8 << 20, 16 << 20, 40 << 20])
def test_little_workspace(plans, ws):
    # partial sums fit, no part is empty and the parts cover every strip; never
    # fewer teams than whole strips would have
    for (r, n), p in zip(_sizes(), plans([(r, n, ws) for r, n in _sizes()])):
        if p["shape"] >= 0:
            continue
        assert p["need"] <= ws, (r, n)
        assert p["lq"] >= 1 and 0 <= p["lr"] < p["teams"]
        length = p["lq"] * p["teams"] + p["lr"]
        assert length * p["unit"] == p["TM"] * p["KB"]
        assert p["teams"] >= min(p["TM"], max(1, 512 // p["TN"]))
        assert p["wq"] * p["TN"] + p["wr"] == -(-n // 16)
        if ws == 0 and p["KB"] > 1:
            assert p["unit"] == p["KB"] or p["TM"] % p["teams"] == 0


def test_wide_products_stay_in_the_cache(plans):
    # a launch takes as many columns as 256 MiB hold, whole tiles of 128
    ms = [10, 4000, 8000, 12000, 16000, 30000, 60000, 200000]
    for m, p in zip(ms, plans([(2 * m, 128, 0) for m in ms])):
        g = p["group"]
        assert g % 128 == 0 and g >= 128
        assert g == 128 or 16 * m * g <= 256 << 20 < 16 * m * (g + 128), m
    assert [p["group"] for p in plans([(60000, 1, 0), (32000, 1, 0)])] == [512, 1024]


def test_near_ties_of_the_largest_products(plans):
    wide = plans([(2 * m, n, 1 << 40) for m in (16000, 20000, 30000) for n in (384, 768)])
    assert all(p["wq"] == 8 and p["wr"] == 0 for p in wide)
    assert plans([(60000, 320, 1 << 40)])[0]["TN"] == 4
