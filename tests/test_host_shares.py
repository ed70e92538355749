"""Workgroups of a launch over a nest's grids (nest_shares and GridShares on
the host; hipcc only, no GPU): each group belongs to one grid and to one place
in it, and a large grid among small ones keeps most of the launch."""
import os
import shutil
import subprocess

import pytest

from paper_1705_00614_amd import build

SOURCE = r"""
#include "%s"
#include <cstdio>

static int bad = 0;
#define EXPECT(c) do { if (!(c)) { ++bad; printf("line %%d: %%s\n", __LINE__, #c); } } while (0)

// groups of every grid of a launch, by its index in `tiles`
static std::vector<int> groups(const std::vector<int>& tiles) {
    std::vector<int> order, got(tiles.size(), 0), of(tiles.size(), -1);
    const swe::GridShares s = swe::nest_shares(tiles, order);
    std::vector<std::vector<char>> seen(tiles.size());
    for (int t = 0; t < s.groups(); ++t) {
        int grid, before, all;
        s.at(t, grid, before, all);
        EXPECT(grid >= 0 && grid < (int)tiles.size() && before >= 0 && before < all);
        const int k = order[grid];
        EXPECT(of[k] == -1 || of[k] == all);
        of[k] = all;
        seen[k].resize(all, 0);
        EXPECT(!seen[k][before]);
        seen[k][before] = 1;
        ++got[k];
    }
    for (size_t k = 0; k < tiles.size(); ++k) EXPECT(got[k] == of[k] && got[k] >= 1);
    return got;
}

int main() {
    using V = std::vector<int>;
    // equal grids: as many each, a workgroup per tile where that is enough
    EXPECT((groups(V{256, 169, 169}) == V{32, 22, 22}));
    EXPECT((groups(V{169, 169}) == V{22, 22}));
    EXPECT((groups(V{4096, 4096, 4096}) == V{42, 42, 42}));
    // one large among many small: nearly all of the launch, wherever it stands
    for (int small = 1; small <= 64; ++small)
        for (int at : {0, small / 2, small}) {
            V t(small, 2);
            t.insert(t.begin() + at, 4096);
            const V g = groups(t);
            EXPECT(g[at] >= 120);
            EXPECT(g[at == 0 ? 1 : 0] == 1);
        }
    // 64 patches with a few more tiles each still leave the large grid most
    {
        V t(64, 16);
        t.push_back(16384);
        const V g = groups(t);
        EXPECT(g[64] >= 100 && g[0] == 2);
    }
    // many different counts, more than there are levels
    for (int n = 1; n <= 65; ++n) {
        V t;
        for (int k = 0; k < n; ++k) t.push_back(1 + (k * 7919) %% 977);
        const V g = groups(t);
        long long sum = 0;
        for (int k = 0; k < n; ++k) sum += g[k];
        EXPECT(sum <= 2 * (swe::NEST_GROUPS + swe::NEST_LEAST * n));
    }
    EXPECT((groups(V{(1 << 20) - 1}) == V{128}));
    EXPECT((groups(V{1}) == V{1}));
    printf("%%d wrong\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_shares_of_a_nest(tmp_path):
    src, exe = tmp_path / "shares.hip", tmp_path / "shares"
    src.write_text(SOURCE % os.path.join(build.CSRC, "swe_nest.hpp"))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run(["hipcc"] + flags + ["-o", str(exe), str(src)], check=True, capture_output=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
