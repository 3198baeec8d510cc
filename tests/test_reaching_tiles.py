"""The tiles whose deposits reach a field task, and a lane of it (reaching_tiles of pic_internal.h, compiled for
the host), against every image of every tile: open and periodic axes, whole and cut last tiles."""
import subprocess

from paper_2501_07465_amd import build as B

SOURCE = r'''
#include "pic_internal.h"
#include <cstdio>
#include <set>
using namespace pic;
static SimDev S;
static int tile_of(int u)  // -1: none
{
    const int k = S.ntile[0];
    return S.periodic[0] ? ((u % k) + k) % k : (u < 0 || u >= k ? -1 : u);
}
static std::set<int> by_images(int x0, int x1)
{
    std::set<int> r;
    for (int t = 0; t < S.ntile[0]; ++t)
        for (int k = -3; k <= 3; ++k) {
            const int s = t * S.T[0] + k * S.n[0];
            if ((k == 0 || S.periodic[0]) && s - kGL <= x1 && s + S.T[0] - 1 + kGHj >= x0) r.insert(t);
        }
    return r;
}
int main()
{
    long tasks = 0, wrong = 0;
    for (int sh = 0; sh <= 6; ++sh)
        for (int n = 2; n <= 200; ++n)
            for (int per = 0; per < 2; ++per) {
                const int T = 1 << sh, nt = (n + T - 1) / T;
                if (per ? 2 * n <= (nt - 1) * T + T + 2 : n < 4) continue;  // refused grids
                S.T[0] = T; S.Tshift[0] = sh; S.n[0] = n; S.periodic[0] = per; S.ntile[0] = nt;
                S.tcut[0] = per ? nt * T - n : 0;
                for (int F : {1, 2, 3, 6, 10, 61, 256})
                    for (int x0 = 0; x0 < n; x0 += F) {
                        const int x1 = per && x0 + F > n ? n : x0 + F;
                        int lo, count, l, c;
                        reaching_tiles(S, 0, x0, x1, lo, count);
                        std::set<int> got;
                        for (int u = lo; u < lo + count; ++u)
                            if (tile_of(u) >= 0) got.insert(tile_of(u));
                        ++tasks;
                        wrong += got != by_images(x0, x1);
                        for (int g = x0; g <= x1 && g <= n; ++g) {  // the task's bits that a node takes
                            reaching_tiles(S, 0, g, g, l, c);
                            got.clear();
                            for (int u = l > lo ? l : lo; u < l + c && u < lo + count; ++u)
                                if (tile_of(u) >= 0) got.insert(tile_of(u));
                            wrong += got != by_images(g, g);
                        }
                    }
            }
    std::printf("%ld tasks, %ld wrong\n", tasks, wrong);
    return tasks > 100000 && wrong == 0 ? 0 : 1;
}
'''


def test_reaching_tiles_are_those_of_the_images(tmp_path):
    src, exe = tmp_path / "reach.cpp", tmp_path / "reach"
    src.write_text(SOURCE)
    subprocess.run([B.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I" + B.ROOT + "/include",
                    "-I" + B.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
