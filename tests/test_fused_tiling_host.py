"""The tiling of the fused envelope groups (csrc/fdetd_envelope.h), compiled for the host: over random batches every
cell is an output of exactly one tile, no tile marches more rows than the row table holds, and a grid whose rows have
more bytes than an int counts -- the group kernel's row offsets -- is not taken."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12132_amd", "csrc")

PROGRAM = r'''
#include "fdetd_envelope.h"
#include <cstdio>
#include <vector>
using namespace fdetd;
int main() {
    unsigned s = 7;
    auto rnd = [&](int lo, int hi) { s = s * 1103515245u + 12345u; return lo + (int)((s >> 8) % (unsigned)(hi - lo + 1)); };
    for (int trial = 0; trial < 3000; ++trial) {
        const int nd = rnd(1, kEnvFuseND), count = rnd(1, 4), lag = (env_depth(nd) - 1) * nd, oc = env_out_columns(nd);
        int nz[4], nr[4], seg = 0, tiles = 0, all = 0;
        for (int t = 0; t < count; ++t) { nz[t] = rnd(2 * nd + 1, 400); nr[t] = rnd(nd + 1, rnd(0, 9) ? 200 : 3000); }
        if (!env_tiling(nd, count, nz, nr, seg, tiles) || seg < 1) return printf("FAIL tiling %d\n", trial), 1;
        for (int t = 0; t < count; ++t) {
            std::vector<char> seen((size_t)nz[t] * nr[t], 0);
            const int n = fused_tiles(nz[t], nr[t], seg, oc);
            all += n;
            for (int r = 0; r < n; ++r) {
                FuseTile c;
                if (!decode_fused(nz[t], nr[t], r, seg, oc, c) || c.k1 > nr[t]) return printf("FAIL tile %d\n", trial), 1;
                if (c.k1 - c.k0 + 3 * lag + 4 > kEnvRows) return printf("FAIL rows %d\n", trial), 1;
                for (int k = c.k0; k < c.k1; ++k)
                    for (int i = c.o0; i < c.o0 + oc && i < nz[t]; ++i) ++seen[(size_t)k * nz[t] + i];
            }
            for (char v : seen) if (v != 1) return printf("FAIL cover %d\n", trial), 1;
        }
        if (all != tiles) return printf("FAIL count %d\n", trial), 1;
    }
    int nz = kEnvColumns, nr = 2, seg, tiles;
    if ((long long)nz * 16 > 0x7fffffffll || !env_tiling(1, 1, &nz, &nr, seg, tiles)) return printf("FAIL widest\n"), 1;
    if (++nz, env_tiling(1, 1, &nz, &nr, seg, tiles)) return printf("FAIL wider\n"), 1;
    printf("tiling ok\n");
}
'''


def test_fused_tiles_cover_every_grid_once(tmp_path):
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__", "-I",
                    "/opt/rocm/include", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "tiling ok" in r.stdout, r.stdout + r.stderr
