"""CPU check of the 32-bit byte counts of buffer resources: where the host lets a
lattice onto the tile kernels (tile_fits) or the SAP kernel (sap_fits), every
resource they form holds its components whole."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_06347_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# sites around the limits of one, two and three components of 4, 8 and 16 bytes, and 112 x 96^3
EDGES = sorted({((1 << 32) // (n * s) + d) for n in (1, 2, 3) for s in (4, 8, 16) for d in (-1, 0, 1)} | {112 * 96 ** 3})


def widths(name):
    """Components of every resource that a source file forms."""
    src = open(os.path.join(CSRC, name)).read()
    src = re.sub(r"//[^\n]*", "", src)
    calls = re.findall(r"comp_rsrc(?:<(\w+)>)?\(([^;]*)", src)
    out = set()
    for n, args in calls:
        if args.startswith("S* f"):     # the definition
            continue
        out.add(n or re.search(r", (\d), \w+\)", args).group(1))
    return out


@pytest.fixture(scope="module")
def fits(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("bounds")
    (d / "b.hip").write_text("""#include "tile.h"
#include <cstdio>
int main() {
    const size_t V[] = {%s};
    for (size_t v : V) std::printf("%%zu %%d %%d %%d %%d\\n", v, (int)tile_fits(v, 4), (int)tile_fits(v, 8),
                                   (int)tile_fits(v, 16), (int)sap_fits(v));
    std::printf("%%d %%d\\n", TILE_COMPS, SAP_COMPS);
}
""" % ", ".join(map(str, EDGES)))
    r = subprocess.run([HIPCC, "-std=c++17", "--offload-host-only", "-I", CSRC, str(d / "b.hip"), "-o", str(d / "b")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = subprocess.run([str(d / "b")], capture_output=True, text=True, check=True).stdout.splitlines()
    tile, sap = map(int, lines.pop().split())
    return [list(map(int, l.split())) for l in lines], {"TILE_COMPS": tile, "SAP_COMPS": sap}


def test_no_resource_wraps(fits):
    rows, comps = fits
    n = lambda w: comps[w] if w in comps else int(w)   # noqa: E731
    tile = max(map(n, widths("tile.h") | widths("dslash.hip")))
    sap = max(map(n, widths("tile.h") | widths("sap.hip")))
    assert len(rows) == len(EDGES)
    for V, f16, f32, f64, s in rows:
        for ok, size, most in ((f16, 4, tile), (f32, 8, tile), (f64, 16, tile), (s, 8, sap)):
            assert not ok or most * V * size < 1 << 32, (V, size)
    # 112 x 96^3 in FP64 (two columns in and out fit the device) stays on the tile kernels
    assert [r[3] for r in rows if r[0] == 112 * 96 ** 3] == [1]
