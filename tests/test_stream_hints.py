"""The particle passes stream non-temporally where they are said to, which no result shows.  The
compiler drops the hint of an access that it folds with one without it, so the gfx950 assembly of
the passes is read: each form has to hold exactly the non-temporal loads and stores that its
particle arrays need.  And the host's choice of the form, at its lines."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2606_28534_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled name -> (non-temporal loads, non-temporal stores) of both passes' kernels."""
    out = {}
    tmp = tmp_path_factory.mktemp("asm")
    runs = []
    for src in ("pic_pass32", "pic_pass64"):
        cmd = [build.HIPCC, "-x", "hip", *build.COMMON, "-S", "--cuda-device-only", "-c",
               os.path.join(build.CSRC, src + ".hip"), "-o", str(tmp / (src + ".s"))]
        runs.append((src, subprocess.Popen(cmd, stderr=subprocess.DEVNULL)))
    for src, p in runs:
        assert p.wait() == 0, src
        parts = re.split(r"^(_ZN3pic\w+):.*$", (tmp / (src + ".s")).read_text(), flags=re.M)
        for name, body in zip(parts[1::2], parts[2::2]):
            body = body.split(".Lfunc_end")[0]
            out[name] = tuple(len(re.findall(rf"global_{a}\S* .*\bnt\b", body)) for a in ("load", "store"))
    return out


CACHED, STORES, STREAM = 0, 1, 2
PUSH, FUSED, FUSED_PLAIN = 1, 7, 5


def of(kernels, *args):
    """The counts of k_pass32<stages, particles per thread, access, sorting, candidates inside>."""
    want = "k_pass32I" + "".join(f"L{'b' if i == 3 else 'i'}{int(a)}E" for i, a in enumerate(args)) + "E"
    (hit,) = [v for k, v in kernels.items() if want in k]
    return hit


# the arrays a pass reads: cell, offset, three velocities and, with collisions, the id; it writes all but
# the id in place (a sorting pass scatters them with ordinary stores).  With candidates inside (1, or 2
# with relative-speed charge exchange) their velocities are written again with ordinary stores.
@pytest.mark.parametrize("ppt", [4, 8])
@pytest.mark.parametrize("stages,arrays,inside", [(FUSED, 6, 0), (FUSED, 6, 1), (FUSED, 6, 2), (PUSH, 5, 0), (FUSED_PLAIN, 5, 0)])
def test_passes(kernels, ppt, stages, arrays, inside):
    runs = ppt // 4  # 16-byte accesses per thread and array
    assert of(kernels, stages, ppt, CACHED, False, inside) == (0, 0)
    assert of(kernels, stages, ppt, STREAM, False, inside) == (arrays * runs, 5 * runs)
    if stages != FUSED or ppt == 8:
        assert of(kernels, stages, ppt, STORES, False, inside) == (0, 5 * runs)


@pytest.mark.parametrize("ppt", [4, 8])
@pytest.mark.parametrize("inside", [0, 1, 2])
def test_sorting_pass(kernels, ppt, inside):
    assert of(kernels, FUSED, ppt, CACHED, True, inside) == (0, 0)
    assert of(kernels, FUSED, ppt, STREAM, True, inside) == (6 * ppt // 4, 0)


def test_fp64_push(kernels):
    # four arrays, two 16-byte accesses each
    hits = {k.split("k_particlesI")[1][:9]: v for k, v in kernels.items() if "k_particlesILi1E" in k}
    assert hits == {"Li1ELb0EE": (0, 0), "Li1ELb1EE": (8, 8)}


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """The host's rules, compiled for the CPU: slots -> lines, (coll, inside, ppt, lines, always) -> access."""
    tmp = tmp_path_factory.mktemp("rules")
    (tmp / "r.cpp").write_text('''#include "pic_rules.h"
extern "C" int lines(long n) { return pic::stream_lines(n); }
extern "C" int access(int coll, int inside, int ppt, int lines, int always)
{
    return pic::pass32_access(coll != 0, inside != 0, ppt, lines, always != 0);
}
extern "C" int push64(int lines) { return pic::pass64_streams(lines); }
''')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(tmp / "r.cpp"), "-o",
                    str(tmp / "r.so")], check=True)
    return ctypes.CDLL(str(tmp / "r.so"))


SIZES = [(1, 4, 10_000_000, 10_000_000), (0, 4, 14_000_000, 16_500_000), (1, 8, 14_000_000, 21_000_000),
         (0, 8, 14_000_000, 21_000_000)]


@pytest.mark.parametrize("coll,ppt,stores,stream", SIZES)
@pytest.mark.parametrize("inside", [0, 1])
def test_choice_by_size(rules, coll, ppt, stores, stream, inside):
    for n in (0, 1, stores - 1, stores, stream - 1, stream, 2**32 - 1):
        want = STREAM if n >= stream else STORES if n >= stores else CACHED
        assert rules.access(coll, inside, ppt, rules.lines(ctypes.c_long(n)), 0) == want, n


@pytest.mark.parametrize("coll,ppt,stores,stream", SIZES)
@pytest.mark.parametrize("inside", [0, 1])
def test_the_option_never_streams_less(rules, coll, ppt, stores, stream, inside):
    for n in (0, stores, stream):
        lines = rules.lines(ctypes.c_long(n))
        got = rules.access(coll, inside, ppt, lines, 1)
        assert got == (STREAM if coll and not inside else rules.access(coll, inside, ppt, lines, 0)), n


def test_choice_of_the_fp64_push(rules):
    assert [rules.push64(rules.lines(ctypes.c_long(n))) for n in (0, 9_999_999, 10_000_000, 2**32 - 1)] == [0, 0, 1, 1]
