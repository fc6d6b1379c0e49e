"""Which sizes the FP32 products take (csrc/extents.hpp, compiled for the host): byte offsets of 32 bits that run over the
padded rows must not come round to an operand's first ones, and a call has the same limit whether its D is read in place
or from a padded copy."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_14973_amd", "csrc")

# one call's products at (nr, ns), D in place (pitch nr) or padded: r = D X - U, D^H r, [a | b]
PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "extents.hpp"
using namespace tlr;
int main() {
    long long nr, ns, in_place;
    while (std::scanf("%lld %lld %lld", &nr, &ns, &in_place) == 3) {
        const long long lds = (ns + 127) / 128 * 128, ldk = (nr + 127) / 128 * 128, ld = in_place ? nr : ldk;
        const long long kr = (nr + 15) / 16 * 16, ks = (ns + 15) / 16 * 16;
        const Extents r = gemm_extents(lds, ldk, kr, ns, kr, false, ld, ldk, 0);
        const Extents w = gemm_extents(ldk, ldk, ks, nr, ns, true, ld, ld, 0);
        const Extents l = gemm_extents(lds, ldk, kr, ns, kr, false, ldk, ldk, ldk * ldk);
        std::printf("%d %d %d %d %lld %lld %lld\n", field_fits(lds, ldk), r.fit, w.fit, l.fit, (long long)r.bytesA,
                    (long long)w.bytesA, (long long)l.bytesB);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is missing")
    d = tmp_path_factory.mktemp("extents")
    (d / "extents.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + CSRC, str(d / "extents.cpp"), "-o", str(d / "extents")], check=True)

    def ask(cases):
        text = "\n".join("%d %d %d" % c for c in cases) + "\n"
        out = subprocess.run([str(d / "extents")], input=text, capture_output=True, text=True, check=True).stdout
        return [[int(v) for v in line.split()] for line in out.splitlines()]
    return ask


def _up(n, m):
    return (n + m - 1) // m * m


# true sizes below 4 GiB, padded ones not: offsets of the last row block, or of the last k step, pass 2^32
@pytest.mark.parametrize("nr,ns", [(16000, 33537), (16000, 33554), (23170, 23170), (1000, 536870), (1152, 466033),
                                   (8320, 64520), (8320, 64527)])
@pytest.mark.parametrize("in_place", [0, 1])
def test_sizes_that_pass_4_gib_with_their_padding_are_refused(sizes, nr, ns, in_place):
    assert ns * nr * 8 < 2 ** 32 <= _up(ns, 128) * _up(nr, 128) * 8
    assert sizes([(nr, ns, in_place)])[0][0] == 0


def test_every_offset_of_an_accepted_size_fits(sizes):
    rng = random.Random(5)
    cases = []
    while len(cases) < 4000:
        nr = int(2 ** rng.uniform(0, 17))
        ns = max(1, int(2 ** 29 / nr * 2 ** rng.gauss(0, 0.02)) if rng.random() < 0.7 else int(2 ** rng.uniform(0, 20)))
        cases.append((nr, ns, rng.randint(0, 1)))
    seen = [0, 0]
    for (nr, ns, in_place), (field, fr, fw, fl, ar, aw, bl) in zip(cases, sizes(cases)):
        lds, ldk, kr, ks = _up(ns, 128), _up(nr, 128), _up(nr, 16), _up(ns, 16)
        ld = nr if in_place else ldk
        # as before D was read in place: the padded field decides for D, and X (line products: X2 after X1) for B
        assert field == (lds * ldk * 8 < 2 ** 32)
        if field:
            assert fw and fr == (kr * ldk * 8 < 2 ** 32) and fl == ((kr + ldk) * ldk * 8 < 2 ** 32)
        if fr:   # largest offsets: row M - 1, k K - 1
            assert ((lds - 1) * ld + kr) * 8 <= 2 ** 32 and ((kr - 1) * ldk + ldk) * 8 < 2 ** 32 and ar == ns * ld * 8
        if fw:
            assert ((ks - 1) * ld + ldk) * 8 < 2 ** 32 and aw == ns * ld * 8
        if fl:
            assert bl == (kr + ldk) * ldk * 8
        seen[field] += 1
    assert min(seen) > 500
