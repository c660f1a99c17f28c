"""The divisions that kernels do by multiplying (FastDiv, Cut in csrc/launch.h) against the compiler's own, on the host."""
import os
import shutil
import subprocess

import pytest

from paper_2309_16119_amd import build

PROGRAM = r"""
#include "launch.h"
#include <cstdio>
using namespace mlr;
static uint64_t state = 1;
static uint32_t draw() { state = state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(state >> 33) << 1 ^ (uint32_t)(state >> 40); }
static int bad = 0;
static void one(uint32_t n, uint32_t d) {
    uint32_t rest;
    const uint32_t q = fast_div(d).div(n, rest);
    if (q != n / d || rest != n % d) { if (++bad < 9) printf("%u / %u: %u rest %u\n", n, d, q, rest); }
}
static void cut(uint32_t total, uint32_t parts) {
    const Cut c = make_cut(total, parts);
    for (uint32_t i = 0; i <= parts; ++i)
        if (c.begin(i) != (uint32_t)((uint64_t)total * i / parts)) { if (++bad < 9) printf("part %u of %u in %u: %u\n", i, parts, total, c.begin(i)); }
}
int main() {
    const uint32_t edges[] = {0, 1, 2, 3, 255, 256, 257, 65535, 65536, 0x7FFFFFFF, 0x80000000u, 0x80000001u, 0xFFFFFFFEu, 0xFFFFFFFFu};
    for (uint32_t n : edges)
        for (uint32_t d : edges)
            if (d) { one(n, d); if (n >= 1) { one(n - 1, d); } one(n / d * d, d); one(n / d * d + d - 1, d); }
    for (int i = 0; i < 2000000; ++i) {
        const uint32_t d = (draw() >> (draw() & 31)) | 1u << (draw() & 7), n = draw() >> (draw() & 31);
        one(n, d);
        one(n / d * d, d);
    }
    for (uint32_t parts = 1; parts <= 600; ++parts)
        for (uint32_t total : {0u, 1u, 31u, 64u, 172u, 688u, 11008u, 0x03FFFFFFu, 0x7FFFFFFFu, draw() >> 8}) cut(total, parts);
    printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def _hipcc():
    for cand in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    return None


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_quotients_and_cuts_are_exact(tmp_path):
    src, exe = tmp_path / "divisions.hip", tmp_path / "divisions"
    src.write_text(PROGRAM)
    res = subprocess.run([_hipcc(), *build.HIPCC_FLAGS, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:]
