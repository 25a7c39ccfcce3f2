"""The split of the QR's products over row chunks (csrc/qr_split.h, host code)."""
import subprocess

from paper_2207_03803_amd import build

PROGRAM = """
#include <stdio.h>
#include "qr_split.h"
int main()
{
    long rows, pw, nt, fp32, target, cap;
    while (scanf("%ld %ld %ld %ld %ld %ld", &rows, &pw, &nt, &fp32, &target, &cap) == 6) {
        const gap::QrSplit q = gap::qr_split(rows, pw, nt, 128, fp32 ? 128 : 64, fp32 != 0, target, cap);
        printf("%d %ld %ld %ld %ld\\n", (int)q.small, (long)q.nq, (long)q.np, (long)q.chunk, (long)q.nch);
    }
}
"""


def _ceil(a, b):
    return -(-a // b)


def test_fp32_sums_are_no_longer_than_2048_workgroups_make_them(tmp_path):
    """A chunk's rows are added up in FP32. Their number is bounded by that of 2,048 (or the
    given number of) workgroups of 128 x 128 tiles, whole stages of 16 rows, at least 256; the
    chunks cover the rows and fit the partial sums' space, which holds `cap` of them."""
    src = tmp_path / "split.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "split"
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    cases = [(rows, pw, nt, fp32, target, cap)
             for rows in (1, 63, 64, 700, 2_259, 4_096, 4_097, 7_118, 10_256, 16_257, 18_250, 34_000, 110_000)
             for pw in (1, 64, 100, 128, 160, 256)
             for nt in (1, 64, 65, 128, 129, 245, 856, 1_995, 3_745, 9_745)
             for fp32 in (0, 1)
             for target in (0, 256, 1_024, 2_048)
             # a product of a few columns takes more chunks: the space is (32, columns) or (256, 128)
             for cap in ((32,) if nt > 256 else (32, 128, 256))]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                         text=True, check=True).stdout.split("\n")
    for (rows, pw, nt, fp32, target, cap), line in zip(cases, out):
        small, nq, np_, chunk, nch = map(int, line.split())
        what = (rows, pw, nt, fp32, target, cap, line)
        assert 1 <= nch <= cap and (nch - 1) * chunk < rows <= nch * chunk and chunk % 16 == 0, what
        assert nq * (64 if small else (128 if fp32 else 64)) >= nt and np_ * (64 if small else 128) >= pw, what
        if fp32:
            n = min(_ceil(target or 2_048, _ceil(nt, 128) * _ceil(pw, 128)), cap)
            assert chunk <= max(256, _ceil(_ceil(rows, n), 16) * 16), what
