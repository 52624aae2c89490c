"""The delta of two symbols, compiled for the host from the header that the kernels take it from: what the
definition says for symbols of the stated numbers of bins, and a delta that fits its field for any other bits."""
import subprocess

from paper_2306_11800_amd import build

PROGRAM = r"""
#include "inshr_dev.h"
#include <algorithm>
#include <cstdio>
int main()
{
    const u32 bins[] = {2, 3, 4, 6, 8, 12, 16, 32, 64, 128, 256};
    int bad = 0;
    for (u32 Kp : bins)
        for (u32 Kc : bins) {
            const u32 B = std::max(Kp, Kc) + 2u;
            for (u32 prev = 0; prev < Kp + 2u; prev++)
                for (u32 cur = 0; cur < 1u << inshr::symbol_bits(Kc); cur++) {
                    const u32 d = inshr::delta_of(prev, cur, B);
                    if (d >= B || (cur < B && d != (prev + B - cur) % B)) {
                        if (bad++ < 5) printf("K %u %u, symbols %u %u: %u\n", Kp, Kc, prev, cur, d);
                    }
                }
        }
    return bad != 0;
}
"""


def test_deltas_fit_their_field(tmp_path):
    src, exe = tmp_path / "delta.hip", tmp_path / "delta"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", "--offload-host-only", "-O1", "-std=c++17", "-Wno-everything", "-I", build.CSRC, str(src),
                    "-o", str(exe)], check=True, capture_output=True, timeout=100)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
