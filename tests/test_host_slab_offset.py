"""The scalar offset of the small-tile and split products' loads (gemm_tile.h) stays below the declared buffer size for
every slab that is fetched, those past the end of K included, with operands just under 2 GiB."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "gemm_tile.h"
using namespace d2ft;
int main() {
    const long limit = 1L << 31;
    for (long ld : {64L, 768L, 3072L, 4096L, 65536L})
        for (int es : {2, 4}) {
            const int bk = 128 / es;                          // 64-wide tiles: 128 bytes of k per slab; split products 32
            const int K = (int)((limit - 1) / (ld * es));     // the largest K of such an operand
            const unsigned sk = (unsigned)(ld * es);
            for (int k0 = K / bk * bk - 4 * bk; k0 <= K + 4 * 4 * bk; k0 += bk) {   // up to four slabs ahead in each of four K groups
                const unsigned at = slab_offset(k0, k0, K, sk);
                if (at >= kBufBytes || (k0 < K && at != (unsigned)k0 * sk)) {
                    printf("ld %ld es %d K %d k0 %d: %u\n", ld, es, K, k0, at);
                    return 1;
                }
            }
        }
    return 0;
}
"""


def test_offsets_stay_inside_the_buffer(tmp_path):
    from paper_2504_12471_amd import build
    src, exe = tmp_path / "slab.hip", tmp_path / "slab"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
