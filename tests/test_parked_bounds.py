"""The reads of the launch that finishes parked logits stay inside the workspace the library asks for, whatever the longest sequence: the
kernel's own index, compiled for the host, against fastocr_workspace_bytes."""
import ctypes
import os
import subprocess

import pytest

from paper_2605_17447_amd import binding as fb
from paper_2605_17447_amd._build import CSRC, INCLUDE
from test_abi_host import _bv, _kv

# prints, for every longest sequence asked for, the first and one past the last byte that any lane's load of logits touches
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "kernels.hpp"
int main(int n, char **a)
{
    const int rows = atoi(a[1]);                                     // batch x query heads
    for (int i = 2; i < n; ++i) {
        const int S = atoi(a[i]);
        const int64_t pitch = fastocr::logit_pitch(S);
        const int tokens = 256 * ((S + 255) / 256 > 1 ? (S + 255) / 256 : 1);     // of whole workgroups, at least one
        int64_t lo = 1 << 30, hi = 0;
        for (int p = 0; p < tokens; p += 4)
            for (int row : {0, rows - 1}) {
                const int64_t at = 4 * (row * pitch + fastocr::parked_token(p, pitch));
                lo = at < lo ? at : lo;
                hi = at + 16 > hi ? at + 16 : hi;
            }
        printf("%lld %lld\n", (long long)lo, (long long)hi);
    }
}
"""


@pytest.fixture(scope="module")
def reads(tmp_path_factory):
    d = tmp_path_factory.mktemp("parked")
    (d / "reads.hip").write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", INCLUDE, "-I", CSRC, str(d / "reads.hip"), "-o", str(d / "reads")])

    def run(rows, lengths):
        out = subprocess.check_output([str(d / "reads"), str(rows), *map(str, lengths)], text=True)
        return [tuple(map(int, l.split())) for l in out.splitlines()]

    return run


@pytest.mark.parametrize("B,Hq,Hkv,d", [(1, 1, 1, 64), (2, 64, 8, 128), (3, 28, 4, 128), (5, 16, 16, 64)])
def test_reads_stay_inside_the_workspace(reads, B, Hq, Hkv, d):
    lib = fb.load_library()
    lengths = [0, 1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 700, 4097]
    for S, (lo, hi) in zip(lengths, reads(B * Hq, lengths)):
        for op in (fb.OP_FOCAL_SCORE, fb.OP_FOCAL_ATTN_SCORE):
            kv, bv = _kv(Hkv=Hkv, d=d, S=max(S, 1)), _bv(B, S, S)
            need = lib.fastocr_workspace_bytes(op, ctypes.byref(kv), ctypes.byref(bv), Hq, 0)
            assert 0 <= lo and hi <= need, f"{S} tokens: bytes {lo} .. {hi} of a workspace of {need}"
