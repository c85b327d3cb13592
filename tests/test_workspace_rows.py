"""The workspace covers the range counts the library chooses: its own choice and its own row count, compiled for the host, over every head
dimension, type, batch and length of a wide grid (no GPU: 256 compute units are assumed)."""
import os
import subprocess

from paper_2605_17447_amd import binding as fb
from paper_2605_17447_amd._build import CSRC, INCLUDE, LIB

PROGRAM = r"""
#include <cstdio>
#include "api.hip"
int main()
{
    long n = 0, bad = 0;
    const int heads[][2] = {{1, 1}, {4, 1}, {8, 1}, {16, 2}, {28, 4}, {9, 3}, {40, 10}, {64, 8}, {16, 16}, {128, 8}};
    const int ops[] = {FASTOCR_OP_FOCAL_SCORE, FASTOCR_OP_SPARSE_DECODE_ATTN, FASTOCR_OP_DENSE_DECODE_ATTN};
    for (auto &h : heads)
        for (int d : {128, 64})
            for (int f32 = 0; f32 < 2; ++f32)
                for (int B = 1; B < 900; B += B < 70 ? 1 : 7)
                    for (int tiles = 0; tiles < 1300; tiles += tiles < 130 ? 1 : 37)
                        for (int op : ops)
                            for (int form = 0; form < 3; ++form) {              // launched, replayed, parking its logits
                                if (form == 2 && (op != FASTOCR_OP_DENSE_DECODE_ATTN || f32)) continue;
                                Shape s{};
                                s.batch = B; s.n_q_heads = h[0]; s.kv.n_kv_heads = h[1]; s.kv.head_dim = d;
                                s.fast = !f32; s.fast32 = f32; s.dtype = f32 ? FASTOCR_F32 : FASTOCR_BF16;
                                const int L = tiles ? 32 * tiles - 5 : 0;
                                const int ranges = choose_splits(op, s, L, nullptr, form == 1, form == 2);
                                const size_t rows = partial_rows(op, s, L, choose_splits(op, s, L, nullptr, 0, form == 2), form == 2);
                                ++n;
                                if ((size_t)B * h[0] * ranges > rows && bad++ < 10)
                                    printf("%d/%d heads of %d, fp32 %d, batch %d, %d tokens, call %d, form %d: %d ranges, %zu rows\n", h[0], h[1], d, f32, B, L, op, form, ranges, rows);
                            }
    printf("%ld checked, %ld beyond their workspace\n", n, bad);
    return bad != 0;
}
"""


def test_chosen_ranges_stay_inside_the_workspace(tmp_path):
    fb.load_library()
    (tmp_path / "rows.hip").write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-c", "-fPIE", "-O2", "-std=c++17", "-w", "-I", INCLUDE, "-I", CSRC,
                           str(tmp_path / "rows.hip"), "-o", str(tmp_path / "rows.o")])
    rocm = os.path.join(os.path.dirname(os.path.dirname(hipcc)), "lib")
    # (the launches and the timers it names come from the library itself; nothing is launched)
    subprocess.check_call(["g++", str(tmp_path / "rows.o"), "-o", str(tmp_path / "rows"), LIB, "-L" + rocm, "-lamdhip64",
                           "-Wl,-rpath," + os.path.dirname(LIB), "-Wl,-rpath," + rocm])
    r = subprocess.run([str(tmp_path / "rows")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 beyond" in r.stdout, r.stdout
