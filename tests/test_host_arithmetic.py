"""The arithmetic that kernels do on lengths from device memory, on the host: division by a launch's reciprocals against the
compiler's, and the rows that helper workgroups touch, also for offsets that no request can have.  No GPU is touched."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "common.h"
using namespace specvlm;

static int fail(const char* what, int a, int b, int c) { printf("%s %d %d %d\n", what, a, b, c); return 1; }

int main()
{
    const int edges[] = {0, 1, 2, 3, 7, 63, 64, 65, 1000, 65535, 65536, 1 << 24, 0x3fffffff, 0x7ffffffe, 0x7fffffff};
    srand(1);
    for (int i = 0; i < 2000000; ++i) {
        const int d = i & 1 ? 1 + rand() % 4096 : 1 + rand() % 0x7fffffff;
        const int x = i % 3 == 0 ? edges[i / 3 % 15] : i % 3 == 1 ? rand() : (int)((int64_t)d * (rand() % (0x7fffffff / d + 1)) - (i & 4 ? 1 : 0));
        if (x < 0) continue;
        const QuotRem got = divide(x, d, reciprocal(d));
        if (got.q != x / d || got.r != x % d) return fail("divide", x, d, got.q);
    }
    for (int n_help = 1; n_help <= 15; ++n_help) {
        for (int keys = -40000; keys <= 4000; keys += keys < -100 ? 97 : 1) {
            for (int queries = -2; queries <= 64; queries += queries < 8 ? 1 : 28) {
                const bool any = queries > 0 && keys >= queries;
                int next = 0;
                for (int k = 0; k < n_help; ++k) {
                    const RowRange r = helper_rows(queries, keys, k, n_help, reciprocal(n_help));
                    if (r.n < 0 || (r.n > 0 && (r.first != next || r.first + r.n > keys))) return fail("rows", keys, queries, n_help);
                    next += r.n;
                }
                if (next != (any ? keys : 0)) return fail("all rows", keys, queries, n_help);
            }
        }
    }
    puts("ok");
}
"""


def test_divisions_and_helper_rows(tmp_path):
    source, program = tmp_path / "arithmetic.hip", tmp_path / "arithmetic"
    source.write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2508_16201_amd", "csrc"), "-o", str(program), str(source)], check=True)
    res = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout == "ok\n", res.stdout + res.stderr
