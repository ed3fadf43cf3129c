"""Stores through the L2 are assembly, where the compiler does not see the wait states that a store of 16 bytes needs before its data may be overwritten: two of them behind
every such store, as the compiler's own stores get, whatever it schedules there."""
import os
import re
import shutil
import subprocess

import pytest

import test_gpu_store_through
from paper_2603_05232_amd import binding, build

PROBE = """
#include "ss_common.h"
__global__ void probe(uint4* p, uint32_t a, uint32_t b, uint32_t n)
{
    uint4 v = make_uint4(a + threadIdx.x, b, threadIdx.x, a * threadIdx.x);
    for (uint32_t i = 0; i < n; ++i) {
        ss::store_through(p + threadIdx.x + i * 64, v);
        v.x = v.x * 3 + i; v.y ^= v.x; v.z += v.y; v.w -= v.z;
    }
}
"""


def _assembly(source, target):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    subprocess.run([hipcc, *build.FLAGS, "-S", "--cuda-device-only", str(source), "-o", str(target)], check=True, stderr=subprocess.DEVNULL)
    with open(target) as f:
        return f.read()


def _own_wait_states(text):
    """For each 16-byte store through the L2: the wait states that its statement ends with."""
    found = []
    for behind in re.findall(r"global_store_dwordx4 [^\n]* sc0 sc1\n(.*?);;#ASMEND", text, re.S):
        lines = [line.split() for line in behind.splitlines() if line.strip()]
        found.append(sum(int(line[1]) + 1 if line[0] == "s_nop" else 1 for line in lines))
    return found


def test_wait_states_behind_a_store_of_16_bytes(tmp_path):
    (tmp_path / "probe.hip").write_text(PROBE)
    states = _own_wait_states(_assembly(tmp_path / "probe.hip", tmp_path / "probe.s"))
    assert states and min(states) >= 2, states


def test_pruning_has_them_only_where_they_are_taken(tmp_path):
    """k_prune_rows<TIN, OUT, N>: 8-bit codes (OUT 0 and 1) whose unit, the fewest blocks of 2N weights that fill 16-byte vectors, is one store of 8 or 16 bytes."""
    text = _assembly(os.path.join(build.CSRC, "prune_quant.hip"), tmp_path / "prune_quant.s")
    have = set()
    for name, body in re.findall(r"^(_ZN2ss12k_prune_rows\w+):(.*?)s_endpgm", text, re.M | re.S):
        tin, out, n = re.match(r"_ZN2ss12k_prune_rowsI(\w)Li(\d)ELi(\d)E", name).groups()
        if " sc0 sc1" in body:
            have.add(({"f": 4, "t": 2}[tin], int(out), int(n)))
    wanted = set()
    for size in (2, 4):
        for n in range(2, 9):
            block = 2 * n * size
            codes = next(b for b in (1, 2, 4) if b * block % 16 == 0) * 2 * n
            if codes in (8, 16):
                wanted |= {(size, 0, n), (size, 1, n)}
    assert have == wanted, (sorted(have - wanted), sorted(wanted - have))


RULE = """
#include "quant_common.h"
#include <stdio.h>
int main()
{
    int es, vec, N; long long M, row;
    while (scanf("%d %d %lld %lld %d", &es, &vec, &M, &row, &N) == 5) printf("%d\\n", (int)ss::lift_through(es, vec, M, row, N));
}
"""


@pytest.fixture(scope="module")
def through(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(RULE)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def ask(es, vec, M, row, N):
        return subprocess.run([str(d / "rule")], input=f"{es} {vec} {M} {row} {N}\n", stdout=subprocess.PIPE, text=True, check=True).stdout.strip() == "1"
    return ask


def test_quantiser_rule(through):
    for act, dtype, K, N, last in test_gpu_store_through.ROWS:
        vec, row = (4 if act == "fp32" else 8), binding.slide_lifted_ld(K, N, dtype)
        for megabytes, beyond, expected in ((4, -1, False), (4, 1, True), (last, -1, True), (last, 1, False)):
            assert through(1, vec, test_gpu_store_through.rows_of(megabytes, beyond, dtype, K, N), row, N) == expected, (act, dtype, K, N, megabytes, beyond)
    # rows of a length that a GEMM of few channels would wait for; 16-bit codes, and stores of four bytes
    for row in (1920, 2048, 2944):
        assert not any(through(1, 8, (mb << 20) // row, row, 2) for mb in (5, 7, 12, 24))
    for row in (2048, 3072, 4096, 5504):
        for N in (2, 4):
            assert not any(through(1, 8, (mb << 20) // row, row, N) for mb in (9, 12, 24)) and through(1, 8, (5 << 20) // row, row, N) == (N == 4 or row >= 3072)
    assert not through(2, 8, 3000, 2048, 4) and not through(1, 4, 5000, 1024, 2)
