"""Rows start at any element's address, so the vector loads and stores of the activations must be
declared at element alignment: the compiler takes a wider claim at its word (a load whose address
is the same for the whole wave goes through the scalar cache, which drops the low address bits).
Compiles the vector helpers for gfx950 and reads the alignment of each access.  CPU only."""
import os
import re
import subprocess

from paper_2408_03865_amd import build as B

PROBE = r"""
#include <hip/hip_runtime.h>
#include "common.hpp"
namespace pm {
template <typename T, int K>
__global__ void loads(const T* row, int64_t l0, int64_t L, T* o) {
    float v[K];
    unpack_run(load_raw<T, K>(row, l0), v);
    for (int i = 0; i < K; ++i) Storage<T>::store1(o++, v[i]);
    unpack_run(load_raw_nt<T, K>(row, l0 + 99), v);
    for (int i = 0; i < K; ++i) Storage<T>::store1(o++, v[i]);
    unpack_run(load_part<T, K, false>(row, l0 + 199, L), v);
    for (int i = 0; i < K; ++i) Storage<T>::store1(o++, v[i]);
}
template <typename T, int K>
__global__ void runs(const T* row, T* out, int64_t l0, int64_t L) {
    float v[K];
    load_run<T, K>(row, l0, L, v);
    store_run<T, K>(out, l0, L, v);
    store_run<T, K, true, false>(out + 99, l0, L, v);
}
#define LOADS(T, K) template __global__ void loads<T, K>(const T*, int64_t, int64_t, T*);
#define RUNS(T, K) template __global__ void runs<T, K>(const T*, T*, int64_t, int64_t);
LOADS(float, 4) LOADS(float, 16) RUNS(float, 4) RUNS(float, 8)
LOADS(bf16_t, 4) LOADS(bf16_t, 8) LOADS(bf16_t, 16) RUNS(bf16_t, 4) RUNS(bf16_t, 8)
}
"""


def test_vector_accesses_claim_element_alignment(tmp_path):
    src, ir = tmp_path / "probe.hip", tmp_path / "probe.ll"
    src.write_text(PROBE)
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", str(src), "-o", str(ir)], check=True,
                   capture_output=True)
    seen = set()
    for fn in re.split(r"^define ", ir.read_text(), flags=re.M)[1:]:
        name = fn.split("(", 1)[0]
        if not re.search(r"pm[0-9]+(loads|runs)I", name):
            continue
        elem = 2 if "bf16" in name else 4
        for kind, width, align in re.findall(r"(load|store) <([24]) x (?:i32|float)>.*addrspace\(1\).*align ([0-9]+)", fn):
            assert int(align) <= elem, (name, kind, width, align)
            seen.add((kind, width, elem))
    assert seen >= {("load", "4", 4), ("load", "4", 2), ("load", "2", 2), ("store", "4", 4), ("store", "4", 2), ("store", "2", 2)}, seen
