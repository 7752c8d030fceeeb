"""Which kernels the float32 GEMMs of the GPU tests' sizes take, from the library's own plan (host code, compiled here)."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2603_04135_amd import build as B
from test_gpu_head import FP32_DW_TILES, FP32_SIZES

BIG, MID, DIRECT_4, DIRECT_8 = range(4)
SOURCE = """
#include "gemm_f32_plan.h"
extern "C" void plan(int M, int N, int K, long long room, int cus, int* out) {
    const dppo::F32Plan p = dppo::plan_gemm_f32(M, N, K, room, cus);
    out[0] = p.kernel;
    out[1] = p.parts;
}
extern "C" int max_parts(long long K) { return dppo::gemm_f32_max_parts(K); }
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans(tokens, D, V) -> {logits, dH, dW: (kernel, parts)} of a loss call whose tokens are one chunk."""
    d = tmp_path_factory.mktemp("plan")
    src, so = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-shared", "-fPIC", "-I", B.CSRC, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.plan.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong, ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    lib.max_parts.argtypes = [ctypes.c_longlong]

    def pick(M, N, K, room):
        out = (ctypes.c_int * 2)()
        lib.plan(M, N, K, room, 256, out)
        return tuple(out)

    def get(tokens, D, V):
        rows, Vp = -(-tokens // 256) * 256, -(-V // 256) * 256
        parts = min(Vp // D, lib.max_parts(V))                       # sums of all rows that the scratch of dH holds
        return dict(logits=pick(tokens, V, D, 1), dH=pick(tokens, D, V, parts * rows // tokens if parts > 1 else 1),
                    dW=pick(V, D, tokens, 1))

    return get


def test_sizes_of_the_error_test_take_every_kernel_in_every_gemm(plans):
    taken = {gemm: set() for gemm in ("logits", "dH", "dW")}
    split = set()
    for size in FP32_SIZES:
        for gemm, (kernel, parts) in plans(*size).items():
            taken[gemm].add(kernel)
            if parts > 1:
                split.add(kernel)
    for gemm, kernels in taken.items():
        assert kernels == {BIG, MID, DIRECT_4, DIRECT_8}, (gemm, kernels)
    assert split == {BIG, MID, DIRECT_4, DIRECT_8}
    assert all(k == BIG for k, _ in plans(*FP32_SIZES[-1]).values())


def test_sizes_of_the_few_token_tests_take_three_kernels_of_dw(plans):
    for tokens in (1, 2, 3, 40):
        assert [plans(tokens, D, V)["dW"][0] for D, V in FP32_DW_TILES] == [DIRECT_4, MID, BIG]
