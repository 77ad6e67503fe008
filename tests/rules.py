"""The library's route rules (csrc/rules.h, host code without HIP), compiled for the tests: a test that is meant
for one route asserts with them that its sizes still take it."""
import ctypes as C
import os
import subprocess
import tempfile

_HERE = os.path.dirname(os.path.abspath(__file__))
_WRAPPER = """
#include "rules.h"
extern "C" int split_wm(int M, int N, int K, int ks_min, int ks_max) { return san::gemm_split_shape(M, N, K, ks_min, ks_max).wm; }
extern "C" int split_ks(int M, int N, int K, int ks_min, int ks_max) { return san::gemm_split_shape(M, N, K, ks_min, ks_max).ks; }
extern "C" int few_rows(int dtype, int rows, int d) { return san::few_rows_faster(dtype, rows, d); }
extern "C" int skinny(int dtype, int M, int N, int K, int kind, int ks) { return san::gemm_skinny_faster(dtype, M, N, K, kind, ks); }
extern "C" int small_model(int d, int F, int V, int layers, int beam, int batch) { return san::small_model_faster(d, F, V, layers, beam, batch); }
extern "C" int small_model_at(int d, int F, int V, int layers, int beam, int batch, int H, int keys) { return san::small_model_faster(d, F, V, layers, beam, batch, H, (float)keys); }
extern "C" int lds_variant(int M, int N, int K, int kind, int ks, int ragged) { return san::gemm_lds_variant(M, N, K, kind, ks, ragged != 0); }
extern "C" int k_groups(int M, int N, int K, int ks, int partials) { return san::gemm_k_groups(M, N, K, ks, partials != 0); }
extern "C" int kwaves_variant(int M, int N, int K, int ks) { return san::gemm_kwaves_variant(M, N, K, ks); }
extern "C" int cand_n(int N) { return san::gemm_skinny_cand_n(N); }
extern "C" int pick_ksplit(int M, int N, int K, int dtype) { return san::gemm_pick_ksplit(M, N, K, dtype, false); }
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            src, so = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "librules.so")
            with open(src, "w") as fh:
                fh.write(_WRAPPER)
            subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                            os.path.join(_HERE, "..", "paper_1906_11024_amd", "csrc"), src, "-o", so], check=True)
            _lib = C.CDLL(so)
    return _lib
