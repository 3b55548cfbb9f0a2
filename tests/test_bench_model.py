"""The bytes that the benchmark charges the vectorial solve with, against the streams of its kernels."""

import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_vectorial_bytes_count_the_streams_of_the_kernels():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    # fields read and written by k_vpupd, k_vpost<DOT_V>, k_vsupd, k_vpost<DOT_T> and k_vxr
    vector = (3 + 1) + (3 + 1) + (2 + 1) + (2 + 1) + (5 + 2)
    conv = 1 + 2 + 2 + 2 + 2 + 1       # row transforms in and out (2 n planes), the planes between (rho = 2)
    N = 32 ** 3
    assert bench.vec_bytes_per_tx_iteration(32, 64, N) == 3 * N * 16 * (2 * conv + vector)
    # the adjoint writes each convolution's input (k_vpre reads one field and writes one)
    assert bench.vec_bytes_per_tx_iteration(32, 64, N, adjoint=True) == 3 * N * 16 * (2 * (conv + 2) + vector)
