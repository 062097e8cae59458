"""The bytes that the batch line of bench.py divides by: one Jacobi-CG iteration
is the product and ten passes over vectors (three read and one written by the
update, four read and two written by the direction)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_a_batch_iteration_moves_ten_vectors():
    n, nnz, s = 65 ** 3, 193 ** 3, 16
    assert bench.batch_iteration_bytes(n, nnz, s, 8.0) == bench.spmv_bytes(n, nnz, s, 8.0) + 10 * n * s * 8
    src = open(os.path.join(ROOT, "bench.py")).read()
    assert "k * batch_iteration_bytes(n, nnz, s, 8.0)" in src
