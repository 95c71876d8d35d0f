"""GPU parity at the sizes where a kernel's tiles, remainders and dispatch rules can go wrong: one small test per kernel
or dispatch rule, against the CPU oracle.  Tolerances are those of the whole suite (per tensor max|x - ref| / max|ref|):
1e-5 where everything is fp32 (a few hundred roundings of 6e-8 each), 1e-2 where rows are stored as bf16 (2^-9 per
rounding, a handful of storage points deep)."""
import numpy as np
import pytest

from synth import graphs
from synth.configs import CONFIGS, Workload

from helpers import make_problem
from test_gpu_parity import TOL_BF16, TOL_F32, _parity, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,widths", [
    ("f32", (1, 3, 4, 5)), ("f32", (63, 64, 65, 61)), ("f32", (127, 128, 129, 131)), ("f32", (255, 256, 257, 259)), ("f32", (512, 515)),
    ("bf16", (2, 6, 10, 12)), ("bf16", (100, 126, 130, 134)), ("bf16", (250, 254, 258, 262)), ("bf16", (510, 514, 518))])
def test_vector_alu_aggregation_at_tile_edges(dtype, widths):
    """Widths on both sides of the 16-, 32- and 64-lane tiles, rows that end inside a 16-byte vector, and rows long enough
    to be cut into pieces (power-law graph), forward and transposed."""
    w = Workload("edges", "rmat", 1201, 91, list(widths), 4, dtype=dtype, n_candidates=14_000)
    p = make_problem(w, chunk_ptr=graphs.ragged_chunks(1201, 4, 3), bias_std=0.05, first_stage=False)
    assert np.diff(p.row_ptr).max() > 3 * 32
    _parity(p, TOL_F32 if dtype == "f32" else TOL_BF16)


@pytest.mark.parametrize("dims,n,k,variant,drop", [
    ((1, 2, 3, 5), 301, 3, "gcn", 0.0), ((3, 4, 1), 130, 2, "sage", 0.3), ((15, 16, 17, 33), 517, 4, "gcn", 0.5),
    ((31, 32, 36, 65), 260, 2, "sage", 0.5), ((100, 100, 100), 700, 5, "gcnii", 0.0), ((67, 67), 411, 3, "resgcn", 0.0),
    ((300, 130, 72), 90, 3, "gcn", 0.0),
    ((70, 132, 260), 12001, 1, "gcn", 0.5), ((68, 68), 33001, 1, "gcnii", 0.0)])  # 64 x 64 tiles: 512 and more of them
def test_fp32_products_at_tile_edges(dims, n, k, variant, drop):
    """Rows, columns and reduction lengths on both sides of the 16-, 32- and 64-wide tiles, partial reduction groups,
    operands narrower than a 16-byte vector, chunks of a few rows; every epilogue, dropout in the forward one."""
    w = small(n=n, k=k, dims=dims, variant=variant, deg=3.0)
    cp = None if k == 1 else graphs.ragged_chunks(n, k, 12)
    p = make_problem(w, chunk_ptr=cp, bias_std=0.05, dropout_p=drop, dropout_seed=99, first_stage=False)
    _parity(p, TOL_F32)
