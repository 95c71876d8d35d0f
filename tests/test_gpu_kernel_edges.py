"""GPU parity at the sizes where a kernel's tiles, remainders and dispatch rules can go wrong: one small test per kernel
or dispatch rule, against the CPU oracle.  Tolerances are those of the whole suite (per tensor max|x - ref| / max|ref|):
1e-5 where everything is fp32 (a few hundred roundings of 6e-8 each), 1e-2 where rows are stored as bf16 (2^-9 per
rounding, a handful of storage points deep)."""
import numpy as np
import pytest
import torch

from synth import graphs
from synth.configs import CONFIGS, Workload

from gpu_harness import GpuRun
from helpers import make_problem, max_rel, run_oracle
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


@pytest.mark.parametrize("d0", [1, 3, 5, 67, 201, 301])
def test_raw_features_of_odd_width_become_bf16_rows(d0):
    """fp32 rows of odd width aggregated into bf16 rows: the last vector of a row starts at an odd column, off the 4-byte grid
    of a vector store.  Whole rows and rows cut into pieces, one tile of columns and more."""
    w = Workload("edges", "rmat", 1201, 91, [d0, 32, 24], 4, variant="sage", dtype="bf16", level0_f32=True, n_candidates=14_000)
    p = make_problem(w, chunk_ptr=graphs.ragged_chunks(1201, 4, 3), bias_std=0.05)
    assert np.diff(p.row_ptr).max() > 3 * 64
    _parity(p, TOL_BF16, need_input_grad=False, alias_hist0=True)


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


@pytest.mark.parametrize("widths", [(3, 5), (64, 100), (128, 130), (257, 516)])
def test_fp32_aggregation_of_rows_longer_than_a_piece(widths, monkeypatch):
    """Forward pieces of 256 entries (full batches of 64 entries and of 16 in flight, and their remainders) and the sum of the
    pieces; without source classes, which would cut these rows into shorter ones."""
    monkeypatch.setenv("GNNSTAGE_XCD_CLASSES", "1")
    w = Workload("edges", "rmat", 1201, 91, list(widths), 4, dtype="f32", n_candidates=14_000)
    p = make_problem(w, chunk_ptr=graphs.ragged_chunks(1201, 4, 3), bias_std=0.05, first_stage=False)
    assert np.diff(p.row_ptr).max() > 256 + 64
    _parity(p, TOL_F32)


@pytest.mark.parametrize("dims", [(100, 128), (65, 300), (128, 64)])
def test_fp32_forward_sums_do_not_depend_on_the_chunks(dims):
    """One layer over rows that are never cut: every element is one chain of multiply-adds in a fixed order, whichever
    tile computes it (one chunk: 64 x 64 tiles per workgroup, 33 chunks: 32 x 32), so the results are the same bits."""
    top = []
    for k in (1, 33):
        p = make_problem(small(n=33001, k=k, dims=dims, deg=4.0), bias_std=0.05)
        assert np.diff(p.row_ptr).max() < 128
        top.append(GpuRun(p, alias_hist0=True, need_input_grad=False))
        top[-1].forward()
    assert torch.equal(top[0].cur[1], top[1].cur[1])


def _whole_equals_chunks(p, **kw):
    whole, by_chunk = GpuRun(p, **kw), GpuRun(p, **kw)
    for _ in range(2):  # the second pass finds the scratch of the first
        whole.run()
    for _ in range(2):
        if p.dropout_p > 0:
            by_chunk.stage.gnnstage_set_dropout_seed(p.dropout_seed)
        for pos, c in enumerate(p.order):
            by_chunk.stage.stage_forward_chunk(int(c), pos)
        for c in reversed(list(p.order)):
            by_chunk.stage.stage_backward_chunk(int(c), by_chunk.grad_out[by_chunk.stage.rows(int(c))])
    torch.cuda.synchronize()
    for a, b in zip(whole.cur + [whole.grad_in], by_chunk.cur + [by_chunk.grad_in]):
        assert torch.equal(a, b)
    if whole.grad_h0 is not None:
        assert torch.equal(whole.grad_h0, by_chunk.grad_h0)
    for name in ("dW", "dbias", "d_ln_gamma", "d_ln_beta"):
        for a, b in zip(getattr(whole, name) or [], getattr(by_chunk, name) or []):
            assert (a - b).abs().max() <= 1e-5 * b.abs().max() + 1e-30, name


@pytest.mark.parametrize("variant,dtype,dims,k,kw", [
    ("gcn", "f32", (20, 24, 40, 16, 32), 5, {}), ("gcn", "bf16", (100, 128, 64, 64), 7, {}), ("sage", "f32", (33, 36, 20), 4, {"dropout_p": 0.4}),
    ("sage", "bf16", (64, 128, 128), 3, {}), ("gcnii", "bf16", (64,) * 12, 11, {}), ("gcnii", "f32", (40, 40), 6, {}),
    ("resgcn", "f32", (36,) * 5, 6, {"dropout_p": 0.3}), ("resgcn", "bf16", (128,) * 4, 9, {}), ("gcn", "bf16", (602, 100, 100), 3, {})])
def test_whole_pass_calls_equal_the_chunk_calls(variant, dtype, dims, k, kw):
    """More and fewer chunks than layers, more and fewer than groups of LayerNorm sums, an empty chunk: levels and what flows back
    are the same bits; parameter gradients the same sums in another order (fp32, a few hundred terms)."""
    n = 700
    cp = np.sort(np.concatenate([[0, n], np.random.default_rng(3).integers(1, n, k - 1)])).astype(np.int64)
    if k > 3:
        cp[2] = cp[1]
    p = make_problem(small(n=n, k=k, dims=dims, variant=variant, dtype=dtype, deg=9.0), chunk_ptr=cp, bias_std=0.05, first_stage=False, dropout_seed=5, **kw)
    _whole_equals_chunks(p)


@pytest.mark.parametrize("variant,dims", [("gcn", (64, 128, 128, 256, 256)), ("gcnii", (128,) * 6)])
def test_whole_pass_weight_stationary_products_equal_tiled_ones_of_the_chunks(variant, dims, monkeypatch):
    """Chunks of 100 rows are below the rows from which the weight-stationary product runs, all 700 rows above them: whole passes take
    that kernel, the chunk calls the tiled one; the results are the same bits."""
    monkeypatch.setenv("GNNSTAGE_GEMM_WS_MIN_ROWS", "250")
    _whole_equals_chunks(make_problem(small(n=700, k=7, dims=dims, variant=variant, dtype="bf16", deg=9.0), bias_std=0.05, first_stage=False))


@pytest.mark.parametrize("dtype,n,bound", [("f32", 169343, 1.8e-7), ("bf16", 300000, 1.2e-7)])
def test_bias_gradients_over_all_rows_are_as_exact_as_by_chunk(dtype, n, bound):
    """Column sums of the top layer's gradient rows (transform-first, so that they are a kernel of their own), all rows in one
    sum and chunk by chunk, against 64 bits; errors relative to the root of the sum of squares.  Rows of a split in one chain came
    to 3.3e-7 (f32) and 1.6e-7 (bf16) over all rows; the bounds are what eight chunks one after the other came to, which all rows in
    one sum must not fall behind, and a sixth part for the columns drawn."""
    ring = (np.arange(n + 1, dtype=np.int64) * 2, np.sort(np.stack([np.arange(n), (np.arange(n) + 1) % n], 1), axis=1).astype(np.int32).ravel())
    p = make_problem(small(n=n, k=8, dims=(72, 72, 64), dtype=dtype), graph=ring, bias_std=0.05, first_stage=False, history="random")
    runs = [GpuRun(p), GpuRun(p)]
    assert runs[0].stage.gnnstage_layer_order(1) == 1
    runs[0].run()
    for pos, c in enumerate(p.order):
        runs[1].stage.stage_forward_chunk(int(c), pos)
    for c in reversed(list(p.order)):
        runs[1].stage.stage_backward_chunk(int(c), runs[1].grad_out[runs[1].stage.rows(int(c))])
    for r in runs:
        dY = r.grad_out.double() * (r.cur[2] > 0)
        err = ((r.dbias[1].double() - dY.sum(0)).norm() / dY.square().sum(0).sqrt().norm()).item()
        assert err <= bound


@pytest.mark.parametrize("n,d", [(5196, 1000), (33333, 100), (2077, 3)])
def test_fp32_weight_gradients_over_all_rows_against_64_bits(n, d):
    """x0^T dY and the column sums of dY of one layer over self-loops of weight 1 (the aggregation hands the rows on), errors
    relative to the products of the factors' norms over the root of n.  One chain of additions over all rows of a wave came to
    3.3e-7, 1.6e-7 and 0.9e-7; the bound is a sixth over what chains of 32 products, added up afterwards, come to."""
    loops = (np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32))
    p = make_problem(small(n=n, k=1, dims=(d, d)), graph=loops, bias_std=0.05, history="random")
    p.val[:] = 1.0
    r = GpuRun(p, need_input_grad=False, alias_hist0=True).run()
    x, dY = r.cur[0].double(), r.grad_out.double() * (r.cur[1] > 0)
    err = ((r.dW[0].double() - x.T @ dY).norm() / (x.square().sum(0).sqrt()[:, None] * dY.square().sum(0).sqrt() / n ** 0.5).norm()).item()
    errb = ((r.dbias[0].double() - dY.sum(0)).norm() / dY.square().sum(0).sqrt().norm()).item()
    assert err <= 1.5e-7 and errb <= 1.5e-7


@pytest.mark.parametrize("dtype,width", [("f32", 36), ("bf16", 128)])
def test_layers_with_one_layernorm_gradient_buffer(dtype, width):
    """Tied LayerNorm parameters: the layers' gradients add up in the buffer that they share, of the current rows and, in the part of a
    backward pass that follows its last chunk, of the historical ones."""
    import paper_2308_10087_amd as g
    p = make_problem(small(n=900, k=6, dims=(width,) * 5, variant="resgcn", dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False)
    ref = run_oracle(p)
    r = GpuRun(p)
    dg, db = torch.zeros(width, device=r.device), torch.zeros(width, device=r.device)
    r.stage = g.GnnStage(p.row_ptr, p.col, p.chunk_ptr, p.dims, W=r.W, cur=r.cur, hist=r.hist, dW=r.dW, bias=r.bias, dbias=r.dbias, edge_val=p.val,
                         variant=g.GNNSTAGE_RESGCN, dtype=g.GNNSTAGE_BF16 if p.quant else g.GNNSTAGE_F32, grad_in=r.grad_in, device=r.device,
                         ln_gamma=r.ln_gamma, ln_beta=r.ln_beta, d_ln_gamma=[dg] * 4, d_ln_beta=[db] * 4)
    r.run()
    tol = TOL_BF16 if p.quant else TOL_F32
    assert max_rel(r.np(dg), sum(ref.d_ln_g)) <= tol and max_rel(r.np(db), sum(ref.d_ln_b)) <= tol


@pytest.mark.parametrize("variant,dims,dtype", [
    ("gcn", (24, 24, 24, 24), "f32"), ("gcn", (40, 32, 24, 16), "f32"), ("gcn", (128, 64, 32, 16), "bf16"), ("gcn", (40, 24, 32, 16), "f32"), ("sage", (24, 24, 24, 24), "f32"),
    ("resgcn", (36, 36, 36, 36), "f32"), ("resgcn", (64,) * 4, "bf16")])
@pytest.mark.parametrize("whole", [True, False])
def test_levels_that_are_their_own_history(variant, dims, dtype, whole):
    """What a chunk selects are rows of this pass and what it does not are rows of the last one, also where the aggregation reads a
    table made of them (layers that transform first, ResGCN+).  Three passes against the oracle, all levels but the lowest and then that one too."""
    import paper_2308_10087_amd as g
    for lowest in (1, 0):
        p = make_problem(small(n=500, k=5, dims=dims, variant=variant, dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False, noise_std=0.3)
        ref, r = p.new_oracle(), GpuRun(p)
        for j in range(lowest, p.L):
            ref.hist[j], r.hist[j] = ref.cur[j], r.cur[j]
        ref._refresh()
        r.stage = g.GnnStage(p.row_ptr, p.col, p.chunk_ptr, p.dims, W=r.W, cur=r.cur, hist=r.hist, dW=r.dW, bias=r.bias, dbias=r.dbias, edge_val=p.val,
                             variant=dict(gcn=g.GNNSTAGE_GCN, sage=g.GNNSTAGE_SAGE, resgcn=g.GNNSTAGE_RESGCN)[variant], dtype=g.GNNSTAGE_BF16 if p.quant else g.GNNSTAGE_F32,
                             grad_in=r.grad_in, device=r.device, ln_gamma=r.ln_gamma, ln_beta=r.ln_beta, d_ln_gamma=r.d_ln_gamma, d_ln_beta=r.d_ln_beta)
        tol = TOL_BF16 if p.quant else TOL_F32
        first = r.cur[0].clone()
        for i in range(3):
            fresh = first * (1.0 + 0.5 * i)  # (exact in bf16 for these factors or rounded alike on both sides)
            ref.begin_pass()
            for pos, c in enumerate(p.order):
                rows = r.stage.rows(int(c))
                if lowest == 0 and not whole:  # a chunk's input arrives with the chunk
                    r.cur[0][rows] = fresh[rows]
                    ref.cur[0][rows] = r.np(fresh[rows])
                ref.forward_chunk(int(c))
                if not whole:
                    r.stage.stage_forward_chunk(int(c), pos)
            if whole:
                r.forward()
            torch.cuda.synchronize()
            for j in range(1, p.L + 1):
                assert max_rel(r.np(r.cur[j]), ref.cur[j]) <= tol, (lowest, i, j)
                r.cur[j].copy_(torch.from_numpy(ref.cur[j]).to(r.cur[j].dtype))  # one side's decisions, and rows of the last pass
        ref.backward_pass(p.grad_out)
        r.backward()
        torch.cuda.synchronize()
        assert max_rel(r.np(r.grad_in), ref.grad_in) <= tol
        for j in range(p.L):
            if not r.stage.gnnstage_layer_order(j):
                assert max_rel(r.np(r.dW[j]), ref.dW[j]) <= tol
            if variant == "resgcn":
                assert max_rel(r.np(r.d_ln_gamma[j]), ref.d_ln_g[j]) <= tol and max_rel(r.np(r.d_ln_beta[j]), ref.d_ln_b[j]) <= tol


def test_passes_that_cannot_run_whole_behave_like_the_chunk_calls():
    """Levels that are their own history (what is not selected are rows of the last pass), and orders that are none."""
    import paper_2308_10087_amd as g
    p = make_problem(small(n=500, k=5, dims=(24, 24, 24, 24), deg=9.0), bias_std=0.05, first_stage=False)
    runs = [GpuRun(p), GpuRun(p)]
    for r in runs:
        r.hist[1:] = r.cur[1:3]
        r.stage = g.GnnStage(p.row_ptr, p.col, p.chunk_ptr, p.dims, W=r.W, cur=r.cur, hist=r.hist, dW=r.dW, bias=r.bias, dbias=r.dbias, edge_val=p.val,
                             variant=g.GNNSTAGE_GCN, dtype=g.GNNSTAGE_F32, grad_in=r.grad_in, device=r.device)
    for _ in range(2):
        runs[0].run()
        for pos, c in enumerate(p.order):
            runs[1].stage.stage_forward_chunk(int(c), pos)
        for c in reversed(list(p.order)):
            runs[1].stage.stage_backward_chunk(int(c), runs[1].grad_out[runs[1].stage.rows(int(c))])
    torch.cuda.synchronize()
    for a, b in zip(runs[0].cur + [runs[0].grad_in], runs[1].cur + [runs[1].grad_in]):
        assert torch.equal(a, b)
    st = runs[0].stage
    with pytest.raises(g.GnnStageError) as e:
        st.forward_pass([0, 1, 1, 2, 3])
    assert e.value.code == -3
    st.forward_pass([0, 1, 2, 3, 4])
    with pytest.raises(g.GnnStageError) as e:
        st.backward_pass([1, 0, 2, 3, 4][::-1], runs[0].grad_out)
    assert e.value.code == -3


@pytest.mark.parametrize("n,k,d,dtype,bound", [(8_000_000, 32, 64, "f32", 3.4e-7), (8_000_000, 9, 100, "f32", 3.4e-7), (4_000_000, 9, 512, "bf16", 3.4e-7)])
def test_layernorm_gradients_over_all_rows_against_64_bits(n, k, d, dtype, bound):
    """Rows over self-loops of weight 1 behind a unit weight, every activation above zero: the gradient of a LayerNorm's offset is the sum
    of the upstream rows, that of its scale their products with the normalised rows.  Errors relative to the root of the sum of
    squares: a wavefront's rows in one chain came to 5e-7 - 6e-7.  A chain of m terms of random sign adds the root of m / 2
    roundings of 0.4 x 2^-23 or less; 32 rows, 31 chains, 4 wavefronts, 16 parts of 16 each, 8 groups make 107: 3.4e-7."""
    import paper_2308_10087_amd as g
    dev, T = "cuda:0", torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device=dev).manual_seed(n + k)
    x, up = (torch.randn((n, d), generator=gen, device=dev).to(T) for _ in range(2))
    dg, db, dbias = (torch.zeros(d, device=dev) for _ in range(3))
    st = g.GnnStage(np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.arange(k + 1, dtype=np.int64) * n // k, [d, d], W=[torch.eye(d, device=dev).to(T)],
                    cur=[x, torch.zeros_like(x)], hist=[x.clone()], dW=[torch.zeros((d, d), device=dev)], bias=[torch.zeros(d, device=dev)], dbias=[dbias],
                    edge_val=np.ones(n, np.float32), variant=g.GNNSTAGE_RESGCN, dtype=g.GNNSTAGE_F32 if dtype == "f32" else g.GNNSTAGE_BF16,
                    grad_in=torch.zeros_like(x), ln_gamma=[torch.ones(d, device=dev)], ln_beta=[torch.full((d,), 20.0, device=dev)], d_ln_gamma=[dg], d_ln_beta=[db], device=dev)
    st.forward_pass(np.arange(k))
    st.backward_pass(np.arange(k), up)
    torch.cuda.synchronize()
    sums = torch.zeros((4, d), dtype=torch.float64, device=dev)
    for i in range(0, n, 500_000):
        xd, ud = x[i:i + 500_000].double(), up[i:i + 500_000].double()
        terms = (xd - xd.mean(1, keepdim=True)) / (xd.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt() * ud
        sums += torch.stack([ud.sum(0), ud.square().sum(0), terms.sum(0), terms.square().sum(0)])
    for got, total, squares in ((db, sums[0], sums[1]), (dg, sums[2], sums[3])):
        assert ((got.double() - total) / squares.sqrt()).square().mean().sqrt().item() <= bound
