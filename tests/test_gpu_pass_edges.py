"""Whole passes at the sizes where their launches go wrong: more chunks than a mask word has bits, rows of every short length,
products whose epilogue reads another operand, weight gradients that must not share a launch.  Tolerances are those of the whole
suite (1e-5 where everything is fp32, 1e-2 where rows are stored as bf16) or equal bits."""
import numpy as np
import pytest
import torch

from gpu_harness import GpuRun, GpuTrainRun
from synth.configs import Workload
from helpers import make_problem, make_train_problem, max_rel, run_oracle
from test_gpu_kernel_edges import _whole_equals_chunks
from test_gpu_parity import TOL_BF16, TOL_F32, _parity, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [64, 65, 130])
@pytest.mark.parametrize("variant,dtype,dims", [
    ("gcn", "bf16", (128, 256, 128)), ("resgcn", "bf16", (128,) * 3), ("sage", "bf16", (100, 102, 64)), ("gcn", "f32", (36, 40, 24))])
def test_chunks_beyond_one_mask_word(k, variant, dtype, dims, monkeypatch):
    """64 chunks are one word of selects, more are a table: short rows, whole rows and pieces of long ones on both kernels."""
    monkeypatch.setenv("GNNSTAGE_CLASS_MIN_ROW", "24")
    p = make_problem(small(n=1111, k=k, dims=dims, variant=variant, dtype=dtype, deg=14.0), bias_std=0.05, first_stage=False, noise_std=0.3)
    _whole_equals_chunks(p)
    _parity(p, TOL_F32 if dtype == "f32" else TOL_BF16)


def _graph_of_lengths(n, lengths, seed):
    """Row i has lengths[i % len] entries, columns drawn without repetition; the transposed rows are of all short lengths too."""
    rng = np.random.default_rng(seed)
    ln = np.resize(lengths, n)
    row_ptr = np.concatenate([[0], np.cumsum(ln)]).astype(np.int64)
    step = rng.integers(1, max(2, n // 40), n)  # row i: an arithmetic progression from a random start, short enough not to close
    k = np.arange(row_ptr[-1]) - np.repeat(row_ptr[:-1], ln)
    col = (np.repeat(rng.integers(0, n, n), ln) + k * np.repeat(step, ln)) % n
    order = np.lexsort((col, np.repeat(np.arange(n), ln)))
    return row_ptr, col[order].astype(np.int32)


@pytest.mark.parametrize("n,k", [(1283, 3), (61, 1), (5, 2)])
@pytest.mark.parametrize("dims", [(128, 128, 128), (64, 256, 128), (512, 128)])
def test_short_rows_are_the_bits_of_whole_waves(n, k, dims, monkeypatch):
    """Rows of 1 .. 18 entries, four to a wave up to 16: the bits of a row to a wave, whatever rows are left for the last wave."""
    graph = _graph_of_lengths(n, np.minimum(n - 1, [1, 16, 2, 15, 17, 4, 3, 8, 5, 18, 9, 12, 7, 16, 16, 13, 1]), 7)
    p = make_problem(small(n=n, k=k, dims=dims, dtype="bf16"), graph=graph, bias_std=0.05, first_stage=False, noise_std=0.3)
    p.val[:] = np.random.default_rng(2).uniform(0.02, 0.3, p.val.size)  # (of any graph: not from its degrees)
    runs = []
    for most in ("0", "4", "16"):
        monkeypatch.setenv("GNNSTAGE_SHORT_ROW", most)
        runs.append(GpuRun(p).run())
    for r in runs[1:]:
        for a, b in zip(r.cur + [r.grad_in] + r.dW, runs[0].cur + [runs[0].grad_in] + runs[0].dW):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n,d", [(4090, 64), (4097, 64), (8190, 128), (8193, 128)])
def test_short_rows_go_four_to_a_wave_from_64_per_column_on(n, d, monkeypatch):
    """On both sides of the number of short rows from which they share waves: the bits of both forms."""
    p = make_problem(small(n=n, k=1, dims=(d, d), dtype="bf16"), graph=_graph_of_lengths(n, np.array([1, 16, 2, 15, 4, 3, 8, 5, 9, 12, 7, 13]), 7), first_stage=False, noise_std=0.3)
    p.val[:] = np.random.default_rng(2).uniform(0.02, 0.3, p.val.size)
    runs = []
    for most in (None, "0", "16"):
        monkeypatch.setenv("GNNSTAGE_SHORT_ROW", most) if most else monkeypatch.delenv("GNNSTAGE_SHORT_ROW", raising=False)
        runs.append(GpuRun(p).run())
    for r in runs[1:]:
        for a, b in zip(r.cur + [r.grad_in] + r.dW, runs[0].cur + [runs[0].grad_in] + runs[0].dW):
            assert torch.equal(a, b)


def test_short_rows_of_tables_beyond_the_caches(monkeypatch):
    """Tables of over 256 MB: rows of up to 4 entries on the vector ALU, four to a wave.  Against a row to a wave: weights in fp32 instead
    of two bf16 parts, another order of at most 4 products, so a bf16 rounding of the result apart."""
    n = 1_060_001
    graph = _graph_of_lengths(n, np.array([1, 4, 2, 5, 3, 4, 6, 0]), 3)
    p = make_problem(small(n=n, k=3, dims=(128, 128), dtype="bf16"), graph=graph, first_stage=False)
    p.val[:] = np.random.default_rng(2).uniform(0.02, 0.3, p.val.size)
    runs = []
    for most in ("0", None):
        monkeypatch.setenv("GNNSTAGE_SHORT_ROW", most) if most else monkeypatch.delenv("GNNSTAGE_SHORT_ROW")
        runs.append(GpuRun(p))
        runs[-1].forward()
    runs[1].cur[1].copy_(runs[0].cur[1])  # (both decide on the same levels)
    for r in runs:
        r.backward()
    torch.cuda.synchronize()
    for a, b in ((runs[1].grad_in, runs[0].grad_in), (runs[1].dW[0], runs[0].dW[0])):
        assert (a.float() - b.float()).abs().max() <= TOL_BF16 * b.float().abs().max()
    runs[1].forward()
    torch.cuda.synchronize()
    a, b = runs[1].cur[1], runs[0].cur[1]
    assert (a.float() - b.float()).abs().max() <= TOL_BF16 * b.float().abs().max()


@pytest.mark.parametrize("width", [64, 128, 256])
@pytest.mark.parametrize("n,k", [(513, 1), (1031, 4), (37, 2)])
def test_identity_mapping_in_the_weight_stationary_product(width, n, k, monkeypatch):
    """GCNII products from every row count on in the weight-stationary kernel (the identity mapping's other operand is the A tile in LDS,
    grad_h0 comes half before and half behind the products): the bits of the tiled kernel, and the oracle's values."""
    p = make_problem(small(n=n, k=k, dims=(width,) * 4, variant="gcnii", dtype="bf16", deg=min(9.0, n / 8)), first_stage=False, noise_std=0.3)
    runs = []
    for least in ("1", "1000000"):
        monkeypatch.setenv("GNNSTAGE_GEMM_WS_MIN_ROWS", least)
        runs.append(GpuRun(p).run())
    a, b = runs
    for x, y in zip(a.cur + [a.grad_in, a.grad_h0], b.cur + [b.grad_in, b.grad_h0]):
        assert torch.equal(x, y)
    monkeypatch.setenv("GNNSTAGE_GEMM_WS_MIN_ROWS", "1")
    _parity(p, TOL_BF16)


@pytest.mark.parametrize("dtype,width", [("f32", 36), ("bf16", 128)])
def test_layers_with_one_weight_gradient_buffer(dtype, width):
    """Tied weights: layers of one width go to one launch of weight gradients unless they share a buffer, which then holds their sum."""
    import paper_2308_10087_amd as g
    p = make_problem(small(n=900, k=6, dims=(width,) * 5, dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False)
    ref = run_oracle(p)
    r = GpuRun(p)
    dW, db = torch.zeros((width, width), device=r.device), torch.zeros(width, device=r.device)
    r.stage = g.GnnStage(p.row_ptr, p.col, p.chunk_ptr, p.dims, W=r.W, cur=r.cur, hist=r.hist, dW=[dW] * 4, bias=r.bias, dbias=[db] * 4, edge_val=p.val,
                         variant=g.GNNSTAGE_GCN, dtype=g.GNNSTAGE_BF16 if p.quant else g.GNNSTAGE_F32, grad_in=r.grad_in, device=r.device)
    r.forward()
    torch.cuda.synchronize()
    for j in range(1, 5):
        r.cur[j].copy_(torch.from_numpy(ref.cur[j]).to(r.cur[j].dtype))  # ReLU decisions of one side
    r.backward()
    torch.cuda.synchronize()
    tol = TOL_BF16 if p.quant else TOL_F32
    assert max_rel(r.np(dW), sum(ref.dW)) <= tol and max_rel(r.np(db), sum(ref.db)) <= tol


def test_tied_parameters_are_updated_one_after_the_other():
    """An epoch's update of one parameter listed twice is two updates, the second from the weights of the first; 35 parameters take two
    launches.  One SGD step without gradients other than a constant per entry: p <- p (1 - lr wd) per listing."""
    import paper_2308_10087_amd as g
    tp = make_train_problem(n=600, stage_dims=((16, 16),), K=3)
    run = GpuTrainRun(tp, optimizer="sgd", lr=0.5, weight_decay=0.25)
    extra = [torch.full((300 + i,), 2.0, device="cuda:0") for i in range(35)]
    zeros = [torch.zeros_like(x) for x in extra]
    run.params += [(x, None, z) for x, z in zip(extra, zeros)] + [(extra[3], None, zeros[3])]
    run.trainer = g.GnnTrainer(run.stages, head_W=run.head_W, head_b=run.head_b, head_dW=run.head_dW, head_db=run.head_db, labels=run.labels,
                               train_mask=run.mask, params=run.params, device="cuda:0", optimizer=g.GNNTRAIN_SGD, lr=0.5, beta1=0.9, beta2=0.999,
                               eps=1e-8, weight_decay=0.25, shuffle=True, seed=0, alpha_hist=1)
    run.epoch(0)
    torch.cuda.synchronize()
    for i, x in enumerate(extra):
        assert torch.equal(x, torch.full_like(x, 2.0 * (0.875 ** (2 if i == 3 else 1)))), i


@pytest.mark.parametrize("variant,dtype,dims", [("gcn", "bf16", (128, 256, 128)), ("gcn", "f32", (36, 40, 24)), ("resgcn", "bf16", (128,) * 3)])
@pytest.mark.parametrize("k,blocks", [(7, 150), (70, 100), (5, 1)])
def test_a_layer_that_is_too_much_for_one_launch(k, blocks, variant, dtype, dims, monkeypatch):
    """A launch takes as many chunks as keep below the most workgroups, one at least: the bits of the chunk calls."""
    monkeypatch.setenv("GNNSTAGE_LAUNCH_BLOCKS", str(blocks))
    monkeypatch.setenv("GNNSTAGE_CLASS_MIN_ROW", "24")
    _whole_equals_chunks(make_problem(small(n=1111, k=k, dims=dims, variant=variant, dtype=dtype, deg=14.0), bias_std=0.05, first_stage=False, noise_std=0.3))


@pytest.mark.parametrize("variant,dtype,dims,dense", [
    ("gcn", "bf16", (128, 256, 128), True), ("resgcn", "bf16", (128,) * 3, True), ("sage", "bf16", (128, 128), True), ("gcn", "f32", (36, 40, 24), False), ("gcnii", "bf16", (64,) * 3, False)])
@pytest.mark.parametrize("k,room", [(7, 0), (7, 300000), (70, 0), (70, 300000)])
def test_a_layer_whose_partial_sums_have_no_room_together(k, room, variant, dtype, dims, dense, monkeypatch):
    """A layer in several launches, one behind the other through the same scratch: the bits of the chunk calls, the oracle's values."""
    monkeypatch.setenv("GNNSTAGE_PARTIAL_ROOM", str(room))
    monkeypatch.setenv("GNNSTAGE_CLASS_MIN_ROW", "24")
    if dense:
        monkeypatch.setenv("GNNSTAGE_DENSE_MIN_ENTRIES", "0")
        monkeypatch.setenv("GNNSTAGE_DENSE_MIN_SHARE", "0")
        monkeypatch.setenv("GNNSTAGE_DENSE_MIN_NNZ", "12")
    w = Workload("room", "rmat", 1201, 91, list(dims), k, variant=variant, dtype=dtype, n_candidates=20_000)
    p = make_problem(w, bias_std=0.05, first_stage=False, noise_std=0.3)
    assert (GpuRun(p).stage.gnnstage_dense_entries(True) > 0) == dense
    _whole_equals_chunks(p)
    _parity(p, TOL_F32 if dtype == "f32" else TOL_BF16)


def test_more_elements_than_a_grid_has_threads():
    """4.29 M rows of 1002 bf16 columns: dropout and the ReLU derivative over all rows take two launches; the
    bits of launches over a chunk."""
    import paper_2308_10087_amd as g
    n, d0, d1, K, dev = 4_290_001, 1008, 1002, 3, "cuda:0"
    assert n * d1 > 2 ** 32
    rows = lambda d, s: torch.randn((5003, d), generator=torch.Generator(device=dev).manual_seed(s), device=dev).to(torch.bfloat16).repeat(n // 5003 + 1, 1)[:n]
    cur = [rows(d0, 1), torch.zeros((n, d1), dtype=torch.bfloat16, device=dev)]
    W, bias = (torch.randn((d0, d1), device=dev) / 30).to(torch.bfloat16), torch.randn(d1, device=dev) / 10
    dW, dbias, grad_in = torch.zeros((d0, d1), device=dev), torch.zeros(d1, device=dev), torch.zeros((n, d0), dtype=torch.bfloat16, device=dev)
    st = g.GnnStage(np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.arange(K + 1, dtype=np.int64) * n // K, [d0, d1], W=[W], cur=cur,
                    hist=[cur[0]], dW=[dW], bias=[bias], dbias=[dbias], variant=g.GNNSTAGE_GCN, dtype=g.GNNSTAGE_BF16, grad_in=grad_in, device=dev, dropout_p=0.5)
    assert st.gnnstage_layer_order(0) == 1
    grad_out = rows(d1, 2)
    st.forward_pass([0, 1, 2])
    st.backward_pass([0, 1, 2], grad_out)
    level, back = cur[1].clone(), grad_in.clone()
    for x in (cur[1], grad_in):
        x.zero_()
    for pos in range(K):
        st.stage_forward_chunk(pos, pos)
    for c in reversed(range(K)):
        st.stage_backward_chunk(c, grad_out[st.rows(c)])
    torch.cuda.synchronize()
    assert torch.equal(level, cur[1]) and torch.equal(back, grad_in)
    kept = (level[-4000:] > 0).float().mean().item()  # half of what passes ReLU
    assert 0.2 < kept < 0.3


@pytest.mark.parametrize("dtype,width", [("f32", 36), ("bf16", 128)])
@pytest.mark.parametrize("k,first", [(1, 0), (2, 1), (9, 0), (9, 4), (9, 8), (32, 13)])
def test_history_that_nobody_reads_may_hold_anything(k, first, dtype, width):
    """The rows of the chunk that comes first in the order are never read as historical ones, also not by the LayerNorm parameters'
    gradients: rows that hold no numbers there leave every result as it is."""
    p = make_problem(small(n=900, k=k, dims=(width,) * 4, variant="resgcn", dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False)
    p.order = np.roll(np.arange(k, dtype=np.int32), -first)
    runs = [GpuRun(p), GpuRun(p)]
    for h in runs[1].hist:
        h[runs[1].stage.rows(first)] = float("nan")
    for r in runs:
        r.run()
    a, b = runs
    for x, y in zip(a.cur + [a.grad_in] + a.dW + a.d_ln_gamma + a.d_ln_beta, b.cur + [b.grad_in] + b.dW + b.d_ln_gamma + b.d_ln_beta):
        assert torch.equal(x, y)
    ref = run_oracle(p)
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    assert max(max_rel(b.np(x), y) for x, y in zip(b.d_ln_gamma + b.d_ln_beta, ref.d_ln_g + ref.d_ln_b)) <= tol


@pytest.mark.parametrize("dtype,width", [("f32", 36), ("bf16", 128)])
@pytest.mark.parametrize("k,first", [(2, 1), (9, 4)])
def test_timed_passes_take_the_historical_part_of_layernorm_gradients(k, first, dtype, width):
    """While launches are timed the historical rows go chunk by chunk behind a backward pass, all chunks but the first of the order."""
    p = make_problem(small(n=900, k=k, dims=(width,) * 4, variant="resgcn", dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False)
    p.order = np.roll(np.arange(k, dtype=np.int32), -first)
    r = GpuRun(p)
    r.stage.gnnstage_profile_enable(True)
    r.run()
    ref = run_oracle(p)
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    assert max(max_rel(r.np(x), y) for x, y in zip(r.d_ln_gamma + r.d_ln_beta, ref.d_ln_g + ref.d_ln_b)) <= tol


@pytest.mark.parametrize("variant,dims,dtype", [("gcn", (40, 24, 32), "f32"), ("gcn", (256, 128, 64), "bf16"), ("resgcn", (36,) * 3, "f32"), ("resgcn", (64,) * 3, "bf16")])
def test_a_level_0_that_is_its_own_history(variant, dims, dtype):
    """Of a stage that hands a gradient down: whole passes make one table of it, chunk calls two; the same bits, the oracle's values."""
    p = make_problem(small(n=700, k=5, dims=dims, variant=variant, dtype=dtype, deg=9.0), bias_std=0.05, first_stage=False, noise_std=0.3)
    _whole_equals_chunks(p, alias_hist0=True)
    p.hist[0] = p.x0
    _parity(p, TOL_F32 if dtype == "f32" else TOL_BF16, alias_hist0=True)
