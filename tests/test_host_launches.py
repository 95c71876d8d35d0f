"""What the library launches, on a CPU: its host side runs in a process of its own over host_launches.c, which lists kernel
launches instead of running them."""
import ctypes as C
import json
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "libhostlaunches.so")
    subprocess.run(["cc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host_launches.c"), "-o", so], check=True)
    return so


def _child(runtime, what, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, what, json.dumps(args)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


# ---- in the child -----------------------------------------------------------------------------------------------
class _Launch(C.Structure):
    _fields_ = [("name", C.c_char_p), ("grid", C.c_uint32 * 3), ("args", C.c_uint8 * 256)]


class _Stage:
    """A stage handle over host buffers (values never matter: nothing is computed)."""

    def __init__(self, variant, dims, K, n=400, tied=False, bf16=False, dropout_p=0.0, own_history=False):
        import paper_2308_10087_amd as g
        from paper_2308_10087_amd import binding
        self.g, self.lib = g, binding.lib
        L, two = len(dims) - 1, 2 if variant == "sage" else 1  # GraphSage: [W_self ; W_neigh]
        col = (np.arange(n)[:, None] + np.array([0, 1, 7, 50])) % n
        row_ptr, col = np.arange(n + 1, dtype=np.int64) * 4, np.sort(col, axis=1).astype(np.int32).ravel()
        chunk_ptr, dims = (np.arange(K + 1, dtype=np.int64) * n) // K, np.asarray(dims, np.int32)
        rows = lambda ws: [np.zeros((n, int(w)), np.float32) for w in ws]
        vec = lambda ws: [np.zeros(int(w), np.float32) for w in ws]
        self.keep = dict(row_ptr=row_ptr, col_idx=col, chunk_ptr=chunk_ptr, dims=dims)
        lists = dict(W=[np.zeros((two * int(dims[j]), int(dims[j + 1])), np.float32) for j in range(L)], cur=rows(dims), hist=rows(dims[:-1]),
                     dW=[np.zeros((two * int(dims[j]), int(dims[j + 1])), np.float32) for j in range(L)], bias=vec(dims[1:]), dbias=vec(dims[1:]))
        if own_history:
            lists["hist"][0] = lists["cur"][0]
        if variant == "resgcn":
            lists.update(ln_gamma=vec(dims[:-1]), ln_beta=vec(dims[:-1]))
            for i, name in enumerate(("d_ln_gamma", "d_ln_beta")):
                lists[name] = [np.zeros(int(dims[0]), np.float32)] * L if tied else vec(dims[:-1])
        d = binding.gnnstage_desc()
        d.n_vertices, d.nnz, d.n_chunks, d.n_layers = n, len(col), K, L
        for name, a in self.keep.items():
            setattr(d, name, a.ctypes.data)
        for name, a in lists.items():
            p = (C.c_void_p * len(a))(*[x.ctypes.data for x in a])
            self.keep["list " + name] = (a, p)
            setattr(d, name, C.cast(p, C.c_void_p))
        self.grad_in, self.grad_out = np.zeros((n, int(dims[0])), np.float32), np.zeros((n, int(dims[-1])), np.float32)
        d.dropout_p = dropout_p
        d.variant, d.dtype, d.need_input_grad, d.grad_in, d.ln_eps = dict(gcn=0, sage=2, resgcn=3)[variant], g.GNNSTAGE_BF16 if bf16 else g.GNNSTAGE_F32, 1, self.grad_in.ctypes.data, 1e-5
        size = self.lib.gnnstage_workspace_size(C.byref(d))
        self.ws = np.zeros(size + 256, np.uint8)
        d.workspace, d.workspace_bytes = (self.ws.ctypes.data + 255) // 256 * 256, size
        self.h = C.c_void_p(None)
        rc = self.lib.gnnstage_create(C.byref(d), C.byref(self.h))
        assert rc == 0, (rc, self.lib.gnnstage_last_error(None))
        self.K, self.L, self.chunk_ptr, self.order = K, L, chunk_ptr, np.arange(K, dtype=np.int32)[::-1].copy()

    def forward(self):
        return self.lib.gnnstage_forward_pass(self.h, self.order.ctypes.data, self.K, None)

    def backward(self):
        return self.lib.gnnstage_backward_pass(self.h, self.order.ctypes.data, self.K, self.grad_out.ctypes.data, None)

    def by_chunk(self):
        for pos, k in enumerate(self.order):
            assert self.lib.stage_forward_chunk(self.h, int(k), pos, None) == 0
        for k in self.order[::-1]:
            assert self.lib.stage_backward_chunk(self.h, int(k), self.grad_out[self.chunk_ptr[k]:].ctypes.data, None) == 0


def _launches(rt):
    return [rt.host_launch(i).contents for i in range(rt.host_launches())]


def _ln_reduces(rt, tied, whole, timed):
    """Destinations (gamma, beta) of every launch that adds up LayerNorm parameter gradients, a list per launch."""
    st = _Stage("resgcn", [32] * 5, 6, tied=tied)
    assert st.lib.gnnstage_profile_enable(st.h, int(timed)) == 0
    rt.host_clear(-1)
    if whole:
        assert st.forward() == 0 and st.backward() == 0
    else:
        st.by_chunk()
    out = []
    for l in _launches(rt):
        if b"ln_param_reduce" in l.name:
            a = np.frombuffer(bytes(l.args), np.uint64).reshape(8, 4)  # per plane: partial, (n_parts, d), dgamma, dbeta
            out.append([int(x) for x in a[:l.grid[2], 2:].ravel()])
    return out


def _long_products(rt, n, K):
    """Grids of the weight-stationary products of a forward pass over one transform-first bf16 layer, 256 -> 200."""
    st = _Stage("gcn", [256, 200], K, n=n, bf16=True)
    rt.host_clear(-1)
    assert st.forward() == 0
    return [list(l.grid) for l in _launches(rt) if b"gemm_nt_bf16_ws" in l.name]


def _forward_kinds(rt, variant, dims, K):
    """Aggregations (a) and products (p) of a forward pass in the order of their launches."""
    st = _Stage(variant, dims, K)
    rt.host_clear(-1)
    assert st.forward() == 0
    return "".join("a" if b"spmm" in l.name else "p" if b"gemm_nt" in l.name else "" for l in _launches(rt))


def _tables(rt, variant, dims, whole):
    """Launches of a forward pass that make a table of a level's rows, where level 0 is its own history."""
    st = _Stage(variant, dims, 6, own_history=True)
    rt.host_clear(-1)
    if whole:
        assert st.forward() == 0
    else:
        for pos, k in enumerate(st.order):
            assert st.lib.stage_forward_chunk(st.h, int(k), pos, None) == 0
    return sum(b"ln_relu" in l.name if variant == "resgcn" else b"gemm_nt" in l.name for l in _launches(rt))


def _timed(rt, variant, dims):
    """[kind][layer] timed launches of a whole pass with every kind switched on."""
    st = _Stage(variant, dims, 6)
    assert st.lib.gnnstage_profile_enable(st.h, 1) == 0
    assert st.forward() == 0 and st.backward() == 0
    ms, n, out = C.c_double(0), C.c_int64(0), []
    for kind in range(8):
        out.append([])
        for j in range(st.L):
            assert st.lib.gnnstage_profile_read(st.h, kind, j, C.byref(ms), C.byref(n)) == 0
            out[-1].append(n.value)
    return out


def _all_rows(rt, variant, dims, n, bf16):
    """Return codes of a whole pass, and how many launches it made (its buffers are never touched, so they take no memory)."""
    st = _Stage(variant, dims, 3, n=n, bf16=bf16, dropout_p=0.5)
    rt.host_clear(-1)
    return [st.forward(), st.backward(), rt.host_launches()]


def _refused(rt, variant, dims):
    """A pass in which one launch is refused, at a few places: return codes of the pass and of the calls that follow it."""
    out = {"forward": [], "backward": []}
    st = _Stage(variant, dims, 6)
    rt.host_clear(-1)
    assert st.forward() == 0
    n_fwd = rt.host_launches()
    assert st.backward() == 0
    n_bwd = rt.host_launches() - n_fwd
    for at in (0, n_fwd // 2, n_fwd - 1):
        rt.host_clear(at)
        rc = st.forward()
        rt.host_clear(-1)
        out["forward"].append([rc, st.backward(), st.lib.gnnstage_update_history_swap(st.h, None), rt.host_launches()])
    for at in (0, n_bwd // 3, n_bwd // 2):
        rt.host_clear(-1)
        assert st.forward() == 0
        rt.host_clear(at)
        rc = st.backward()
        rt.host_clear(-1)
        out["backward"].append([rc, st.lib.gnnstage_flush_weight_gradients(st.h, None), st.backward(), rt.host_launches()])
    rt.host_clear(-1)
    assert st.forward() == 0 and st.backward() == 0 and rt.host_launches() == n_fwd + n_bwd  # the handle is as good as new
    return out


if __name__ == "__main__":
    _rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # before the library, whose calls it takes
    _rt.host_launches.restype = C.c_size_t
    _rt.host_launch.restype, _rt.host_launch.argtypes = C.POINTER(_Launch), [C.c_size_t]
    _rt.host_clear.argtypes = [C.c_int64]
    sys.path.insert(0, os.path.dirname(HERE))
    print(json.dumps(globals()[sys.argv[2]](_rt, *json.loads(sys.argv[3]))))
    sys.stdout.flush()
    os._exit(0)  # the handles' buffers are never freed one by one


# ---- tests ------------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("whole,timed", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("tied", [True, False])
def test_no_launch_adds_to_a_layernorm_gradient_twice(runtime, tied, whole, timed):
    """Layers may share a parameter-gradient buffer (tied parameters): the sums of one launch run side by side and add without
    atomics, so a buffer may come up once per launch; buffers of their own go together, unless launches are timed."""
    launches = _child(runtime, "_ln_reduces", tied, whole, timed)
    # the rows of every chunk and layer, and the historical rows of all chunks but the first
    assert sum(len(l) for l in launches) == 2 * (6 + 5) * 4
    for l in launches:
        assert len(set(l)) == len(l)
    assert tied or max(len(l) for l in launches) == (2 if timed else 2 * 4)


@pytest.mark.parametrize("variant,dims", [("resgcn", [32] * 5), ("gcn", [64, 32, 16, 8])])
def test_timed_launches_are_booked_on_their_own_layer(runtime, variant, dims):
    """Six chunks: an aggregation per chunk and layer, and after the last chunk another one for every chunk (ResGCN+: but the
    first) behind the parameters that historical rows went through."""
    timed = _child(runtime, "_timed", variant, dims)
    L = len(dims) - 1
    assert timed[0] == [6] * L and timed[2] == [6 + (5 if variant == "resgcn" else 6)] * L
    assert timed[4] == [timed[4][0]] * L


@pytest.mark.parametrize("variant,dims", [("resgcn", [32] * 5), ("gcn", [64, 32, 40, 8])])
def test_a_pass_that_fails_does_not_count_as_run(runtime, variant, dims):
    """A whole pass in which a launch is refused returns that error.  A forward pass that failed is no pass to run backward or to
    take the history from; one that failed on its way back leaves no weight gradients of rows that it never reached to add."""
    EHIP, EORDER = -5, -3
    got = _child(runtime, "_refused", variant, dims)
    assert got["forward"] == [[EHIP, EORDER, EORDER, 0]] * 3
    assert got["backward"] == [[EHIP, 0, EORDER, 0]] * 3


@pytest.mark.parametrize("variant,dims,bf16,n", [
    ("gcn", [1008, 1002], True, 4_290_001), ("gcn", [1008, 1000], False, 4_300_001), ("resgcn", [1000, 1000], True, 4_300_001)])
def test_launches_over_all_rows_stay_below_2_to_32_threads(runtime, variant, dims, bf16, n):
    """Rows times columns over 2^32: chunk by chunk a thread per element is a launch that the runtime takes, over all rows it is not."""
    assert n * max(dims) >= 2 ** 32
    forward, backward, launches = _child(runtime, "_all_rows", variant, dims, n, bf16)
    assert (forward, backward) == (0, 0) and launches > 0


@pytest.mark.parametrize("n", [65600, 66000, 98000, 131500])
def test_one_long_product_fills_the_chip(runtime, n):
    """Two persistent workgroups on each of the 256 compute units whatever the number of 64-row tiles (historical and current
    rows of a single chunk: two products, one after the other)."""
    assert _child(runtime, "_long_products", n, 1) == [[512, 1, 1]] * 2


@pytest.mark.parametrize("K", [1, 3])
def test_graphsage_adds_its_two_products_one_after_the_other(runtime, K):
    """The product with W_self writes fp32 rows that the layer's other product reads: with the aggregation between the two they
    have left the caches."""
    got = _child(runtime, "_forward_kinds", "sage", [32, 24, 40], K)
    assert set(got.replace("aa", "a").split("a")[1:]) == {"pp"}


@pytest.mark.parametrize("variant,dims", [("gcn", [40, 24]), ("resgcn", [32, 32])])
def test_a_level_0_that_is_its_own_history_is_one_table_in_a_whole_pass(runtime, variant, dims):
    """Of a stage that hands a gradient down: a chunk's rows may come with the chunk, those of a whole pass are there when it begins."""
    assert _child(runtime, "_tables", variant, dims, True) == 1
    assert _child(runtime, "_tables", variant, dims, False) == 1 + 6
