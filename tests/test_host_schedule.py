"""Which rows, entries and partial sums the aggregation launches of a pass serve, on a CPU: the library's host side runs over
host_schedule.c, and the launches' operands are walked as the kernels walk them."""
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
    so = str(tmp_path_factory.mktemp("host") / "libhostschedule.so")
    subprocess.run(["cc", "-O1", "-shared", "-fPIC", "-I", HERE, os.path.join(HERE, "host_schedule.c"), "-o", so], check=True)
    return so


P, I32, I64, U32 = C.c_void_p, C.c_int32, C.c_int64, C.c_uint32


class _Mask(C.Structure):
    _fields_ = [("w", C.c_uint64 * 4)]


class _Spmm(C.Structure):  # SpmmArgs
    _fields_ = [("pidx", P), ("val", P), ("task_row", P), ("task_e0", P), ("task_ne", P), ("task_slot", P), ("cls_begin", I32 * 32), ("cls_end", I32 * 32),
                ("xcd", (I32 * 4) * 8), ("n_class_blocks", I32), ("tail0", I64), ("n_tail", I64),
                ("short0", I64), ("n_short", I64), ("mix", C.c_uint64), ("short_rows", I32), ("slot_class", P), ("active_classes", U32), ("all_classes_active", I32),
                ("lr_row", P), ("lr_slot0", P), ("lr_nslots", P), ("n_long", I64), ("partial", P), ("slot0", I64), ("lr_dense0", P), ("lr_ndense", P),
                ("lr_item0", P), ("item_chunks", P), ("dense_partial", P), ("item0", I64), ("drop_unselected", I32), ("src_sel", P), ("src_unsel", P),
                ("d", I32), ("src_ld", I32), ("vbits", I32), ("many_chunks", I32), ("pass_", P), ("mask", _Mask), ("out", P), ("out_ld", I32), ("out_row0", I64)]


class _Dense(C.Structure):  # DenseArgs
    _fields_ = [("item_rs", P), ("item_chunk", P), ("item_b0", P), ("item_nb", P), ("item_chunks", P), ("n_items", I32), ("blk_cb", P), ("tiles", P), ("bits", P),
                ("colscale", P), ("rowscale", P), ("zero_row", P), ("colslot", P), ("src_sel", P), ("src_unsel", P), ("d", I32), ("src_ld", I32), ("vbits", I32),
                ("pass_", P), ("mask", _Mask), ("partial", P)]


class _Tables(C.Structure):  # PassTableArgs
    _fields_ = [("forward", P), ("backward", P), ("earlier", P), ("K", I32), ("pos", C.c_uint8 * 256), ("classes_backward", U32 * 256), ("classes_earlier", U32 * 256)]


class _Begin(C.Structure):  # StageArgs: weights to stage (planes of the grid), and the tables in a plane of their own
    _fields_ = [("w", C.c_uint8 * 48 * 8), ("n", I32), ("tables", _Tables)]


def _arr(p, n, dtype):
    return np.frombuffer((C.c_char * (int(n) * np.dtype(dtype).itemsize)).from_address(p), dtype=dtype, count=int(n)) if n else np.zeros(0, dtype)


def _tasks(a, name, grid):
    """(task, class) of every wave of a main launch; 16 short rows to a workgroup, or 4, among the others."""
    ring, out = b"ring" in name, []
    for b in range(grid[0]):
        p = b - a.n_class_blocks
        before, upto = p * a.mix >> 32, (p + 1) * a.mix >> 32
        if ring and a.d <= 256 and a.short_rows != 2 and p >= 0 and upto > before:
            out += [(a.short0 + t, -1) for t in range(before * 16, min(before * 16 + 16, a.n_short))]
            continue
        for w in range(4):
            if b < a.n_class_blocks:
                (cls, group0, groups, _), g = a.xcd[b & 7], b >> 3
                if g >= groups:
                    continue
                g += group0
                for q in range(cls, 32):
                    nt = a.cls_end[q] - a.cls_begin[q]
                    ng = (nt + 3) >> 2 if (a.active_classes >> q) & 1 else 0
                    if g < ng:
                        if g * 4 + w < nt:
                            out.append((a.cls_begin[q] + g * 4 + w, q))
                        break
                    g -= ng
                continue
            t, first, n = (before * 4 + w, a.short0, a.n_short) if upto > before else ((p - before) * 4 + w, a.tail0, a.n_tail)
            if t < n:
                out.append((first + t, -1))
    assert len({t for t, _ in out}) == len(out)
    return out


def _mask_words(sees):
    return np.array([sum(1 << k for k in range(len(sees[64 * i:64 * i + 64])) if sees[64 * i + k]) for i in range(4)], np.uint64)


def _walk(rt, first, ptr, dense_on, chunk_ptr, order):
    """Entries gathered by the launches from `first` on, per aggregation (main launches over one source table and output, with
    their reduces): {(transposed, earlier): entries of every (row, source)}; asserts that every row is finished once."""
    K, n, got, most = len(chunk_ptr) - 1, chunk_ptr[-1], {}, int(os.environ.get("GNNSTAGE_LAUNCH_BLOCKS", 2 ** 24 - 1))
    chunk_of = np.searchsorted(chunk_ptr, np.arange(n), side="right") - 1
    pos = np.empty(K, int)
    pos[order] = np.arange(K)
    tables = main = dense = None
    for i in range(first, rt.host_launches()):
        l = rt.host_launch(i).contents
        if b"stage_weights" in l.name:
            begin = _Begin.from_buffer_copy(C.string_at(rt.host_operands(i), C.sizeof(_Begin)))
            if l.grid[1] == begin.n:
                continue
            assert l.grid[1] == begin.n + 1
            tables = begin.tables
            assert list(tables.pos[:K]) == list(pos)
        if b"spmm" not in l.name:
            continue
        operands = _Dense if b"dense" in l.name else _Spmm
        a = operands.from_buffer_copy(C.string_at(rt.host_operands(i), C.sizeof(operands)))
        drop, kind = not a.src_unsel, 0
        assert operands is _Dense or drop == bool(a.drop_unselected)
        if a.pass_:
            kind = {tables.forward: 0, tables.backward: 1, tables.earlier: 2}[a.pass_]
        elif K == 1 and drop:  # no tables
            kind = 1 if a.mask.w[0] else 2

        def sees(c):  # the source chunks that rows of chunk c select
            if not a.pass_:
                return np.array([(a.mask.w[k >> 6] >> (k & 63)) & 1 for k in range(K)], bool)
            return [pos <= pos[c], pos >= pos[c], pos < pos[c]][kind]

        def classes(c):
            return 0xffffffff if not a.pass_ or kind == 0 else [0, tables.classes_backward, tables.classes_earlier][kind][c]

        if operands is _Dense:  # what every item (a run of 128 x 64 blocks) adds to its rows, by place in the row block; None: not run
            dense = []
            for t in range(a.n_items):
                c, b0, nb = (int(_arr(p + t * s, 1, d)[0]) for p, s, d in ((a.item_chunk, 4, "i4"), (a.item_b0, 8, "i8"), (a.item_nb, 4, "i4")))
                bits = _arr(a.bits + 1024 * b0, nb * 256, "u4").reshape(nb, 128, 2)
                words = np.stack([_arr(a.colslot + 256 * int(cb), 64, "u4") for cb in _arr(a.blk_cb + 4 * b0, nb, "i4")])
                on = ((bits[:, :, :, None] >> np.arange(32, dtype=np.uint32)) & 1).astype(bool).reshape(nb, 128, 64)
                assert (words[np.nonzero(on.any(1))] != 0xffffffff).all()
                blk, place, column = np.nonzero(on)
                words, run = words[blk, column], (_arr(a.item_chunks + 32 * t, 4, "u8") & _mask_words(sees(c))).any()
                kept = sees(c)[words >> a.vbits] | (not drop)
                assert run or not drop or not kept.any()
                dense.append((c, None if drop and not run else list(zip(place[kept].tolist(), (words[kept] & ((1 << a.vbits) - 1)).tolist()))))
            continue
        if b"reduce" not in l.name:
            main = a
            key = (a.src_sel, a.out, kind, drop)
            entries, rows, slots, chunks = got.setdefault(key, ([], [], set(), []))
            slots.clear()
            chunks.append(set())
            for t, q in _tasks(a, l.name, l.grid):
                row, e0, ne, slot = (_arr(p + t * s, 1, d)[0] for p, s, d in ((a.task_row, 4, "i4"), (a.task_e0, 8, "i8"), (a.task_ne, 4, "u4"), (a.task_slot, 4, "i4")))
                if row < 0:
                    continue
                c = int(ne) >> 24
                assert chunk_of[row] == c
                chunks[-1].add(c)
                words = _arr(a.pidx + 4 * int(e0), int(ne) & 0xffffff, "u4")
                src, kept = words & ((1 << a.vbits) - 1), sees(c)[words >> a.vbits]
                assert (chunk_of[src] == words >> a.vbits).all()
                assert dense_on or (ptr[drop][row] <= e0 and e0 + len(src) <= ptr[drop][row + 1])
                if q >= 0 and not (classes(c) >> q) & 1:
                    assert not kept.any()  # left out: nothing to gather
                    continue
                entries += [(int(row), int(u)) for u in (src[kept] if drop else src)]
                if slot >= 0:
                    assert slot not in slots and slot >= a.slot0
                    slots.add(int(slot))
                else:
                    rows.append(int(row))
            assert len(chunks[-1]) <= 1 or l.grid[0] <= most
        else:
            assert l.grid[0] == a.n_long
            entries, rows, slots, chunks = got.setdefault((a.src_sel, a.out, kind, drop), ([], [], set(), []))
            if main is None or (a.src_sel, a.out, a.slot0) != (main.src_sel, main.out, main.slot0):  # cut rows alone, none of whose pieces gathers
                slots.clear()
                chunks.append(set())
            assert len(chunks[-1]) <= 1 or l.grid[0] <= most
            for r in range(a.n_long):
                row, s0, ns = (int(_arr(p + 4 * r, 1, "u4")[0]) for p in (a.lr_row, a.lr_slot0, a.lr_nslots))
                c, ns = ns >> 24, ns & 0xffffff
                assert chunk_of[row] == c
                for s in range(s0, s0 + ns):
                    q = int(_arr(a.slot_class + s, 1, "u1")[0])
                    ran = q >= 32 or bool((a.active_classes & classes(c)) >> q & 1) or not drop
                    assert ran == (s in slots)
                if a.lr_ndense:
                    nd, first, it0 = (int(_arr(p + 4 * r, 1, "i4")[0]) for p in (a.lr_ndense, a.lr_dense0, a.lr_item0))
                    for g in range(nd):
                        at, place = divmod(first + (g - a.item0) * 128, 128)
                        used = not drop or (_arr(a.item_chunks + 32 * (it0 + g), 4, "u8") & _mask_words(sees(c))).any()
                        assert dense[at][0] == c and used == (dense[at][1] is not None)
                        entries += [(row, u) for p, u in dense[at][1] or [] if p == place]
                rows.append(row)
            dense = None
    return got


def _stage(variant, dims, chunk_ptr, row_ptr, col, bf16):
    """A stage handle over host buffers, and what has to stay alive with it (nothing is computed)."""
    from paper_2308_10087_amd import binding
    n, L, elt = len(row_ptr) - 1, len(dims) - 1, 2 if bf16 else 4
    dims = np.asarray(dims, np.int32)
    d, keep = binding.gnnstage_desc(), [row_ptr, col, chunk_ptr, dims]
    d.n_vertices, d.nnz, d.n_chunks, d.n_layers = n, len(col), len(chunk_ptr) - 1, L
    d.row_ptr, d.col_idx, d.chunk_ptr, d.dims = (x.ctypes.data for x in keep)

    def pointers(name, sizes):
        a = [np.zeros(int(s) + 16, np.uint8) for s in sizes]
        p = (C.c_void_p * len(a))(*[(x.ctypes.data + 15) // 16 * 16 for x in a])
        keep.append((a, p))
        setattr(d, name, C.cast(p, C.c_void_p))
    two = 2 if variant == "sage" else 1
    for name, sizes in dict(W=[two * dims[j] * dims[j + 1] * elt for j in range(L)], dW=[two * dims[j] * dims[j + 1] * 4 for j in range(L)],
                            cur=[n * w * elt for w in dims], hist=[n * w * elt for w in dims[:-1]], bias=dims[1:] * 4, dbias=dims[1:] * 4,
                            ln_gamma=dims[:-1] * 4, ln_beta=dims[:-1] * 4, d_ln_gamma=dims[:-1] * 4, d_ln_beta=dims[:-1] * 4).items():
        pointers(name, sizes)
    grad = [np.zeros(n * int(w) * elt + 16, np.uint8) for w in (dims[0], dims[-1])]
    at = [(x.ctypes.data + 15) // 16 * 16 for x in grad]
    d.variant, d.dtype, d.need_input_grad, d.grad_in, d.ln_eps = dict(gcn=0, sage=2, resgcn=3)[variant], int(bf16), 1, at[0], 1e-5
    size = binding.lib.gnnstage_workspace_size(C.byref(d))
    ws = np.zeros(size + 256, np.uint8)
    d.workspace, d.workspace_bytes = (ws.ctypes.data + 255) // 256 * 256, size
    h = C.c_void_p(None)
    rc = binding.lib.gnnstage_create(C.byref(d), C.byref(h))
    assert rc == 0, (rc, binding.lib.gnnstage_last_error(None))
    return binding.lib, h, at[1], keep + [grad, ws]


def _pass(rt, variant, dims, K, n, deg, hub, bf16):
    """Aggregations of a whole pass that gathered what they should: [forward, backward, historical, all entries], and the launches that
    each was served in."""
    rng = np.random.default_rng(n + K)
    cols = [np.unique(np.concatenate([[v], rng.integers(0, n, deg if v % 37 else hub)])) for v in range(n)]
    cols[3 % n] = np.zeros(0, np.int64)
    row_ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    col = np.concatenate(cols).astype(np.int32)
    cut = np.sort(rng.integers(0, n + 1, K - 1)) if K > 1 else np.zeros(0, np.int64)
    chunk_ptr = np.concatenate([[0], cut, [n]]).astype(np.int64)
    if K > 3:
        chunk_ptr[2] = chunk_ptr[1]  # an empty chunk
    lib, h, grad_out, keep = _stage(variant, dims, chunk_ptr, row_ptr, col, bf16)
    order = rng.permutation(K).astype(np.int32)
    rt.host_clear(-1)
    assert lib.gnnstage_forward_pass(h, order.ctypes.data, K, None) == 0
    assert lib.gnnstage_backward_pass(h, order.ctypes.data, K, grad_out, None) == 0
    t_ptr = np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))])
    dense_on = lib.gnnstage_dense_entries(h, 0) > 0
    assert dense_on == (lib.gnnstage_dense_entries(h, 1) > 0) == ("GNNSTAGE_DENSE_MIN_ENTRIES" in os.environ)
    got = _walk(rt, 0, [row_ptr, t_ptr], dense_on, chunk_ptr, order)
    rows = np.repeat(np.arange(n), np.diff(row_ptr))
    chunk_of, pos = np.searchsorted(chunk_ptr, np.arange(n), side="right") - 1, np.empty(K, int)
    pos[order] = np.arange(K)
    current = pos[chunk_of[col]] <= pos[chunk_of[rows]]  # the reader saw the source's current row
    pairs = lambda on: sorted(zip(col[on].tolist(), rows[on].tolist()))
    want = [sorted(zip(rows.tolist(), col.tolist())), pairs(current), pairs(~current), pairs(col >= 0)]
    seen = [0, 0, 0, 0]
    for (_, _, kind, drop), (entries, done, _, _) in got.items():
        which = kind if kind else 3 if drop else 0
        assert sorted(entries) == want[which] and sorted(done) == list(range(n))
        seen[which] += 1
    return seen, [len(chunks) for _, _, _, chunks in got.values()]


if __name__ == "__main__":
    sys.path.insert(0, HERE)
    import test_host_launches as _H
    _rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # before the library, whose calls it takes
    _rt.host_launches.restype = C.c_size_t
    _rt.host_launch.restype, _rt.host_launch.argtypes = C.POINTER(_H._Launch), [C.c_size_t]
    _rt.host_operands.restype, _rt.host_operands.argtypes = C.c_void_p, [C.c_size_t]
    _rt.host_operand_bytes.argtypes = [C.c_size_t] * 3
    _rt.host_operand_bytes(C.sizeof(_Spmm), C.sizeof(_Begin), C.sizeof(_Dense))
    _rt.host_clear.argtypes = [C.c_int64]
    sys.path.insert(0, os.path.dirname(HERE))
    print(json.dumps(_pass(_rt, *json.loads(sys.argv[2]))))
    sys.stdout.flush()
    os._exit(0)


def _run(runtime, env, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, json.dumps(args)], capture_output=True, text=True, timeout=300,
                       env={**os.environ, **env})
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


@pytest.mark.parametrize("variant,dims,bf16,seen", [
    ("gcn", [24, 24, 24], 0, [2, 2, 0, 0]), ("gcn", [64, 32, 40], 1, [2, 2, 1, 0]), ("sage", [32, 32, 32], 1, [2, 2, 0, 0]), ("resgcn", [32] * 4, 0, [3, 3, 3, 0])])
@pytest.mark.parametrize("K,n,deg,hub,env", [
    (1, 300, 4, 60, {}), (5, 700, 5, 400, {}), (5, 700, 5, 400, {"GNNSTAGE_SHORT_ROW": "4", "GNNSTAGE_SPLIT_EDGES": "64"}),
    (70, 900, 3, 300, {"GNNSTAGE_SHORT_ROW": "6"}), (6, 500, 2, 200, {"GNNSTAGE_HOT_CLASSES": "3", "GNNSTAGE_HOT_ROWS": "64", "GNNSTAGE_HOT_MIN_ROW": "32"})])
def test_a_pass_gathers_every_entry_once(runtime, variant, dims, bf16, seen, K, n, deg, hub, env):
    """Every aggregation of a whole pass finishes every row once and gathers what its rows' chunks select, once: ragged and empty
    chunks, hubs cut by length and by source class, classes that a chunk gathers nothing from, short rows, more than 64 chunks."""
    if K == 1 and variant == "resgcn":
        seen = seen[:2] + [0, 0]  # no row is read as a historical one
    got, launches = _run(runtime, env, variant, dims, K, n, deg, hub, bf16)
    assert got == seen and set(launches) == {1}


@pytest.mark.parametrize("variant,dims,bf16,seen", [
    ("gcn", [24, 24, 24], 0, [2, 2, 0, 0]), ("gcn", [64, 32, 40], 1, [2, 2, 1, 0]), ("resgcn", [32] * 4, 0, [3, 3, 3, 0])])
@pytest.mark.parametrize("K,n,env", [(7, 700, {"GNNSTAGE_LAUNCH_BLOCKS": "90"}), (70, 900, {"GNNSTAGE_LAUNCH_BLOCKS": "60"}), (5, 700, {"GNNSTAGE_LAUNCH_BLOCKS": "1"}),
                                     (7, 700, {"GNNSTAGE_PARTIAL_ROOM": "0", "GNNSTAGE_CLASS_MIN_ROW": "4"}), (70, 900, {"GNNSTAGE_PARTIAL_ROOM": "5000", "GNNSTAGE_CLASS_MIN_ROW": "4"})])
def test_a_layer_in_several_launches(runtime, variant, dims, bf16, seen, K, n, env):
    """A layer that is too much for one launch, or whose partial sums have no room together, is served in several runs of chunks, one
    chunk at least: the same rows and entries."""
    got, launches = _run(runtime, env, variant, dims, K, n, 5, 300, bf16)
    assert got == seen and min(launches) > 1


@pytest.mark.parametrize("variant,dims,seen", [("gcn", [128] * 3, [2, 2, 0, 0]), ("gcn", [256, 128, 256], [2, 2, 1, 0]), ("resgcn", [128] * 3, [2, 2, 2, 0])])
@pytest.mark.parametrize("K,n,env", [(1, 400, {}), (5, 900, {}), (5, 900, {"GNNSTAGE_PARTIAL_ROOM": "0"}), (70, 1200, {"GNNSTAGE_PARTIAL_ROOM": "200000"}),
                                     (5, 900, {"GNNSTAGE_LAUNCH_BLOCKS": "40"})])
def test_dense_blocks_and_the_rest_gather_every_entry_once(runtime, variant, dims, seen, K, n, env):
    """Entries that are multiplied as blocks of a dense matrix, and those that are left: items by chunk and row block, their tiles
    in the sums of the rows that they are of, in one launch and in several."""
    env = {"GNNSTAGE_DENSE_MIN_ENTRIES": "0", "GNNSTAGE_DENSE_MIN_SHARE": "0", "GNNSTAGE_DENSE_MIN_NNZ": "30", **env}
    if K == 1 and variant == "resgcn":
        seen = seen[:2] + [0, 0]
    got, launches = _run(runtime, env, variant, dims, K, n, 8, 300, 1)
    assert got == seen and (min(launches) > 1 if len(env) > 3 else set(launches) == {1})
