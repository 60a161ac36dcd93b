"""Decoded gate streams (16 layers and more) at the layer sizes where they can
go wrong, bit for bit against the CPU oracle: the shortest stream that is
decoded and the longest that is not, empty layers, layers of one gate, of one
wave's 64 ops and one more, of more than 16 waves, every named gate, ops that
a kernel has to skip, and row groups of every width."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2408_00384_amd import Context
    c = Context(0)
    yield c
    c.close()


def _stream(n, sizes, seed):
    """A layer of sizes[l] ops on distinct qubits each (two-qubit ones while
    the qubits last); every fifth layer has CNOTs alone.  Returns the device
    words with one op out of range after every layer, the layer boundaries and
    the gates as a list."""
    from paper_2408_00384_amd import cliff_encode_gates
    rng = np.random.default_rng([93, n, seed])
    words, offs, gates = [], [0], []
    for l, k in enumerate(sizes):
        perm = rng.permutation(n)
        pairs = min(k, n - k)            # 2 pairs + (k - pairs) <= n
        if pairs < 1 or (l % 5 and k > 1):
            pairs = pairs // 2
        two = np.array([2, 7, 8], np.uint8)            # CNOT, CZ, SWAP
        one = np.array([0, 1, 3, 4, 5, 6], np.uint8)   # H, S, S^-1, X, Y, Z
        ops = np.concatenate([np.full(pairs, 2, np.uint8) if l % 5 == 0 else rng.choice(two, pairs),
                              rng.choice(one, k - pairs)]).astype(np.uint8)
        a = np.concatenate([perm[:pairs], perm[2 * pairs:pairs + k]]).astype(np.uint32)
        b = np.concatenate([perm[pairs:2 * pairs], a[pairs:]]).astype(np.uint32)
        w = np.concatenate([cliff_encode_gates(n, ops, a, b)[0] if k else np.empty(0, np.uint64),
                            np.array([n], np.uint64)])
        words.append(w)
        offs.append(offs[-1] + len(w))
        gates.append((ops, a, b))
    return (np.concatenate(words), np.array(offs, np.uint32),
            tuple(np.concatenate([g[i] for g in gates]) for i in range(3)))


def _ref(n, gates, times=1):
    t = oracle.Tableau(n)
    for _ in range(times):
        t.apply_gates(*gates)
    return t.get()


def _same(got, ref):
    return all(np.array_equal(np.asarray(g).reshape(np.shape(r)), r) for g, r in zip(got, ref))


def _upload(words):
    import torch
    d = torch.from_numpy(words.view(np.int64)).to("cuda:0")
    torch.cuda.synchronize()
    return d


# sizes count the ops that act: 63 and the skipped one fill a step of 64
@pytest.mark.parametrize("n,sizes", [
    (1, [1] * 16), (2, [1, 0, 2] * 5), (2, [1, 0, 2] * 6), (130, [63, 64, 65, 0, 1, 130, 127, 128] * 2),
    (130, [40] * 67 + [0] * 5 + [100] * 60), (1500, [1023, 1024, 1025, 1, 0, 1500, 700, 64] * 2),
    (20352, [20352, 0, 1, 16383, 12000, 64, 63, 5] * 2)])
def test_one_tableau(ctx, n, sizes):
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded
    words, offs, gates = _stream(n, sizes, 0)
    dev = _upload(words)
    t = DeviceTableau(ctx, n, 1)
    for _ in range(2):   # (the second stream starts from the first one's signs)
        cliff_apply_encoded(t.handle, dev.data_ptr(), offs)
    if n <= 2000:
        assert _same(t.export(), _ref(n, gates, 2))
    else:                # the layers one launch each
        from paper_2408_00384_amd import GATES_AUTO, GATES_PER_LAYER, cliff_ctx_set_gate_mode
        u = DeviceTableau(ctx, n, 1)
        cliff_ctx_set_gate_mode(ctx.handle, GATES_PER_LAYER)
        try:
            for _ in range(2):
                cliff_apply_encoded(u.handle, dev.data_ptr(), offs)
        finally:
            cliff_ctx_set_gate_mode(ctx.handle, GATES_AUTO)
        rows = np.concatenate([np.arange(0, 2 * n, 997), [2 * n - 1]]).astype(np.uint32)
        assert _same(t.export_rows(rows), u.export_rows(rows))
        u.close()
    t.close()


@pytest.mark.parametrize("rows", [32, 64, 128])
@pytest.mark.parametrize("short", [16, 15])
def test_many_tableaux(ctx, rows, short):
    """Tableaux of 1 to 700 qubits and streams of 15 or 16 to 1,300 layers."""
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many
    shapes = [(1, [1] * short), (33, [33, 0, 7, 20] * 5), (130, [63, 64, 65, 130] * 8),
              (64, [1, 30] * 650), (700, [700, 1, 0, 320, 319, 63, 64] * 3)]
    streams = [_stream(n, sizes, 1 + i) for i, (n, sizes) in enumerate(shapes)]
    dev = [_upload(w) for w, _, _ in streams]
    tabs = [DeviceTableau(ctx, n, 1) for n, _ in shapes]
    for _ in range(2):
        cliff_apply_encoded_many([t.handle for t in tabs], [d.data_ptr() for d in dev],
                                 [o for _, o, _ in streams], rows)
    for t, (n, _), (_, _, gates) in zip(tabs, shapes, streams):
        assert _same(t.export(), _ref(n, gates, 2)), "n = %d" % n
        t.close()


# streams that pass through the staging area in halves (more than 4 MB, the
# last qubit unpaired), and one whose layers leave most qubits without a gate
@pytest.mark.parametrize("n,npairs,depth,p", [(1501, 750, 900, 0.5), (3000, 10, 1500, 0.01)])
def test_long_layers_through_the_staging_area(ctx, n, npairs, depth, p):
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded, cliff_encode_layers
    rng = np.random.default_rng([97, n])
    h, s = ((rng.random((depth, n)) < p).astype(np.uint8) for _ in range(2))
    perm = rng.permuted(np.tile(np.arange(n, dtype=np.uint32), (depth, 1)), axis=1)
    ctrl, tgt = np.ascontiguousarray(perm[:, :npairs]), np.ascontiguousarray(perm[:, npairs:2 * npairs])
    words, offs = cliff_encode_layers(n, h, s, ctrl, tgt)
    dev = _upload(words)
    t, u = DeviceTableau(ctx, n, 1), DeviceTableau(ctx, n, 1)
    for _ in range(2):
        t.apply_layers(h, s, ctrl, tgt)
        cliff_apply_encoded(u.handle, dev.data_ptr(), offs)
    rows = np.arange(0, 2 * n, 61, dtype=np.uint32)
    assert _same(t.export_rows(rows), u.export_rows(rows))
    bad = ctrl.copy()
    bad[depth - 1, 0] = tgt[depth - 1, 0]          # refused after most of it was staged: no change
    with pytest.raises(Exception, match="control == target"):
        t.apply_layers(h, s, bad, tgt)
    assert _same(t.export_rows(rows), u.export_rows(rows))
    t.close()
    u.close()


@pytest.mark.parametrize("rows", [32, 64])
def test_many_tableaux_in_parts(ctx, rows):
    """Streams of over 512 MB decoded, so that they go through the scratch in
    parts of all tableaux' layers: the shortest stream has 16 layers, the
    longest 80,000 of one gate each."""
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many
    shapes = [(40, [1, 40] * 40000), (3, [1, 2, 3, 0] * 4), (70, [70, 65, 1] * 30)]
    streams = [_stream(n, sizes, 7 + i) for i, (n, sizes) in enumerate(shapes)]
    dev = [_upload(w) for w, _, _ in streams]
    copies = [14, 2, 2]            # 14 x 80,000 steps of 64 ops
    tabs, ds, os_, refs = [], [], [], []
    for (n, _), (_, o, gates), d, k in zip(shapes, streams, dev, copies):
        ref = _ref(n, gates)
        for _ in range(k):
            tabs.append(DeviceTableau(ctx, n, 1))
            ds.append(d.data_ptr())
            os_.append(o)
            refs.append(ref)
    cliff_apply_encoded_many([t.handle for t in tabs], ds, os_, rows)
    for t, ref in zip(tabs, refs):
        assert _same(t.export(), ref)
        t.close()


# n past the one-launch kernels: layers of most qubits go through the cache in
# parts of the row words, layers of few qubits in one launch each
@pytest.mark.parametrize("n,pairs,depth,launches", [(21000, 10, 30, 30), (21000, 10500, 3, 6), (30000, 1, 5, 5)])
def test_row_parts_only_where_layers_fill_them(ctx, n, pairs, depth, launches):
    from paper_2408_00384_amd import (DeviceTableau, cliff_apply_encoded, cliff_ctx_profile, cliff_ctx_profile_read,
                                      cliff_encode_layers)
    rng = np.random.default_rng([98, n, pairs])
    perm = np.stack([rng.permutation(n)[: 2 * pairs] for _ in range(depth)]).astype(np.uint32)
    zero = np.zeros((depth, n), np.uint8)
    words, offs = cliff_encode_layers(n, zero, zero, np.ascontiguousarray(perm[:, :pairs]),
                                      np.ascontiguousarray(perm[:, pairs:]))
    dev = _upload(words)
    t = DeviceTableau(ctx, n, 1)
    cliff_ctx_profile(ctx.handle, True)
    try:
        cliff_apply_encoded(t.handle, dev.data_ptr(), offs)
        got = cliff_ctx_profile_read(ctx.handle, "gate")[1]
    finally:
        cliff_ctx_profile(ctx.handle, False)
    assert got == launches
    # CNOTs on |0...0>: destabilizer X_j and stabilizer Z_j spread as the bits below
    q = perm[:, :].ravel()[:8]
    x, z = np.eye(n, dtype=np.uint8)[q], np.eye(n, dtype=np.uint8)[q]
    for l in range(depth):
        for c, g in zip(perm[l, :pairs], perm[l, pairs:]):
            x[:, g] ^= x[:, c]
            z[:, c] ^= z[:, g]
    gx, gz, gr = t.export_rows(np.concatenate([q, q + n]).astype(np.uint32))
    k = len(q)
    assert np.array_equal(gx[:k], x) and not gz[:k].any() and np.array_equal(gz[k:], z) and not gx[k:].any()
    assert not gr.any()
    t.close()


@pytest.mark.parametrize("n", [4000, 20000])
def test_sparse_layers_decoded_no_slower(ctx, n):
    """16 layers of five CNOTs, which are decoded, take no longer than the
    first 15, which are not: loading and storing the columns is most of it."""
    import time
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded, cliff_encode_layers
    rng = np.random.default_rng([99, n])
    perm = np.stack([rng.permutation(n)[:10] for _ in range(16)]).astype(np.uint32)
    zero = np.zeros((16, n), np.uint8)
    words, offs = cliff_encode_layers(n, zero, zero, np.ascontiguousarray(perm[:, :5]), np.ascontiguousarray(perm[:, 5:]))
    dev = _upload(words)
    t = DeviceTableau(ctx, n, 1)
    best = {}
    for depth in (15, 16):
        times = []
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(4):
                cliff_apply_encoded(t.handle, dev.data_ptr(), offs[: depth + 1])
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best[depth] = min(times)
    assert best[16] < 1.1 * best[15], best
    t.close()


# either side of what decoding needs of many tableaux: 64 layers of one step, 16
# of 24 steps (with the skipped op: 1,537)
@pytest.mark.parametrize("n,sizes", [(30, [5] * 63), (30, [5] * 64), (1600, [1535] * 16), (1600, [1536] * 16)])
def test_many_at_the_least_worth_decoding(ctx, n, sizes):
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many
    words, offs, gates = _stream(n, sizes, 3)
    dev = _upload(words)
    tabs = [DeviceTableau(ctx, n, 1) for _ in range(3)]
    for _ in range(2):
        cliff_apply_encoded_many([t.handle for t in tabs], [dev.data_ptr()] * 3, [offs] * 3)
    ref = _ref(n, gates, 2)
    for t in tabs:
        assert _same(t.export(), ref)
        t.close()


@pytest.mark.parametrize("n,rows", [(200, 32), (200, 64), (64, 32)])
def test_many_tableaux_over_the_scratch(ctx, n, rows):
    """Over 2^20 steps: in parts by layers where a tableau has six row groups
    and more (n = 200), as op words where it has fewer."""
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many
    shapes = [(n, [1, 3] * 40000), (n, [2, 0, min(n, 65), 1] * 5), (n, [1] * 17)]
    streams = [_stream(m, sizes, 11 + i) for i, (m, sizes) in enumerate(shapes)]
    dev = [_upload(w) for w, _, _ in streams]
    tabs, ds, os_, refs = [], [], [], []
    for (m, _), (_, o, gates), d, k in zip(shapes, streams, dev, [14, 1, 1]):
        ref = _ref(m, gates)
        for _ in range(k):
            tabs.append(DeviceTableau(ctx, m, 1))
            ds.append(d.data_ptr())
            os_.append(o)
            refs.append(ref)
    cliff_apply_encoded_many([t.handle for t in tabs], ds, os_, rows)
    for t, ref in zip(tabs, refs):
        assert _same(t.export(), ref)
        t.close()


def test_many_refuses_decreasing_boundaries(ctx):
    """At any layer and by any amount (the check is arithmetic on borrows)."""
    from paper_2408_00384_amd import CLIFF_EINVAL, CliffError, DeviceTableau, cliff_apply_encoded_many
    words, offs, _ = _stream(9, [3] * 70, 5)
    dev = _upload(words)
    t = DeviceTableau(ctx, 9, 1)
    for l, v in [(1, 0xFFFFFFFF), (35, 0x80000000), (70, 0), (70, int(offs[69]) - 1)]:
        bad = offs.copy()
        bad[l] = v
        with pytest.raises(CliffError, match="decrease at layer %d" % (l if l < 70 else 69)) as e:
            cliff_apply_encoded_many([t.handle], [dev.data_ptr()], [bad])
        assert e.value.code == CLIFF_EINVAL
    assert _same(t.export(), _ref(9, (np.empty(0, np.uint8), np.empty(0, np.uint32), np.empty(0, np.uint32))))
    t.close()


def test_many_sparse_layers_no_slower(ctx):
    """16 layers of five CNOTs, and 64, on 8 tableaux of n = 8,000: the longer
    stream is decoded, and loading the columns is still most of it."""
    import time
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many, cliff_encode_layers
    n = 8000
    rng = np.random.default_rng([100, n])
    perm = np.stack([rng.permutation(n)[:10] for _ in range(64)]).astype(np.uint32)
    zero = np.zeros((64, n), np.uint8)
    words, offs = cliff_encode_layers(n, zero, zero, np.ascontiguousarray(perm[:, :5]), np.ascontiguousarray(perm[:, 5:]))
    dev = _upload(words)
    tabs = [DeviceTableau(ctx, n, 1) for _ in range(8)]
    hs, ptrs = [t.handle for t in tabs], [dev.data_ptr()] * 8
    best = {}
    for depth in (15, 64):
        times = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            cliff_apply_encoded_many(hs, ptrs, [offs[: depth + 1]] * 8)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best[depth] = min(times)
    assert best[64] < 1.3 * best[15], best
    for t in tabs:
        t.close()


@pytest.mark.parametrize("rows", [32, 64, 128])
@pytest.mark.parametrize("n", [2, 3, 30])
def test_one_wave_keeps_the_layers_in_order(ctx, n, rows):
    """Layers of one step on the same few columns, each reading what the last
    one wrote, in workgroups of one wave, which has no barrier between them."""
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_encoded_many
    words, offs, gates = _stream(n, [n, max(1, n // 2), 1] * 150, 6)
    dev = _upload(words)
    tabs = [DeviceTableau(ctx, n, 1) for _ in range(2)]
    cliff_apply_encoded_many([t.handle for t in tabs], [dev.data_ptr()] * 2, [offs] * 2, rows)
    ref = _ref(n, gates)
    for t in tabs:
        assert _same(t.export(), ref)
        t.close()


def test_scratch_grows_in_few_steps():
    """Streams a little longer each time do not each reallocate the scratch."""
    import torch
    from paper_2408_00384_amd import Context, DeviceTableau, cliff_apply_encoded
    ctx = Context(0)
    words, offs, _ = _stream(2, [1] * 5000, 8)
    dev = _upload(np.tile(words, 11))
    t = DeviceTableau(ctx, 2, 1)
    free = set()
    for k in range(1, 11):   # 5,000 steps (2.5 MB) more each time
        o = np.concatenate([offs[:-1] + i * offs[-1] for i in range(k)] + [[k * offs[-1]]]).astype(np.uint32)
        cliff_apply_encoded(t.handle, dev.data_ptr(), o)
        torch.cuda.synchronize()
        free.add(torch.cuda.mem_get_info()[0])
    assert len(free) <= 6, free
    t.close()
    ctx.close()
