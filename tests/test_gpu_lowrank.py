"""The automatic mode's measurement (blocks of 64 measurements, each one
low-rank update of the tableau) at the sizes where it can go wrong, bit for
bit against the CPU oracle, or, where that is too slow, against the
per-measurement kernels: tableau bits, every shot's signs, outcomes, random
flags and the device counters."""
import numpy as np
import pytest

import oracle
from inputs import layered_circuit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2408_00384_amd import Context
    c = Context(0)
    yield c
    c.close()


def _check(ctx, c, q, shots):
    from paper_2408_00384_amd import DeviceTableau
    t = DeviceTableau(ctx, c.n, shots).apply_circuit_gates(c)
    out, rnd = t.measure(q, seed=c.seed, circuit=c.circuit_id)
    gx, gz, gr = t.export()
    ref = oracle.Tableau(c.n).apply_circuit_gates(c)
    for s in range(shots):
        r = ref.clone()
        o, k = r.measure_list(q, seed=c.seed, circuit=c.circuit_id, shot=s)
        x, z, rr = r.get()
        assert np.array_equal(rnd, k)
        assert np.array_equal(out[s], o), "shot %d" % s
        assert np.array_equal(gx, x) and np.array_equal(gz, z) and np.array_equal(gr[s], rr)
    assert t.anomalies() == 0
    t.close()
    return rnd


# one unit, whole words and ragged ones, one block and several, the last
# block partial; 1,024 / 1,025: the last size with 32-row units
@pytest.mark.parametrize("n,depth,shots", [(1, 2, 1), (2, 3, 5), (31, 8, 2), (32, 8, 2), (33, 8, 65), (63, 9, 3),
                                           (64, 12, 3), (65, 12, 3), (127, 12, 1), (129, 12, 300), (511, 12, 2),
                                           (1024, 12, 1), (1025, 12, 1)])
def test_dense_vs_oracle(ctx, n, depth, shots):
    c = layered_circuit(n, depth, shots, gen_seed=[90, n], circuit_id=21)
    _check(ctx, c, c.qubits, shots if shots < 8 else 4 if shots > 100 else shots)


# many rows with few bits: the planner's window holds all of them (up to 512)
# or has to search beyond its 128; deterministic outcomes in between
@pytest.mark.parametrize("n,depth", [(100, 1), (300, 1), (700, 2), (1100, 3), (1500, 4)])
def test_shallow_vs_oracle(ctx, n, depth):
    c = layered_circuit(n, depth, 2, gen_seed=[91, n, depth], circuit_id=22)
    rnd = _check(ctx, c, c.qubits, 2)
    assert 0.05 < rnd.mean() < 1.0


def test_deterministic_with_unmeasured_rest_vs_oracle(ctx):
    """Repeated qubits while most of the tableau is unmeasured: the product
    of the selected stabilizers runs over columns with x bits.  A repeat
    inside a block, in a later block, and in a second call."""
    from paper_2408_00384_amd import DeviceTableau
    n, shots = 500, 3
    c = layered_circuit(n, 14, shots, gen_seed=[92], circuit_id=23)
    q1 = np.concatenate([np.arange(0, 40), [5, 39, 5], np.arange(300, 370), [0, 301, 17]]).astype(np.uint32)
    q2 = np.concatenate([[2, 310], np.arange(40, 93)]).astype(np.uint32)
    t = DeviceTableau(ctx, n, shots).apply_circuit_gates(c)
    o1, k1 = t.measure(q1, seed=c.seed, circuit=23)
    o2, k2 = t.measure(q2, seed=c.seed, circuit=23, m0=len(q1))
    gx, gz, gr = t.export()
    ref = oracle.Tableau(n).apply_circuit_gates(c)
    for s in range(shots):
        r = ref.clone()
        o, k = r.measure_list(np.concatenate([q1, q2]), seed=c.seed, circuit=23, shot=s)
        assert np.array_equal(np.concatenate([o1[s], o2[s]]), o)
        assert np.array_equal(np.concatenate([k1, k2]), k)
        x, z, rr = r.get()
        assert np.array_equal(gx, x) and np.array_equal(gz, z) and np.array_equal(gr[s], rr)
    assert not k1[40:43].any() and not k2[:2].any()
    assert t.anomalies() == 0
    t.close()


def test_list_longer_than_n(ctx):
    """More measurements than qubits: several passes in one call."""
    c = layered_circuit(70, 9, 2, gen_seed=[93], circuit_id=24)
    q = np.concatenate([np.arange(70), np.arange(69, -1, -1), [3]]).astype(np.uint32)
    _check(ctx, c, q, 2)


@pytest.mark.parametrize("n,depth", [(200, 12), (600, 2), (1300, 12)])
def test_counters_match_per_measurement_path(ctx, n, depth):
    from paper_2408_00384_amd import (MEASURE_AUTO, MEASURE_PERSISTENT, DeviceTableau, cliff_ctx_set_measure_mode,
                                      cliff_tab_counters, cliff_tab_reset_counters)
    c = layered_circuit(n, depth, 2, gen_seed=[94, n], circuit_id=25)
    res = []
    try:
        for mode in (MEASURE_PERSISTENT, MEASURE_AUTO):
            cliff_ctx_set_measure_mode(ctx.handle, mode)
            t = DeviceTableau(ctx, n, 2).apply_circuit_gates(c)
            cliff_tab_reset_counters(t.handle)
            t.measure(c.qubits, seed=c.seed, circuit=25)
            res.append(cliff_tab_counters(t.handle))
            t.close()
    finally:
        cliff_ctx_set_measure_mode(ctx.handle, MEASURE_AUTO)
    assert res[0] == res[1]


# one and several row tiles, the planner's rows in 2, 11 or 32 registers and
# (above 32,768 qubits) not in registers; shallow circuits make it search
@pytest.mark.parametrize("n,depth,k", [(2049, 14, 70), (4097, 2, 400), (10240, 2, 300), (12000, 2, 300),
                                       (33000, 2, 150)])
def test_large_equals_step(ctx, n, depth, k):
    from paper_2408_00384_amd import (MEASURE_AUTO, MEASURE_STEP, DeviceTableau, cliff_ctx_set_measure_mode,
                                      cliff_tab_counters)
    c = layered_circuit(n, depth, 2, gen_seed=[95, n], circuit_id=26)
    rng = np.random.Generator(np.random.PCG64([96, n]))
    q = np.concatenate([rng.permutation(n)[: k - 4], [7, 7, 8, 7]]).astype(np.uint32)
    rows = np.unique(np.concatenate([rng.integers(0, 2 * n, size=192), [0, n - 1, n, 2 * n - 1]])).astype(np.uint32)
    res = []
    try:
        for mode in (MEASURE_STEP, MEASURE_AUTO):
            cliff_ctx_set_measure_mode(ctx.handle, mode)
            t = DeviceTableau(ctx, n, 2).apply_circuit_gates(c)
            out, rnd = t.measure(q, seed=c.seed, circuit=26)
            res.append((out, rnd, *t.export_rows(rows), cliff_tab_counters(t.handle)))
            t.close()
    finally:
        cliff_ctx_set_measure_mode(ctx.handle, MEASURE_AUTO)
    for a, b in zip(res[0][:-1], res[1][:-1]):
        assert np.array_equal(a, b)
    assert res[0][-1] == res[1][-1]
    assert 0 < int(res[0][1].sum()) < k


# the columns' stabilizer words fill 2, 2, 4, 32 and 64 lanes, and more
@pytest.mark.parametrize("n", [33, 64, 130, 1500, 2049, 4200])
def test_deterministic_terms_by_columns(ctx, n):
    """Repeats while half the qubits are unmeasured, at every packing of the
    columns' words into lanes."""
    from paper_2408_00384_amd import DeviceTableau
    c = layered_circuit(n, 6, 1, gen_seed=[95, n], circuit_id=24)
    rng = np.random.default_rng(n)
    q = rng.permutation(n)[:min(n // 2, 70)]
    q = np.concatenate([q, q[::3]]).astype(np.uint32)
    t = DeviceTableau(ctx, n, 1).apply_circuit_gates(c)
    out, rnd = t.measure(q, seed=c.seed, circuit=24)
    ref = oracle.Tableau(n).apply_circuit_gates(c)
    o, k = ref.measure_list(q, seed=c.seed, circuit=24, shot=0)
    assert np.array_equal(out[0], o) and np.array_equal(rnd, k) and t.anomalies() == 0
    t.close()
