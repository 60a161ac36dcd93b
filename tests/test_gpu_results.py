"""Results and records: conditioned Paulis at the edges of a block's 64 shots,
4 row words and 32 ops, and outcomes and random flags as the device hands them over (transposed in tiles
of 64 measurements by 64 shots), at the edges of the tiles: against the
device's own record of the same measurements."""
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


# k: past n (two passes, the second into later columns); the last two: rows
# handed over in two parts (16 MB each at most)
@pytest.mark.parametrize("n,shots,k", [(1, 1, 1), (2, 64, 2), (63, 65, 63), (64, 63, 64), (65, 1, 65), (130, 128, 127),
                                       (40, 129, 90), (200, 1000, 193), (1030, 3, 1030), (300, 53000, 300),
                                       (64, 262144, 64)])
def test_outcomes_match_the_device_record(ctx, n, shots, k):
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_measure_async, cliff_measure_record, cliff_tab_read_outcomes
    c = layered_circuit(n, 6, 1, gen_seed=[94, n], circuit_id=31)
    q = np.resize(np.random.default_rng(n).permutation(n), k).astype(np.uint32)
    rec = torch.zeros((shots, k), dtype=torch.uint8, device="cuda:0")
    rnd = torch.zeros(k, dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()
    t = DeviceTableau(ctx, n, shots).apply_circuit_gates(c)
    cliff_measure_record(t.handle, q, rec.data_ptr(), k, 0, rnd.data_ptr(), c.seed, c.circuit_id)
    torch.cuda.synchronize()
    t.init_zero()
    out, flags = t.apply_circuit_gates(c).measure(q, seed=c.seed, circuit=c.circuit_id)
    assert np.array_equal(out, rec.cpu().numpy()) and np.array_equal(flags, rnd.cpu().numpy())
    if k <= n:
        t.init_zero()
        t.apply_circuit_gates(c)
        cliff_measure_async(t.handle, q, c.seed, c.circuit_id)
        out, flags = cliff_tab_read_outcomes(t.handle, k)
        assert np.array_equal(out, rec.cpu().numpy()) and np.array_equal(flags, rnd.cpu().numpy())
    t.close()


@pytest.mark.parametrize("n,shots,k", [(1, 1, 1), (31, 63, 3), (32, 64, 31), (127, 65, 32), (129, 130, 33),
                                       (500, 5, 200)])
def test_cond_paulis_vs_oracle(ctx, n, shots, k):
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_cond_paulis
    c = layered_circuit(n, 6, 1, gen_seed=[96, n], circuit_id=32)
    rng = np.random.default_rng([n, k])
    q, p, col = rng.integers(0, n, k).astype(np.uint32), rng.integers(1, 4, k).astype(np.uint8), \
        rng.integers(0, 9, k).astype(np.uint32)
    bits = rng.integers(0, 2, (shots, 9)).astype(np.uint8)
    rec = torch.from_numpy(bits).to("cuda:0")
    torch.cuda.synchronize()
    t = DeviceTableau(ctx, n, shots).apply_circuit_gates(c)
    cliff_apply_cond_paulis(t.handle, q, p, col, rec.data_ptr(), 9)
    gx, gz, gr = t.export()
    for s in {0, shots // 2, shots - 1}:
        r = oracle.Tableau(n).apply_circuit_gates(c)
        for i in range(k):
            if bits[s, col[i]]:
                r.pauli(int(q[i]), int(p[i]))
        x, z, rr = r.get()
        assert np.array_equal(gx, x) and np.array_equal(gz, z) and np.array_equal(gr[s], rr)
    t.close()


# the ops of a wave in fours and one by one, and either side of 16, from where
# on a block's waves share them
@pytest.mark.parametrize("n,shots,k", [(33, 1, 4), (64, 64, 5), (65, 600, 7), (130, 129, 15), (130, 129, 16)])
def test_few_cond_paulis_vs_oracle(ctx, n, shots, k):
    test_cond_paulis_vs_oracle(ctx, n, shots, k)


def test_one_cond_pauli_costs_less_than_sixteen(ctx):
    import time
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_apply_cond_paulis
    n, shots = 100, 1 << 20
    t = DeviceTableau(ctx, n, shots)
    rec = torch.randint(0, 2, (shots, 8), dtype=torch.uint8, device="cuda:0")
    best = {}
    for k in (1, 16):
        q, p, col = np.arange(k, dtype=np.uint32), np.ones(k, np.uint8), np.arange(k, dtype=np.uint32) % 8
        times = []
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(8):
                cliff_apply_cond_paulis(t.handle, q, p, col, rec.data_ptr(), 8)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best[k] = min(times)
    assert best[1] < best[16] / 2, best
    t.close()


# rows of fewer than 48 outcomes of more than 64 shots come without gaps, 16
# bytes a thread: ends inside and at a thread's bytes, either side of both
# limits, and two parts of 16 MB
@pytest.mark.parametrize("n,shots,k", [(9, 64, 9), (9, 65, 9), (16, 255, 16), (20, 257, 17), (70, 100, 47),
                                       (70, 100, 48), (9, 4097, 1), (9, 262147, 7), (9, 3000001, 8)])
def test_few_outcomes_of_many_shots(ctx, n, shots, k):
    import torch
    from paper_2408_00384_amd import DeviceTableau, cliff_measure_async, cliff_measure_record, cliff_tab_read_outcomes
    c = layered_circuit(n, 6, 1, gen_seed=[97, n], circuit_id=33)
    q = np.random.default_rng(k).permutation(n)[:k].astype(np.uint32)
    rec = torch.zeros((shots, k), dtype=torch.uint8, device="cuda:0")
    rnd = torch.zeros(k, dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()
    t = DeviceTableau(ctx, n, shots).apply_circuit_gates(c)
    cliff_measure_record(t.handle, q, rec.data_ptr(), k, 0, rnd.data_ptr(), c.seed, c.circuit_id)
    torch.cuda.synchronize()
    t.init_zero()
    t.apply_circuit_gates(c)
    cliff_measure_async(t.handle, q, c.seed, c.circuit_id)
    out, flags = cliff_tab_read_outcomes(t.handle, k)
    assert np.array_equal(out, rec.cpu().numpy()) and np.array_equal(flags, rnd.cpu().numpy())
    t.init_zero()
    many = np.concatenate([np.arange(n), q]).astype(np.uint32)   # (past n: a second pass into later columns)
    out, flags = t.apply_circuit_gates(c).measure(many, seed=c.seed, circuit=c.circuit_id)
    assert np.array_equal(out[:, n:], out[:, q]) and not flags[n:].any()   # (a Z outcome repeats)
    t.close()


def test_one_outcome_costs_less_than_many(ctx):
    """One outcome of 2^20 shots is read in a fraction of the time of 64."""
    import time
    from paper_2408_00384_amd import DeviceTableau, cliff_measure_async, cliff_tab_read_outcomes
    t = DeviceTableau(ctx, 64, 1 << 20)
    cliff_measure_async(t.handle, np.arange(64, dtype=np.uint32))
    best = {}
    for k in (1, 64):
        times = []
        for _ in range(6):
            t0 = time.perf_counter()
            cliff_tab_read_outcomes(t.handle, k)
            times.append(time.perf_counter() - t0)
        best[k] = min(times)
    assert best[1] < best[64] / 4, best
    t.close()
