"""Calls recorded in a HIP graph and replayed: the allocation-free measurement
in the automatic mode (any n), the per-measurement kernels, and a device-
resident gate stream layer by layer.  Every replay
is compared with the eager call on the same state, with eager measurements of
another size and synchronizations between the replays."""
import numpy as np
import pytest

from inputs import layered_circuit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,shots,step,noalloc", [(64, 64, 16, False, True), (300, 120, 2, False, True),
                                                    (4096, 200, 1, False, True), (10300, 40, 1, False, True),
                                                    (300, 120, 2, True, False), (10300, 40, 1, False, False)])
def test_replayed_measurement(n, k, shots, step, noalloc):
    import torch
    import paper_2408_00384_amd as P
    c = layered_circuit(n, 6, shots, gen_seed=[110, n], circuit_id=41)
    other = layered_circuit(70, 6, 1, gen_seed=[111], circuit_id=42)
    q = np.concatenate([np.arange(k - 2), [0, 3]]).astype(np.uint32)
    rows = np.unique(np.linspace(0, 2 * n - 1, 300).astype(np.uint32))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        if step:
            P.cliff_ctx_set_measure_mode(ctx.handle, P.MEASURE_STEP)
        t, u = P.DeviceTableau(ctx, n, shots), P.DeviceTableau(ctx, 70, 1)
        rec = torch.zeros((shots, k), dtype=torch.uint8, device="cuda:0")
        rnd = torch.zeros(k, dtype=torch.uint8, device="cuda:0")
        measure = P.cliff_measure_record_noalloc if noalloc else P.cliff_measure_record

        def record():
            measure(t.handle, q, rec.data_ptr(), k, 0, rnd.data_ptr(), c.seed, c.circuit_id)

        def state():
            rec.zero_()
            rnd.zero_()
            t.init_zero().apply_circuit_gates(c)

        def result():
            torch.cuda.synchronize()
            return [rec.cpu().numpy(), rnd.cpu().numpy(), *t.export_rows(rows), P.cliff_tab_counters(t.handle)]

        state()
        record()
        want = result()
        P.cliff_graph_begin(ctx.handle)
        record()
        graph = P.cliff_graph_end(ctx.handle)
        for _ in range(3):
            state()
            P.cliff_graph_launch(graph)
            got = result()
            assert all(np.array_equal(a, b) for a, b in zip(got[:-1], want[:-1])) and got[-1] == want[-1]
            u.init_zero().apply_circuit_gates(other).measure(np.arange(70, dtype=np.uint32))
        assert 0 < int(want[1].sum()) < k and want[-1]["anomalies"] == 0
        torch.cuda.synchronize()
        P.cliff_graph_destroy(graph)
        t.close()
        u.close()
        ctx.close()


@pytest.mark.parametrize("n,depth", [(300, 20), (21000, 3)])
def test_replayed_gate_stream(n, depth):
    import torch
    import paper_2408_00384_amd as P
    c = layered_circuit(n, depth, 1, gen_seed=[112, n], circuit_id=43)
    words, offs = P.cliff_encode_layers(n, c.h, c.s, c.ctrl, c.tgt)
    rows = np.unique(np.linspace(0, 2 * n - 1, 300).astype(np.uint32))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = P.Context(0, stream)
        P.cliff_ctx_set_gate_mode(ctx.handle, P.GATES_PER_LAYER if n <= 20352 else P.GATES_AUTO)
        dev = torch.from_numpy(words.view(np.int64)).to("cuda:0")
        t, u = P.DeviceTableau(ctx, n, 1), P.DeviceTableau(ctx, n, 1)
        torch.cuda.synchronize()
        P.cliff_graph_begin(ctx.handle)
        t.init_zero()
        P.cliff_apply_encoded(t.handle, dev.data_ptr(), offs)
        graph = P.cliff_graph_end(ctx.handle)
        u.apply_circuit_gates(c)
        want = u.export_rows(rows)
        for _ in range(3):
            P.cliff_graph_launch(graph)
            assert all(np.array_equal(a, b) for a, b in zip(t.export_rows(rows), want))
            u.init_zero().apply_circuit_gates(c).measure(np.arange(33, dtype=np.uint32))
        torch.cuda.synchronize()
        P.cliff_graph_destroy(graph)
        t.close()
        u.close()
        ctx.close()
