"""Resident reuse with four tokens per step: the repeat that the two fan slots
leave is written by the host copy too.  Plans, tables and buffers equal the
oracle's where an index is missed by all four tokens (no retries: half of the
installs are lost), at the table's capacity, with rows off the 16-byte grid, in
a workspace without the list, and with five tokens, which keep the last launch."""
import numpy as np
import pytest

import oracle as ORC
import workload as W
from harness import HostRows, OracleSide, compare_step, run_parity_modes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_2609_37538_amd import avsg as A
    A.load()
    W.build(force=False)
    ORC.build(force=False)


CASES = [
    ("capacity", dict(batch=3, topk=256, slots=1024, n_q=4, ctx=4000, row_bytes=(1152, 132))),
    ("one_request", dict(batch=1, topk=1024, slots=8192, n_q=4, ctx=60000)),
    ("odd_rows", dict(batch=19, topk=77, slots=512, n_q=4, ctx=1500, row_bytes=(580,))),
    ("five_tokens", dict(batch=3, topk=100, slots=512, n_q=5, ctx=1500)),
]


RUNS = [(name, kw, short) for name, kw in CASES for short in (False, True)
        if not (short and kw["n_q"] != 4)]      # only four tokens have the optional section


@pytest.mark.parametrize("name,kw,short", RUNS, ids=[f"{r[0]}{'_short_workspace' * r[2]}" for r in RUNS])
def test_repeats_of_four_tokens(name, kw, short):
    from paper_2609_37538_amd import avsg as A
    import torch
    spec = W.custom_spec(name=f"four_{name}", steps=8, retention=0.6, **kw)
    if not short:
        run_parity_modes(spec, (A.AVSG_GATHER_RESIDENT,), table_every=2, buffers_every=1,
                         miss_list_requests=3, retry=0)
    wl = W.Workload(spec)
    host = HostRows(wl)
    orc = OracleSide(wl, host, retry=0)
    cfg = A.make_config(spec.batch, spec.topk, spec.n_q, spec.slots, retry=0, row_bytes=spec.row_bytes,
                        gather_mode=A.AVSG_GATHER_RESIDENT)
    op = A.Operator(cfg, host.ptrs, wl.ctx)
    stream = op.stream.cuda_stream
    if short:
        # the same buffers and outputs behind a handle on a workspace that lacks the last section
        h, op.h = op.h, None
        A.avsg_destroy(h)
        size = op.workspace.numel() - 256
        op.h = A.avsg_create(cfg, host.ptrs, wl.ctx, op.workspace.data_ptr(), size,
                             [op.buffers[s][r].data_ptr() for s in range(len(spec.row_bytes))
                              for r in range(spec.batch)], stream)
    repeats = 0
    try:
        for t in range(spec.steps):
            X = wl.topk(t)
            O, n = op.step(torch.from_numpy(np.ascontiguousarray(X, dtype=np.int32)).cuda())
            torch.cuda.synchronize()
            compare_step(t, *orc.step(X, None), O.cpu().numpy(), n.cpu().numpy())
            for s in range(len(spec.row_bytes)):
                assert np.array_equal(op.buffers[s].cpu().numpy(), orc.images[s]), f"step {t} stream {s}"
            repeats += sum(len(op.export_plan(r)[5]) for r in range(spec.batch))
        assert repeats > 0     # some index was missed by four tokens of a step
    finally:
        op.close()
        host.free()


@pytest.mark.parametrize("copies", [2, 5])
def test_index_repeated_within_a_token(copies):
    """An index repeated within a token is the caller's error, but every slot
    that a miss reserved still gets its row: buffers equal those of the
    transfer that reads each miss from the host."""
    from paper_2609_37538_amd import avsg as A
    import torch
    spec = W.custom_spec(name=f"four_repeated_{copies}", batch=3, topk=120, slots=512, n_q=4, steps=6, ctx=3000,
                         retention=0.6, row_bytes=(1152, 132))
    wl = W.Workload(spec)
    host = HostRows(wl)
    ops = [A.Operator(A.make_config(spec.batch, spec.topk, spec.n_q, spec.slots, retry=0, row_bytes=spec.row_bytes,
                                    gather_mode=mode), host.ptrs, wl.ctx)
           for mode in (A.AVSG_GATHER_BALANCED, A.AVSG_GATHER_RESIDENT)]
    try:
        for t in range(spec.steps):
            X = wl.topk(t).copy()
            X[:, :, : 12 * copies] = np.repeat(X[:, :1, :12], copies, axis=2)   # the same twelve in every token
            Xd = torch.from_numpy(np.ascontiguousarray(X, dtype=np.int32)).cuda()
            out = [op.step(Xd) for op in ops]
            torch.cuda.synchronize()
            assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), f"step {t}"
            for s in range(len(spec.row_bytes)):
                assert torch.equal(ops[0].buffers[s], ops[1].buffers[s]), f"step {t} stream {s}"
        a, b = (op.stats() for op in ops)
        assert a["misses"] == b["misses"] and b["duplicate_rows"] > 0 and b["host_bytes"] < a["host_bytes"]
    finally:
        for op in ops:
            op.close()
        host.free()
