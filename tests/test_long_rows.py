"""Rows longer than 4 GiB, on the 16-byte grid and off it: every byte arrives,
also those past the reach of a 32-bit offset."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_bytes", [(1 << 32) + 48, (1 << 32) + 36])
def test_row_past_4_gib(row_bytes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_2609_37538_amd import avsg as A
    A.load()
    region = A.HostRegion(row_bytes)
    op = None
    try:
        host = torch.from_numpy(region.view().view(np.int32))
        want = torch.empty(row_bytes // 4, dtype=torch.int32, device="cuda")
        want.random_(-(1 << 31), (1 << 31) - 1, generator=torch.Generator(device="cuda").manual_seed(5))
        host.copy_(want)
        op = A.Operator(A.make_config(1, 1, 1, 2, row_bytes=(row_bytes,)), [region.ptr], [1])
        print(f"[gpu] one row of {row_bytes} bytes", flush=True)
        slots, misses = op.step(torch.zeros((1, 1, 1), dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        assert misses.item() == 1
        assert torch.equal(op.buffers[0][0, slots.item()].view(torch.int32), want)
    finally:
        if op is not None:
            op.close()
            del op
        del host
        region.free()
        torch.cuda.empty_cache()
