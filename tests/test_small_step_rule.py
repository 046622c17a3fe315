"""Which single-token steps of the paper's Stage Two run as one launch: the edges of
the rule, as the size of a workspace tells them."""
import pytest

from paper_2609_37538_amd import avsg as A


@pytest.fixture(scope="module", autouse=True)
def _lib():
    try:
        A.load()
    except ImportError:
        pytest.skip("libavsg.so not built")


def _one_launch(batch, topk, slots, row_bytes):
    """Whether steps of the configuration run as one launch: their workspace
    then holds a ticket per request, which steps with a worker count lack."""
    a, b = (A.avsg_workspace_bytes(A.make_config(batch, topk, 1, slots, row_bytes=row_bytes, gather_workers=w))
            for w in (0, 1))
    assert a >= b > 0
    return a > b


RULE = [
    # every miss of a request within ten rounds of its workgroups' 256 threads: 32 of
    # them take one row each, of at most 2560 16-byte chunks
    (True, 2, 32, 64, (40960,)), (False, 2, 32, 64, (40964,)), (False, 2, 33, 64, (40960,)),
    (True, 2, 32, 64, (20480, 20480)), (False, 2, 32, 64, (20480, 20484)), (False, 1, 256, 1024, (65536,)),
    # 1024 threads with more slots
    (True, 2, 32, 2048, (163840,)), (False, 2, 32, 2048, (163844,)),
    # together at most 224 * 1024 threads: 8 workgroups of 256 for each of 112 requests, or
    # one for each of 896
    (True, 112, 136, 256, (2304,)), (False, 113, 136, 256, (2304,)),
    (True, 64, 256, 512, (1152,)), (True, 128, 128, 256, (1152,)), (True, 896, 16, 32, (1152,)),
    (False, 897, 16, 32, (1152,)),
    (False, 3, 64, 128, (12,)), (False, 1, 1025, 2048, (1152,)), (False, 17, 1000, 2048, (64,)),
]


@pytest.mark.parametrize("on,batch,topk,slots,row_bytes", RULE)
def test_one_launch_rule(on, batch, topk, slots, row_bytes):
    assert _one_launch(batch, topk, slots, row_bytes) == on
