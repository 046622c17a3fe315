"""Set-up of the step without a handle (avsg_step_static): pointer tables and row
counts that fill one launch's arguments, exceed them by a request and take
several launches, and empty tables whatever the last call left."""
import pytest

import workload as W
from test_zz_no_alloc import _run_pair

pytestmark = pytest.mark.gpu


# two streams: 5 values per request, 480 per launch, up to 48 in the short form
@pytest.mark.parametrize("batch", [9, 10, 96, 97, 300])
@pytest.mark.parametrize("gather_mode", [0, 6], ids=["balanced", "resident"])
def test_static_setup_many_requests(batch, gather_mode):
    spec = W.custom_spec(name=f"static_setup_{batch}", batch=batch, topk=16, slots=64, n_q=2, steps=4, ctx=200,
                         row_bytes=(32, 132))
    _run_pair(spec, gather_mode)


def test_static_setup_dual_pointer():
    spec = W.custom_spec(name="static_setup_dp", batch=161, topk=16, slots=16, n_q=1, steps=4, ctx=100,
                         row_bytes=(32,))
    _run_pair(spec, 0, match_mode=1)
