"""The binding's argument marshalling without a GPU: every call here is refused before anything is launched."""

import pytest
import torch

from paper_2105_09377_amd import binding as gs


def refused(status, call, *args, **kw):
    with pytest.raises(gs.GlensideError) as e:
        call(*args, **kw)
    assert e.value.status == status


@pytest.mark.parametrize("n0,n1", [(-1, -1), (-1, 1), (1, -2), (3, 1)])
def test_cartesian_dot_access_splits_that_do_not_exist(n0, n1):
    a = torch.zeros((4, 8), dtype=torch.bfloat16)
    # results of the shapes that "-1: all of them" would have
    lead = {1: (4,), -1: (4, 8), -2: (4, 8), 3: (4, 8)}
    out = torch.zeros(lead[n0] + lead[n1], dtype=torch.float32)
    refused(gs.GS_ERR_RANK, gs.cartesian_dot, a, a, n0, n1, out=out)
    refused(gs.GS_ERR_RANK, gs.cartesian_dot, a, a, n0, n1)
