"""Which way a launch takes (CPU: the rules on sizes and addresses; 256 compute units are assumed without a GPU)."""
import pytest

from paper_2608_01150_amd import api
from tests import _descs
from tests._route import ONE_LAUNCH, route


def _whole(*lengths):
    cu, m = [0], len(lengths)
    for n in lengths:
        cu.append(cu[-1] + n)
    return _descs.desc(cu_q=cu, kind=(0,) * m, kv_first=range(m), kv_count=(1,) * m, cu_k=cu, block_index=(0,) * m,
                       num_slots=0)


@pytest.mark.parametrize("lengths", [(1560,), (1560,) * 16])
def test_gradients_in_place_take_two_launches(lengths):
    """dq in the memory of q or dout, whole or in part: dK/dV must be done before dQ writes."""
    d, H, hd = _whole(*lengths), 12, 128
    n = sum(lengths) * H * hd * 2
    q, do = 1 << 40, 2 << 40
    for dq, one in ((3 << 40, True), (q + n, True), (q - n, True), (do + n, True), (do - n, True), (q, False),
                    (do, False), (q + n - 256, False), (q - n + 256, False), (do + 256, False)):
        assert bool(route(d, H, hd, api.ZL_OP_BWD, q=q, dout=do, dq=dq) & ONE_LAUNCH) == one, hex(dq)
