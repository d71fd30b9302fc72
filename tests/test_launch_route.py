"""Which way a launch takes (CPU: the rules on sizes and addresses; 256 compute units are assumed without a GPU)."""
import pytest

from paper_2608_01150_amd import api
from tests import _descs
from tests._route import ONE_LAUNCH, TWO_PER_CU, route


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


@pytest.mark.parametrize("lengths,heads,hd,two", [
    ((2048,) * 8, 24, 64, False), ((2048,) * 9, 24, 64, True),      # 12,288 and 13,824 keys per compute unit
    ((1024,) * 32, 24, 64, False), ((1024,) * 33, 24, 64, True),    # 12,288 and 12,672
    ((8160,), 31, 64, False), ((8160,), 32, 64, True),              # 992 and 1024 items
    ((2048,) * 9, 24, 128, False)])                                 # d = 128 has no registers for two
def test_two_workgroups_per_cu(lengths, heads, hd, two):
    assert bool(route(_whole(*lengths), heads, hd, api.ZL_OP_FWD) & TWO_PER_CU) == two
