"""Which way a launch takes (CPU: the rules on sizes and addresses; 256 compute units are assumed without a GPU)."""
import pytest

from paper_2608_01150_amd import api
from tests import _descs
from tests._route import HALVES, ONE_LAUNCH, TWO_PER_CU, route


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


@pytest.mark.parametrize("lengths,heads,fwd,bwd", [
    ((448,), 12, HALVES, HALVES | ONE_LAUNCH),       # 24 items forward; 48 dK/dV and 24 dQ (48 halves)
    ((1560,), 12, HALVES, ONE_LAUNCH),               # 84; 156 + 84, with halves 312
    ((2560,), 12, HALVES, HALVES),                   # 120; 240 dK/dV, 240 halves: apart
    ((2700,), 12, 0, ONE_LAUNCH),                    # 132, 264 halves
    ((256,) * 16, 8, HALVES, HALVES),                # 128, 256 halves: exactly one round; 256 dK/dV
    ((256,) * 16 + (1,), 8, 0, ONE_LAUNCH),          # 136, 264 halves
    ((128,) * 32, 8, HALVES, HALVES),                # 256 either way; 256 dK/dV
    ((128,) * 32 + (1,), 8, 0, ONE_LAUNCH)])         # 264
def test_halved_tiles_and_one_backward_launch(lengths, heads, fwd, bwd):
    d = _whole(*lengths)
    for hd in (64, 128):
        assert route(d, heads, hd, api.ZL_OP_FWD) == fwd
        assert route(d, heads, hd, api.ZL_OP_BWD) == bwd
    assert route(d, heads, 128, api.ZL_OP_FWD, dtype=api.ZL_FP32) == 0


def test_one_backward_launch_up_to_four_million_items():
    """Without work queues every item is a workgroup of 512 threads, 2^32 threads at most in a launch."""
    assert route(_whole(21504), 16384, 64, api.ZL_OP_BWD) & ONE_LAUNCH      # 252 x 16,384
    assert not route(_whole(22528), 16384, 64, api.ZL_OP_BWD) & ONE_LAUNCH  # 264 x 16,384 > 2^22
