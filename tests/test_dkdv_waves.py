"""The workgroup shape of the dkdv pass, by the lengths and heads of a packing (host arithmetic).  The packings are ones
that were timed with both shapes, which differ there by more than 5 %; us with four and with eight waves beside each."""
import pytest

from paper_2511_18871_amd import binding as B

SHORT = (700, [75] * 4)                                  # 1000 tokens


def one(T):
    return [(T // 2 - 64, [T // 16] * 8)]


@pytest.mark.parametrize("groups,heads,waves", [
    (one(1408), (8, 8), 8),              # 50 / 44: eight key tiles, the chip mostly idle
    (one(6400), (28, 4), 8),             # 1098 / 885: 200 workgroups
    (one(9216), (28, 4), 8),             # 1592 / 1281: 288, but the longest one counts
    (one(24576), (32, 8), 4),            # some CUs get several long ones
    ([SHORT] * 8, (28, 4), 8),           # 202 / 170: 256 workgroups, one per CU
    ([SHORT] * 9, (28, 4), 4),           # 292 / 323: the ninth group's longest tiles come second on their CUs
    ([SHORT] * 9, (4, 4), 4),            # 56 / 67
    ([SHORT] * 5, (32, 8), 8),           # 175 / 151
    ([SHORT] * 7, (32, 8), 4),           # 182 / 197
    ([SHORT] * 2, (32, 32), 8),          # 59 / 51
    ([SHORT] * 28, (32, 8), 4),          # 535 / 564
    ([SHORT] * 64, (32, 8), 4),          # beyond the sizes that are played through
])
def test_the_faster_shape_is_taken(groups, heads, waves):
    args = ([p for p, _ in groups], [len(r) for _, r in groups], [n for _, r in groups for n in r])
    assert B.sp_attn_dkdv_waves(*args, *heads) == waves


def test_one_key_tile_that_every_response_sees():
    # the prompt's tile walks 300000 rows, every other one at most 1000: eight waves, however many workgroups there are
    assert B.sp_attn_dkdv_waves([64], [300], [1000] * 300, 8, 8) == 8


def test_response_rows_walk_the_responses_only():
    pack = ([8192], [8], [40] * 8)                       # with its prompt rows, a triangle; without them, 64 tiles alike
    assert B.sp_attn_dkdv_waves(*pack, 32, 8) == 8
    assert B.sp_attn_dkdv_waves(*pack, 32, 8, B.SP_FLAG_RESPONSE_ROWS) == 4


def test_arguments_are_checked():
    with pytest.raises(B.SpAttnError):
        B.sp_attn_dkdv_waves([-1], [1], [5], 8, 8)
    with pytest.raises(B.SpAttnError):
        B.sp_attn_dkdv_waves([5], [1], [5], 8, 3)
    with pytest.raises(B.SpAttnError):
        B.sp_attn_dkdv_waves([5], [1], [5], 8, 8, 4)
