"""How a float32 call spreads its rows and keys over workgroups, by the lengths and heads of a packing (host arithmetic).  The packings
are ones that were timed in every shape; us of the shape that is taken and of the next best beside each (forward; dq; dkdv)."""
import pytest

from paper_2511_18871_amd import binding as B


@pytest.mark.parametrize("groups,heads,head_dim,rows", [
    ([(64, [32] * 4)], (2, 2), 64, (1, 1, 1)),
    ([(191, [38] * 5)], (4, 2), 64, (16, 16, 1)),           # 11 / 19; 14 / 26; 37 / 33
    ([(32, [20] * 40)], (4, 2), 128, (16, 16, 1)),          # 13 / 27; 13 / 42; 69 / 115: few keys that every row sees
    ([(8, [30] * 100)], (4, 2), 64, (16, 16, 1)),           # 30 / 32; 30 / 48; 133 / 210
    ([(0, [3] * 3)] * 25, (4, 2), 128, (4, 4, 1)),          # 14 / 20; 19 / 21; a block of 16 spans three groups
    ([(16, [16] * 4)] * 75, (4, 4), 64, (16, 16, 16)),      # 44 / 57; 42 / 88; 69 / 101: groups that fill their blocks
    ([(100, [90] * 6)] * 9, (4, 2), 128, (16, 16, 16)),     # 90 / 274; 110 / 459; 180 / 666
])
def test_the_faster_shape_is_taken(groups, heads, head_dim, rows):
    args = ([p for p, _ in groups], [len(r) for _, r in groups], [n for _, r in groups for n in r])
    assert B.sp_attn_f32_rows(*args, *heads, head_dim) == rows


def test_response_rows_walk_the_responses_only():
    # the prompt's keys are seen by 40 rows instead of 4136
    assert B.sp_attn_f32_rows([4096], [1], [40], 2, 2, 64)[2] == 16
    assert B.sp_attn_f32_rows([8], [1], [4096], 2, 2, 64, B.SP_FLAG_RESPONSE_ROWS) == B.sp_attn_f32_rows([8], [1], [4096], 2, 2, 64)


def test_arguments_are_checked():
    for bad in (([-1], [1], [5], 8, 8, 64), ([5], [1], [5], 8, 3, 64), ([5], [1], [5], 8, 8, 96), ([5], [1], [5], 8, 8, 64, 4)):
        with pytest.raises(B.SpAttnError):
            B.sp_attn_f32_rows(*bad)
