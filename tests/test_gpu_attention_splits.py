"""Attention whose keys are split over workgroups, end to end against the
float64 oracle: a grouped-query bf16 pair (head dims 64 and 128, 4 query heads
per KV head) over prompts long enough that the rollout (one and two row tiles
of 16 rows, four and eight waves), the verification (row tiles of one or two
per wave) and the last row of the prompt pass each take several key splits.
The tolerance is the harness's for bf16 weights."""
import pytest

import cdsl_inputs as ci
from cdsl_harness import assert_full_or_tie, make_engine, make_setup, run_and_compare

pytestmark = pytest.mark.gpu

DRAFT = ci.ModelShape(2, 512, 8, 2, 1024, 4096)
TARGET = ci.ModelShape(3, 1024, 8, 2, 2048, 4096)


@pytest.mark.parametrize("B,k,d,L", [
    (3, 8, 4, 1201),    # rollout: 32 rows on eight waves; verification: 128 rows, two tiles per wave
    (2, 3, 3, 1090),    # rollout: 12 rows, four key groups; verification: 36 rows, one tile per wave
    (16, 5, 5, 333),    # rollout unsplit, verification: 100 rows (seven tiles), two tiles per wave
])
def test_key_splits_match_oracle(B, k, d, L):
    s = make_setup("small", draft=DRAFT, target=TARGET, batch=B, prompt_len=L, k=k, d=d)
    make_engine(s, B=B, max_steps=3, k=k, d=d)
    try:
        st, reps = run_and_compare(s, B=B, steps=2, check_prompts=[0, B - 1], k=k, d=d)
        assert_full_or_tie(reps, 2)
        st.prefix.free()
    finally:
        s.engine.close()
