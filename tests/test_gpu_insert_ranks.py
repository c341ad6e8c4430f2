"""Order of the inserted candidates, whose ranks come from ballots per wave and
1,024 candidates at a time: sizes around a wave's and a pass's end, most kept,
few kept, and a map that fills up on the way."""
import pytest

from test_gpu_insert_distance import _case

pytestmark = pytest.mark.gpu


# Candidates (centre_only: one per patch, otherwise nine).
@pytest.mark.parametrize("patches,centre_only", [
    (1, True), (63, True), (64, True), (65, True), (1023, True), (1024, True),
    (1025, True), (2049, True), (7, False), (114, False), (400, False)])
@pytest.mark.parametrize("keep", [0.1, 0.9])
def test_order_matches_the_oracle(patches, centre_only, keep):
    print("case insert ranks", patches, centre_only, keep, flush=True)
    _case(61, 500, 8000, K=patches, centre_only=centre_only, tau_q=1 - keep)


def test_a_map_that_fills_up_in_the_second_pass():
    print("case insert ranks overflow", flush=True)
    _case(62, 500, 500 + 1100, K=2000, centre_only=True, tau_q=0.1)
