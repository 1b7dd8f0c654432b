"""Which partials of the one-pass X-cache kernel leave through the L2s to the memory side: the many that would be written back between the launches,
not the few for which the way there is the longer one (up to 1.8 MB 0.25 us a call, from 2.6 MB 0.2 to 1.2 the other way)."""
import pytest

from launch_rules import one_pass_through


@pytest.mark.parametrize("nbytes,through", [(4 * 640, False), (900_000, False), (1_800_000, False), (2_650_000, True), (16_777_216, True), (1 << 33, True)])
def test_few_partials_stay_in_the_l2s(nbytes, through):
    assert one_pass_through(nbytes) == through
