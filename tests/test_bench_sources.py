"""Sources that the counter summaries of the benchmark are tied to."""
import re

import pytest

import bench


def _text():
    return "".join(open(f).read() for f in bench.KERNEL_SRC)


@pytest.mark.parametrize("name", ["k_dns_steps", "k_les_steps", "ms_shape", "collide_q", "ms_tile"])
def test_summaries_are_tied_to_kernels_and_their_shapes(name):
    """What sets the bytes of a launch, its kernel and its strips and segments, is defined
    in the hashed sources: a change of either asks for new counters."""
    assert re.search(rf"^[\w:<>&* ]*\b{name}\([^;]*?\)\s*\{{", _text(), flags=re.M)


def test_summaries_do_not_hang_on_the_plan():
    """Costs by which launches are chosen leave the bytes of each as they are."""
    assert "launch_costs" not in re.sub(r"//[^\n]*", "", _text())
