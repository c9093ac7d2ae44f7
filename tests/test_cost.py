"""The flop model of the streaming kernels follows the passes that they run."""
import pytest

from paper_2002_09217_amd import cost


def further_pass(dim):
    """Flops that one pass more adds, without the terms fixed per pass."""
    fixed = {1: 3 * 16 + 20 + 18 + 20, 2: 6 * 16 + 2 * 20 + 54 + 20, 3: 2 * (3 * 16 + 3 * 20 + 81 + 20)}[dim]
    steps = [cost.stream_flops_per_node(dim, n) for n in (1, 2, 3)]
    assert steps[2] - steps[1] == steps[1] - steps[0]
    return steps[1] - steps[0] - fixed


def test_every_pass_of_one_dimension_forms_populations():
    # 2 sets x 3 moments, each 3 x 4 taps and 3 coefficients by FMA, and 3 products
    assert further_pass(1) == 6 * (2 * (12 + 3) + 3)


@pytest.mark.parametrize("dim", [2, 3])
def test_passes_before_the_last_sum_only(dim):
    # 49 FMA a row of fifteen values of f and g, and 75 to fold an axis
    assert further_pass(dim) == 2 * 49 * 15 ** (dim - 1) + 2 * 75 * dim
