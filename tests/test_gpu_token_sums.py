"""The learned dustbin tokens' gradient sums at the sizes where two sums stop sharing a launch."""
import pytest


# (the second sum's partial sums, ceil(L / 1024) d floats, take the place of two vectors of L + 1 floats, rounded up to 4)
@pytest.mark.gpu
@pytest.mark.parametrize("d,L", [(64, 27), (64, 28), (128, 59), (128, 60), (32, 5), (128, 1025)])
def test_token_sums_with_and_without_room(d, L):
    """Every output against the oracle, within the parity tests' fp32 tolerance."""
    from tests.test_gpu_parity import test_learned_dustbin_tokens as check
    check("f32", d, 2, L)
