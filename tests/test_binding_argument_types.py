"""The torch binding's answer to an argument that is no tensor, without a GPU:
a NumPy array of the right shape and type is a TypeError, for every operator
that checks its arguments in one pass."""
import numpy as np
import pytest

from paper_1802_01439_amd import dgmf

VELOCITY, SCALAR, TAU = np.zeros((3, 8, 27)), np.zeros((8, 27)), np.zeros(8)
CALLS = {
    "laplace": lambda d: dgmf.apply_laplace(d, VELOCITY),
    "helmholtz": lambda d: dgmf.apply_helmholtz(d, VELOCITY, 1.0),
    "convective": lambda d: dgmf.apply_convective(d, VELOCITY),
    "vjp": lambda d: dgmf.vjp_convective(d, VELOCITY, VELOCITY),
    "divergence": lambda d: dgmf.apply_divergence(d, VELOCITY),
    "gradient": lambda d: dgmf.apply_gradient(d, SCALAR),
    "projection": lambda d: dgmf.apply_projection(d, VELOCITY, TAU, TAU),
    "inverse_mass": lambda d: dgmf.apply_inverse_mass(d, VELOCITY),
}


@pytest.mark.parametrize("op", sorted(CALLS))
def test_numpy_array_is_a_type_error(op):
    with pytest.raises(TypeError):
        CALLS[op](dgmf.make_desc(2, (2, 2, 2), n_comp=3))
