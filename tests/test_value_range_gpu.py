"""Values at the ends of the float32 range: what is finite in exact arithmetic with normalised keys comes out finite.

A bf16 or float32 key of norm 1e13 against a state of 1e28 has a raw product beyond float32 although k^ S is far inside."""
import numpy as np
import pytest

from parity_utils import check_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [2, 3, 4])
@pytest.mark.parametrize("d,heads", [(16, 3), (32, 3), (64, 3), (96, 3), (128, 3),
                                     (32, 200), (64, 200), (96, 140), (128, 140),    # shared S rows of the segment modes
                                     (128, 300), (64, 800)])                         # waves of 32 columns
def test_large_keys_against_a_large_state(d, heads, mode, dtype):
    if d == 16 and mode != 2:
        mode = 2   # no segment modes
    rng = np.random.default_rng(d + heads)
    T = 37
    q, k, v = (rng.standard_normal((1, heads, T, d)).astype(np.float32) for _ in range(3))
    S0 = rng.standard_normal((1, heads, d, d)).astype(np.float32)
    scale = np.float32(10.0) ** rng.integers(8, 15, size=(1, heads, T, 1)).astype(np.float32)   # k and its square in range
    errs, _, _ = check_parity(q * np.float32(1e-20), k * scale, v * np.float32(1e28), S0 * np.float32(1e28), dtype=dtype,
                              mode=mode)
    print(d, heads, mode, dtype, errs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_v,T", [(16, 64), (16, 300), (64, 300)])
def test_large_keys_against_a_large_state_in_spans_of_256_tokens(d_v, T, dtype):
    """Key heads of 16 from 64 tokens on: the state passes through the affine maps of the blocks of a span."""
    rng = np.random.default_rng(T)
    q, k = (rng.standard_normal((1, 3, T, 16)).astype(np.float32) for _ in range(2))
    v = rng.standard_normal((1, 3, T, d_v)).astype(np.float32)
    S0 = rng.standard_normal((1, 3, d_v, 16)).astype(np.float32)
    scale = np.float32(10.0) ** rng.integers(8, 15, size=(1, 3, T, 1)).astype(np.float32)
    errs, _, _ = check_parity(q * np.float32(1e-20), k * scale, v * np.float32(1e28), S0 * np.float32(1e28), dtype=dtype,
                              mode=2)
    print(d_v, T, dtype, errs)
