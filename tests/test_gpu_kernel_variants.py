"""The kernel variants a call may be routed to, each at the sizes where it can go wrong: edges of tiles, remainders, the
smallest and largest of its range.  References in float64; tolerances are bounds derived from the operand types."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
U32 = 2.0 ** -24  # half a unit in the last place of a 24-bit significand


@pytest.fixture(scope="module")
def H():
    from paper_2110_08633_amd import hydra
    return hydra


def randn(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda")


def stored(x, ld, shift):
    """x in a buffer with leading dimension ld that starts shift elements past a 256-byte boundary; the gap between the
    rows is NaN.  Returns the matrix view."""
    buf = torch.full((x.shape[0] * ld + shift,), float("nan"), dtype=x.dtype, device="cuda")
    v = buf[shift:].view(x.shape[0], ld)
    v[:, :x.shape[1]] = x
    return v


# M, N, K, extra leading dimension, element shift.  16-byte loads: all of K, M, N, leading dimensions and shift multiples
# of 4; else 4-byte loads.  From 640 64x64 tiles on those are used, below 32x32 tiles.
F32_CASES = [(1, 1, 1, 0, 0), (33, 31, 7, 1, 0), (32, 32, 64, 0, 0), (36, 28, 68, 4, 0), (64, 96, 4, 0, 1),
             (100, 52, 129, 0, 0), (1604, 1700, 36, 4, 0), (1664, 1600, 32, 0, 0), (1601, 1663, 33, 3, 2),
             (2, 3, 5, 7340040, 0)]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K,extra,shift", F32_CASES)
def test_gemm_f32_variants(H, ta, tb, M, N, K, extra, shift):
    A, B, resid = randn(M + K, M, K), randn(N + K + 1, K, N), randn(M + N + 2, M, N)
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    dA, dB = stored(As, As.shape[1] + extra, shift), stored(Bs, Bs.shape[1] + extra, shift)
    ldc = N + (extra if extra < 100 else 0)
    out = torch.full((M, ldc), 7.0, device="cuda")
    H.hydra_op_gemm(0, ta, tb, M, N, K, 0.5, dA, As.shape[1] + extra, dB, Bs.shape[1] + extra, None,
                    stored(resid, ldc, 0), out, None, ldc)
    torch.cuda.synchronize()
    ref = 0.5 * (A.double() @ B.double()) + resid.double()
    # a sum of K products in any order, its scaling and the residual: each of the K + 2 roundings is at most U32 of the
    # sum of magnitudes
    bound = (K + 2) * U32 * (0.5 * (A.double().abs() @ B.double().abs()) + resid.double().abs())
    assert ((out[:, :N].double() - ref).abs() <= bound).all()
    assert (out[:, N:] == 7.0).all()
