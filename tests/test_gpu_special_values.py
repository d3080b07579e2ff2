"""Infinities in the fp32 forward and the fp32 memory build, through the C ABI.

The fp32 products run on the bf16 matrix cores over three planes of each operand, which
cannot hold an infinity; the results are still those of fp32 arithmetic: an infinite operand
times anything but zero is infinite, with the product's sign.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2608_22883_amd as lib

    assert torch.cuda.is_available()
    return lib


def _weights(rng, d, d_m, d_c):
    w = lambda *s: rng.standard_normal(s).astype(np.float32) / np.sqrt(s[-1])  # noqa: E731
    one, zero = (lambda n: np.ones(n, np.float32)), (lambda n: np.zeros(n, np.float32))
    return dict(mem_ln_g=one(d), mem_ln_b=zero(d), W_K=w(d_m, d), W_U=w(d_m, d), q_ln_g=one(d), q_ln_b=zero(d),
                E_dep=w(2, d), W_Q=w(d_m, d), W_c1=w(d_c, d + d_m), b_c1=zero(d_c) + 3, W_c2=w(d, d_c), b_c2=zero(d),
                W_g1=w(d_c, d + d_m), b_g1=zero(d_c), w_g2=np.abs(w(d_c)), b_g2=0.0)


def _context(lib, W, d, d_m, d_c):
    return lib.Fovea(dict(d=d, d_v=d, d_m=d_m, d_c=d_c, n_depth=2, dtype=lib.FOVEA_F32, ln_eps=1e-5, rms_eps=1e-6),
                     W, device="cuda")


def _step(lib, W, n, d, d_m, d_c, h, keys, values):
    dev = "cuda"
    fv = _context(lib, W, d, d_m, d_c)
    M = keys.shape[0]
    inp = dict(mem_off=torch.tensor([0, M], device=dev), keys=torch.tensor(keys, device=dev),
               values=torch.tensor(values, device=dev), valid=None,
               node_off=torch.tensor([0, n], dtype=torch.int32, device=dev), h=torch.tensor(h, device=dev),
               depth=torch.zeros(n, dtype=torch.int32, device=dev), tau=torch.ones(1, device=dev), m_max=M,
               t_max=n, k_min=1, k_max=M)
    print(f"[gpu] special values n={n} d={d} d_m={d_m} d_c={d_c}", flush=True)
    out = fv.retrieve_fuse(inp)
    torch.cuda.synchronize()
    return out


# the layers split along K and whole, in 64- and 128-row tiles
SHAPES = [(5, 256, 128, 128), (300, 256, 128, 128), (70, 128, 64, 64), (20000, 128, 64, 64)]


def _case(n, d, d_m, d_c):
    rng = np.random.default_rng(n + d)
    W = _weights(rng, d, d_m, d_c)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    return W, f(n, d), f(16, d_m), f(16, d_m)


@pytest.mark.parametrize("n,d,d_m,d_c", SHAPES)
def test_infinite_value_row(lib, n, d, d_m, d_c):
    """+inf in one value entry (every node selects it): r, layer 1 (weights of that column
    positive), the gate and layer 2 (rows of W_c2 of one sign, or with a zero) are infinite."""
    W, h, keys, values = _case(n, d, d_m, d_c)
    j = 37
    values[3, j] = np.inf
    W["W_c1"][:, d + j] = np.abs(W["W_c1"][:, d + j]) + 1e-3
    W["W_g1"][:, d + j] = np.abs(W["W_g1"][:, d + j]) + 1e-3
    W["W_c2"] = np.abs(W["W_c2"]) + 1e-3
    W["W_c2"][1::3] *= -1
    W["W_c2"][2::3, 5] = 0
    out = _step(lib, W, n, d, d_m, d_c, h, keys, values)
    r = out.r.cpu().numpy()
    assert np.all(np.isposinf(r[:, j])) and np.all(np.isfinite(np.delete(r, j, 1)))
    assert torch.all(out.gate == 1.0)
    ho = out.h_out.cpu().numpy()
    assert np.all(np.isposinf(ho[:, 0::3])) and np.all(np.isneginf(ho[:, 1::3])) and np.all(np.isnan(ho[:, 2::3]))


@pytest.mark.parametrize("n,d,d_m,d_c", SHAPES)
def test_infinite_weight(lib, n, d, d_m, d_c):
    """+-inf in one weight of layer 2 (positive hidden values): that output is infinite, every
    other as without it."""
    W, h, keys, values = _case(n, d, d_m, d_c)
    W["b_c1"] += 20  # every hidden value positive
    ref = _step(lib, W, n, d, d_m, d_c, h, keys, values).h_out.cpu().numpy()
    W["W_c2"][9, 11], W["W_c2"][d - 1, 0] = np.inf, -np.inf
    ho = _step(lib, W, n, d, d_m, d_c, h, keys, values).h_out.cpu().numpy()
    assert np.all(np.isposinf(ho[:, 9])) and np.all(np.isneginf(ho[:, d - 1]))
    keep = [c for c in range(d) if c not in (9, d - 1)]
    assert np.array_equal(ho[:, keep], ref[:, keep])


@pytest.mark.parametrize("n,d,d_m", [(40, 128, 64), (20000, 128, 64), (40, 1024, 256)])
def test_build_infinite_weight(lib, n, d, d_m):
    """An infinite weight of W_K: that key is infinite (rows of negative mean whose entry there
    is positive: no infinities of both signs meet), values and the other keys as without it."""
    rng = np.random.default_rng(n)
    W = _weights(rng, d, d_m, 64)
    W["mem_ln_b"] += 0.1  # (times the infinite weight: infinite, not NaN)
    V = rng.standard_normal((n, d)).astype(np.float32) - 0.5
    V[:, 17] = np.abs(V[:, 17]) + 0.1
    Vt = torch.tensor(V, device="cuda")
    print(f"[gpu] infinite weight, build n={n} d={d} d_m={d_m}", flush=True)
    k0, u0 = (x.cpu().numpy() for x in _context(lib, W, d, d_m, 64).build_memory(Vt))
    W["W_K"][5, 17] = np.inf
    k1, u1 = (x.cpu().numpy() for x in _context(lib, W, d, d_m, 64).build_memory(Vt))
    assert np.all(np.isposinf(k1[:, 5])) and np.array_equal(u0, u1)
    assert np.array_equal(np.delete(k0, 5, 1), np.delete(k1, 5, 1))


def test_overflowing_planes(lib):
    """Finite operands whose partial products overflow with both signs: a weight of 3.2e38 times
    hidden values just below 2064, which is their first plane, overflows to +inf as in fp32."""
    n, d, d_m, d_c = 6, 128, 64, 64
    W, h, keys, values = _case(n, d, d_m, d_c)
    W["b_c1"] += 2057
    W["W_c2"][9, 11] = 3.2e38
    ho = _step(lib, W, n, d, d_m, d_c, h, keys, values).h_out.cpu().numpy()
    assert np.all(np.isposinf(ho[:, 9])) and np.all(np.isfinite(np.delete(ho, 9, 1)))
