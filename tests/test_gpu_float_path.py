"""GPU parity of the float path at the edges of its tiles, against the CPU oracle."""
import numpy as np
import pytest

from tests import pins
from tests.gpu_util import TOL, run_gpu
from tests.test_gpu_parity import _full_case

pytestmark = pytest.mark.gpu


def _inputs(N, d, H=2):
    rng = np.random.default_rng(N + d)
    x = {k: rng.standard_normal((1, H, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    return x


# one key and one key more than a group of 16, 32 and 64; 34 blocks (aggregation with 64 rows per
# wave), 129 blocks (a second tile of 128 rows with one row, a third indicator word with one bit)
@pytest.mark.timeout(300)
@pytest.mark.parametrize("N,d,phi", [(1, 128, 0), (17, 128, 1), (33, 64, 1), (65, 128, 0), (33 * 64 + 7, 128, 0),
                                     (128 * 64 + 1, 64, 1)])
def test_float_tile_edges(oracle, N, d, phi):
    _full_case(oracle, _inputs(N, d), "fp32", 0.1, 0.2, phi=phi, floor_rms=0.05 if N < 200 else 0.0)


# 8 heads x 100 blocks: enough of them for the key-side kernel that gives a workgroup half of a key
# block's keys (from 768 on, from 384 where long lists are cut, as with 7 x 109 and 4 x 96; a quarter below, as with
# 3 x 127), and four row tiles of 32 in the sums of the states, in both directions; every block of 64 rows of dK and
# dV on its own.  With and without marginal blocks
@pytest.mark.timeout(300)
@pytest.mark.parametrize("H,T,d,phi,k_l", [(8, 100, 64, 0, 0.2), (8, 100, 128, 1, 0.2), (8, 100, 128, 0, 1.0),
                                           (8, 96, 64, 1, 0.1), (7, 109, 64, 0, 0.1), (4, 96, 128, 1, 0.2),
                                           (3, 127, 64, 0, 0.2)])
def test_float_calls_of_many_blocks(oracle, say, H, T, d, phi, k_l):
    _full_case(oracle, _inputs(64 * T - 9, d, H), "fp32", 0.1, k_l, phi=phi)
    say(f"{H} heads x {T} blocks, d = {d}: done")


@pytest.mark.parametrize("T", [12, 40, 130])
def test_a_state_that_is_not_finite_reaches_only_the_rows_that_add_it(oracle, T):
    x = _inputs(64 * T, 64, H=1)
    x["V"][0, 0, 64 * 3 + 5, 7] = np.inf
    x["V"][0, 0, 64 * (T - 1), 9] = np.nan
    Mc = oracle.build_mask(x["Q"], x["K"], 0.1, 0.4)
    f = oracle.forward(x["Q"], x["K"], x["V"], x["Proj"], Mc)
    r = run_gpu(x, "fp32", 0.1, 0.4, backward=False)
    fin = np.isfinite(f["Hi"])
    assert not fin.all() and fin.any()
    assert np.array_equal(np.isfinite(r["Hi"]), fin)
    assert np.abs(r["Hi"][fin] - f["Hi"][fin]).max() <= 1e-5 * np.abs(f["Hi"][fin]).max()


@pytest.mark.parametrize("T,d", [(12, 64), (40, 64), (130, 128)])
def test_states_of_any_magnitude(T, d):
    # V and dO scaled by powers of two, from where a state's last bits are the smallest floats to where a scaled sum of
    # states would overflow; all states, or every second feature, so that the columns differ.  A state is rounded
    # to 2^-149 at most once per product and sum (64 tokens, T blocks), and either side's float sums to 2^-24 of their
    # terms' magnitudes in each addition
    import torch
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    N = 64 * T - 5
    Q, K, V, dO = (torch.randn(1, 1, N, d, generator=g, device="cuda") for _ in range(4))
    W = 0.05 * torch.randn(d, d, generator=g, device="cuda")
    p = sla.make_params(1, 1, N, d, 0.1, 0.2, torch.float32)
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)

    def states(V):
        return sla.saved_views(p, sla.sla_forward(p, Q, K, V, W, Mc, luts)[1])["Hi"].double()   # [.., c, e]

    _, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
    grads = lambda dO: [t.double() for t in sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO)[1:3]]
    ref, mag, gref = states(V), states(V.abs()), grads(dO)
    for e in (-122, -116, -104, -60, 60, 93, 101, 112):
        for step in (1, 2):
            f = torch.ones(d, device="cuda", dtype=torch.float64)
            f[::step] = 2.0 ** e
            got = states((V.double() * f).float())
            bound = 2 * (64 + T) * 2.0 ** -24 * mag * f + 64 * T * 2.0 ** -149
            assert bool(((got - ref * f).abs() <= bound).all()), (e, step)
        for a, b in zip(grads((dO.double() * 2.0 ** e).float()) if e < 0 else (), gref):
            # (rounding to 2^-149 in each of its sums and products: no more than 2^-149 / 2^(e - 6) of the norm each)
            assert (a * 2.0 ** -e - b).norm() <= (1e-6 + 64 * 2.0 ** (-149 - e)) * b.norm(), e


@pytest.mark.parametrize("T,d,k_h", [(1, 64, 0.0), (1, 128, 0.0), (2, 64, 0.0), (3, 128, 0.3), (4, 64, 0.2), (4, 128, 0.0),
                                     (5, 64, 0.2), (5, 128, 0.0)])
def test_sums_of_the_states_of_a_few_blocks(oracle, T, d, k_h):
    # up to eight blocks one thread holds its columns of every state; every row marginal or some, a ragged last block, more heads than one
    x = _inputs(64 * T - 9, d, H=3)
    _full_case(oracle, x, "fp32", k_h, 0.2, floor_rms=0.05 if T < 4 else 0.0)
    if T == 1:
        return
    x["V"][0, 1, 5, 7] = np.inf
    x["V"][0, 2, 64 * (T - 1), 9] = np.nan
    Mc = oracle.build_mask(x["Q"], x["K"], k_h, 0.2)
    f = oracle.forward(x["Q"], x["K"], x["V"], x["Proj"], Mc)
    r = run_gpu(x, "fp32", k_h, 0.2, backward=False)
    fin = np.isfinite(f["Hi"])
    assert not fin.all() and np.array_equal(np.isfinite(r["Hi"]), fin)
    assert np.abs(r["Hi"][fin] - f["Hi"][fin]).max() <= 1e-5 * np.abs(f["Hi"][fin]).max()


@pytest.mark.parametrize("T,d", [(4, 128), (5, 64), (7, 128), (8, 64), (8, 128), (9, 64)])
def test_state_sums_of_many_short_heads(T, d):
    # the sums of a head are the same bits among a few heads and among many, where up to eight blocks a thread takes
    # four columns instead of one; and they are what 64 bits give, within the bound for sums of T floats
    import torch
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    H, N = 130, T * 64 - 9
    Q, K, V = (torch.randn(1, H, N, d, generator=g, device="cuda") for _ in range(3))
    V[0, 3, 70, 5] = float("inf")
    W = torch.zeros(d, d, device="cuda")

    def states(q, k, v):
        p = sla.make_params(1, q.shape[1], N, d, 0.2, 0.2, torch.float32)
        Mc, luts, _ = sla.sla_build_mask(p, q, k)
        _, saved = sla.sla_forward(p, q, k, v, W, Mc, luts)
        return Mc, sla.saved_views(p, saved)

    _, many = states(Q, K, V)
    cut = lambda t: t[:, 2:5].contiguous()
    Mc, few = states(cut(Q), cut(K), cut(V))
    for n in ("Hi", "Zi"):
        assert torch.equal(many[n][:, 2:5].contiguous().view(torch.int32), few[n].contiguous().view(torch.int32)), n
        assert bool(torch.isfinite(few[n]).all()) == (n == "Zi")
    # head 2: the sum over its marginal blocks, from single-block states (exact in 64 bits up to phi's own rounding)
    q, k, v = (t[:, :1].double() for t in (cut(Q), cut(K), cut(V)))
    h = [torch.softmax(k[:, :, 64 * j:64 * j + 64], -1).transpose(-1, -2) @ v[:, :, 64 * j:64 * j + 64] for j in range(T)]
    m = [torch.softmax(k[:, :, 64 * j:64 * j + 64], -1).transpose(-1, -2) @ v[:, :, 64 * j:64 * j + 64].abs() for j in range(T)]
    for i in range(T):
        js = [j for j in range(T) if int(Mc[0, 0, i, j]) == 0]
        ref, mag = (sum((x[j] for j in js), torch.zeros_like(h[0])) for x in (h, m))
        # 2^-24 for each of 64 products and T sums, and a few for phi
        assert bool(((few["Hi"][:, :1, i].double() - ref).abs() <= (64 + T + 16) * 2.0 ** -24 * mag).all())


@pytest.mark.parametrize("T,d", [(257, 64), (300, 128), (380, 64)])
def test_key_side_of_one_and_two_heads_above_256_blocks(oracle, T, d):
    # fewer than 768 blocks in all, whole lists: a quarter of a key block per workgroup with one head and with two,
    # so a head's gradients are the same bits in both; against the oracle
    import torch
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(T)
    N = T * 64 - 21
    x = {k: rng.standard_normal((1, 2, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["K"][:, :, 640:704] += 0.4   # a longer list
    x["Q"] += 0.2
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    two = run_gpu(x, "fp32", 0.01, 0.3)
    x1 = {k: v[:, :1] if v.ndim == 4 else v for k, v in x.items()}
    one = run_gpu(x1, "fp32", 0.01, 0.3)
    for k in ("dK", "dV"):
        assert np.array_equal(one[k], two[k][:, :1]), k
    if T == 300:
        f = oracle.forward(x1["Q"], x1["K"], x1["V"], x1["Proj"], one["Mc"])
        g = oracle.backward(x1["Q"], x1["K"], x1["V"], x1["Proj"], one["Mc"], f, x1["dO"])
        for k in ("dQ", "dK", "dV", "dW"):
            assert pins.rel_l2(one[k], g[k]) <= TOL["fp32"], k


@pytest.mark.parametrize("T,d,k_h,H", [(160, 64, 0.2, 3), (48, 64, 0.3, 8), (122, 128, 0.2, 4)])
def test_key_side_of_whole_lists_up_to_256_blocks(T, d, k_h, H):
    # lists too dense to be cut, 384 to 767 blocks in all: a quarter of a key block per workgroup, as with one head
    # less, so the gradients of the other heads are the same bits in both calls
    x = _inputs(64 * T - 9, d, H)
    less = {k: v[:, :H - 1] if v.ndim == 4 else v for k, v in x.items()}
    a, b = run_gpu(x, "fp32", k_h, 0.1), run_gpu(less, "fp32", k_h, 0.1)
    for k in ("dQ", "dK", "dV"):
        assert np.array_equal(a[k][:, :H - 1], b[k]), k
