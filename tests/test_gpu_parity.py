"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element,
on the same seeded inputs.  Masks and lookup tables bit-exact; floating-point tensors by
relative L2 (1e-5 for float tensors, 1e-2 for bf16 tensors)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_24006_amd import workloads as wl
from tests import pins
from tests.gpu_util import BLOCK_TOL, TOL, check_luts, max_block_rel_l2, per_tile, run_gpu

pytestmark = pytest.mark.gpu


def _oracle_all(oracle, x, k_h, k_l, phi=0, backward=True, bq=64):
    Mc, s = oracle.build_mask(x["Q"], x["K"], k_h, k_l, bq=bq, return_scores=True)
    f = oracle.forward(x["Q"], x["K"], x["V"], x["Proj"], Mc, phi=phi, bq=bq)
    g = oracle.backward(x["Q"], x["K"], x["V"], x["Proj"], Mc, f, x["dO"], phi=phi, bq=bq) if backward else {}
    return Mc, s, f, g


def _compare(name, got, ref, tol, floor_rms=0.0, block_tol=None, token_axis=2, rows=64):
    """Whole-tensor relative L2 <= tol and, with block_tol, the same measure on every block of
    `rows` consecutive indices of token_axis <= block_tol (one bad row cannot hide in a long
    tensor).  floor_rms > 0 (short sequences' gradients only, see the callers) measures the error
    against a norm of at least floor_rms per element."""
    if np.all(ref == 0):
        assert np.all(got == 0), f"{name}: expected exact zeros"
        return
    err = pins.rel_l2(got, ref)
    print(f"  {name}: rel_l2 = {err:.3e} (tol {tol:g})", flush=True)
    # a reference that is pure rounding noise (a gradient that vanishes identically, e.g. dQ
    # of a one-token sequence) is compared absolutely, at the same tolerance
    if np.abs(ref).max() < 1e-12:
        assert np.abs(got).max() <= tol, f"{name}: expected ~0, got {np.abs(got).max():.3e}"
        return
    # floor_rms: where a key block holds one or a few keys, P is 1 (or close) and dS = P (dP - D)
    # cancels exactly in most rows: the norm of the reference gradient is then set by a handful
    # of rows while float rounding noise comes from all of them; the error is measured against a
    # norm of at least floor_rms per element (inputs have unit variance)
    scale = max(np.linalg.norm(ref.ravel()), floor_rms * np.sqrt(ref.size))
    err = np.linalg.norm((got - ref).ravel()) / scale
    assert err <= tol, f"{name}: rel L2 {err:.3e} > {tol:g}"
    if block_tol is not None and floor_rms == 0.0:
        berr, where = max_block_rel_l2(got, ref, token_axis, rows)
        print(f"  {name}: worst block rel_l2 = {berr:.3e} at {where} (tol {block_tol:g})", flush=True)
        assert berr <= block_tol, f"{name}: block {where} rel L2 {berr:.3e} > {block_tol:g}"


def _full_case(oracle, x, dtype, k_h, k_l, phi=0, floor_rms=0.0, bq=64, backward=True):
    print(f"case shape={x['Q'].shape} dtype={dtype} k_h={k_h} k_l={k_l} phi={phi} bq={bq}", flush=True)
    Mc, s, f, g = _oracle_all(oracle, x, k_h, k_l, phi, backward=backward, bq=bq)
    r = run_gpu(x, dtype, k_h, k_l, phi, backward=backward, bq=bq)
    # mask step: bit-exact
    assert np.array_equal(r["scores"], s), "pooled scores differ bitwise"
    assert np.array_equal(r["Mc"], Mc), "mask differs"
    # tables and saved states are kept per 64-token query tile: a tile has its query block's row
    T, rq = Mc.shape[-1], bq // 64
    check_luts(per_tile(r["Mc"], rq, T), r["row_idx"], r["col_ptr"], r["col_rows"], r["ind"], r["ind_t"],
               r["col_order"])
    tol, btol = TOL[dtype], BLOCK_TOL[dtype]
    for k in ("O", "Os", "Ol"):
        _compare(k, r[k], f[k], tol, block_tol=btol)
    for k in ("Hi", "Zi"):   # one state per 64-token tile: every state on its own
        _compare(k, r[k], per_tile(f[k], rq, T), tol, block_tol=btol, rows=1)
    fin = np.isfinite(f["L"])
    assert np.array_equal(np.isfinite(r["L"]), fin)
    if fin.any():
        _compare("L", r["L"][fin], f["L"][fin], tol)
    for k in ("dQ", "dK", "dV", "dW") if backward else ():
        _compare(k, r[k], g[k], tol, floor_rms, block_tol=None if k == "dW" else btol)


@pytest.mark.parametrize("name", ["tiny", "small_fp32", "small_bf16", "small_bf16_d64"])
def test_workload_parity(oracle, name):
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    _full_case(oracle, x, w.dtype, w.k_h, w.k_l)


@pytest.mark.parametrize("k_h,k_l", [(1.0, 0.1), (0.0, 0.0), (0.0, 0.3), (0.4, 0.6), (0.05, 0.9)])
@pytest.mark.parametrize("name", ["small_fp32", "small_bf16", "small_bf16_d64"])
def test_degenerate_masks(oracle, name, k_h, k_l):
    # all critical (dense attention), all marginal (linear attention), no critical block,
    # no marginal block
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    _full_case(oracle, x, w.dtype, k_h, k_l)


@pytest.mark.parametrize("name", ["small_fp32", "small_bf16"])
def test_elu_feature_map(oracle, name):
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    _full_case(oracle, x, w.dtype, w.k_h, w.k_l, phi=1)


@pytest.mark.parametrize("name,bq,k_h,k_l", [
    ("small_bf16", 128, 0.10, 0.10),       # 18 tiles in 9 blocks; last block ragged inside its second tile
    ("small_bf16_d64", 128, 0.12, 0.15),   # 15 tiles: the last block has one tile only
    ("small_bf16_d64", 192, 0.12, 0.15),   # 5 blocks of 3 tiles
    ("small_fp32", 128, 0.15, 0.20),
    ("small_fp32", 256, 0.15, 0.20),       # 9 tiles in blocks of 4, 4, 1
    ("small_bf16", 256, 0.0, 0.3),         # no critical block
    ("small_bf16", 128, 0.4, 0.6),         # no marginal block
])
def test_query_blocks_of_several_tiles(oracle, wide_tiles, name, bq, k_h, k_l):
    # b_q = 128, 192, 256 with b_kv = 64: the mask is predicted per block of b_q queries (pooling,
    # scores and classification on T_q rows); the oracle computes with the b_q x 64 blocks
    # directly, the library gives every 64-token tile of a query block that block's mask row
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    _full_case(oracle, x, w.dtype, k_h, k_l, bq=bq)


@pytest.mark.parametrize("bq", [128, 256])
def test_query_blocks_of_several_tiles_mid_length(oracle, wide_tiles, bq):
    # 41 tiles (ragged tail of 5 tokens), enough key blocks for the matrix-core state aggregation
    N, d = 2565, 128
    rng = np.random.default_rng(N + bq)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, 2, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    _full_case(oracle, x, "bf16", 0.1, 0.2, bq=bq)


@pytest.mark.parametrize("name,scale,backward", [
    ("small_bf16", 0.02, True), ("small_bf16", 2.0, True), ("small_bf16", 6.0, False),
    ("small_fp32", 0.02, True), ("small_fp32", 2.0, True), ("small_fp32", 6.0, True)])
def test_small_and_large_score_magnitudes(oracle, name, scale, backward):
    # nearly uniform attention (scores ~ 1e-3) and peaked attention (raw scores of a hundred and
    # more before the 1/sqrt(d): exponent range of the online softmax and of its lazy rescaling).
    # At the largest scale the bf16 case compares the forward pass only: with P close to one-hot,
    # dS = P (dP - D) is a small difference of terms of which D comes from the O^s saved in the
    # storage type, so in bf16 the gradients of any implementation that follows Alg. 2 lose
    # digits there (1.6 % on dQ), which says nothing about the kernels.  Float tensors save O^s
    # in float and are compared in full.
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    x["Q"] = x["Q"] * np.float32(scale)
    x["K"] = x["K"] * np.float32(scale)
    if w.dtype == "bf16":
        x["Q"], x["K"] = wl.round_to_bf16(x["Q"]), wl.round_to_bf16(x["K"])
    _full_case(oracle, x, w.dtype, w.k_h, w.k_l, backward=backward)


@pytest.mark.parametrize("mag", [1.0e6, 1.1e6, 3.0e9, 1.0e10, 1.0e20, 1.0e30])
@pytest.mark.parametrize("d", [64, 128])
def test_tokens_with_very_large_features(oracle, wide_tiles, d, mag):
    # phi(Q) is formed relative to the token's largest feature, whatever its size (several features share it here);
    # K is as small as the scores need to stay of order one.  Both sides of the size up to which the exponent
    # is one fused multiply-add.
    rng = np.random.default_rng(int(np.log2(mag)) + d)
    N = 5 * 64 + 9
    x = {k: rng.standard_normal((1, 2, N, d)).astype(np.float32) for k in ("Q", "K", "V")}
    for sign, first in ((1.0, 0), (-1.0, 1)):
        big = x["Q"][:, :, first::3]
        x["Q"][:, :, first::3] = sign * mag * (1.0 + 0.01 * big)
    x["K"] *= 0.5 / mag
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    x = {k: wl.round_to_bf16(v) for k, v in x.items()}
    Mc, _, f, _ = _oracle_all(oracle, x, 0.4, 0.0, backward=False, bq=128)
    r = run_gpu(x, "bf16", 0.4, 0.0, backward=False, bq=128)
    assert np.array_equal(r["Mc"], Mc)
    for k in ("O", "Os", "Ol"):
        assert np.isfinite(r[k]).all(), k
        _compare(k, r[k], f[k], TOL["bf16"], block_tol=BLOCK_TOL["bf16"])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("e", [-100, 100, 120])
def test_values_near_the_ends_of_the_float_range(wide_tiles, d, e):
    # V scaled by a power of two scales O, O^l exactly (no sum leaves the normal floats): with nearly equal features
    # phi(Q) is as flat as it gets, and its sums over the features must not overflow before O^l does
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    N = 20 * 64 - 5
    Q, K, V = (torch.randn(1, 2, N, d, generator=g, device="cuda") for _ in range(3))
    Q, K, V = (0.1 * Q).bfloat16(), K.bfloat16(), (0.25 * V + 1).bfloat16()
    W = (0.02 * torch.randn(d, d, generator=g, device="cuda")).bfloat16()
    p = sla.make_params(1, 2, N, d, 0.1, 0.2, torch.bfloat16, bq=128)
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)

    def out(V):
        O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
        return O.double(), sla.saved_views(p, saved)["Ol"].double()

    for a, b in zip(out((V.double() * 2.0 ** e).bfloat16()), out(V)):
        assert torch.equal(a, b * 2.0 ** e)


@pytest.mark.parametrize("N", [1, 63, 64, 65, 130])
def test_short_sequences(oracle, N):
    rng = np.random.default_rng(N)
    d = 64
    x = {k: rng.standard_normal((1, 2, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    _full_case(oracle, x, "fp32", 0.34, 0.34, floor_rms=0.05)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_h", range(9))
def test_every_beginning_and_end_of_the_forward_loop(oracle, wide_tiles, n_h, d):
    # the forward kernel requests tiles two steps ahead, the aggregated state as the tile behind the
    # last one, and runs all but its last steps without conditions: every number of critical blocks
    # from none to beyond that, with marginal blocks and without, a ragged last block, query blocks of
    # one tile and of two (four-wave and eight-wave kernels)
    T = 13
    N = 64 * T - 9
    rng = np.random.default_rng(100 * n_h + d)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, 2, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    for bq, k_l in ((64, 0.1), (64, 1.0), (128, 0.1), (128, 1.0)):
        _full_case(oracle, x, "bf16", n_h / T, k_l, bq=bq, backward=False)


@pytest.mark.parametrize("T,bq,H", [(1, 64, 11), (3, 64, 8), (7, 64, 1), (8, 64, 11), (9, 64, 11), (15, 128, 9),
                                    (16, 128, 11), (17, 128, 3)])
def test_heads_of_a_few_tiles(oracle, wide_tiles, T, bq, H):
    # up to eight workgroups a head stays on one XCD, eight heads to a row of the grid: numbers of
    # heads that are no multiple of eight, both sides of the line for four-wave workgroups (8, 9
    # tiles) and for eight-wave ones (16, 17 tiles of query blocks of two)
    N, d = 64 * T - 9, 64
    rng = np.random.default_rng(T + H)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, H, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    for k_h, k_l in ((0.3, 0.3), (1.0, 0.0), (0.0, 0.0)):
        _full_case(oracle, x, "bf16", k_h, k_l, bq=bq, backward=False)


@pytest.mark.parametrize("N,d", [(2565, 128), (4096, 64), (2048, 128)])
def test_bf16_mid_length_sequences(oracle, N, d):
    # 33..64 blocks: the short-sequence state aggregation with two row tiles, a ragged tail and
    # an exact multiple of the block size
    rng = np.random.default_rng(N + d)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, 2, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    _full_case(oracle, x, "bf16", 0.1, 0.2)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("N,d", [(300 * 64 - 9, 128), (71 * 64 + 3, 64)])
def test_bf16_ragged_tiles_of_the_state_aggregation(oracle, N, d):
    # 300 blocks: two row tiles of the aggregation GEMM, the second with 44 rows, five indicator
    # words per row, the last with 44 bits; 72 blocks: one ragged row tile, two words.  Forward and
    # backward (the column-wise aggregation uses the transposed indicator)
    rng = np.random.default_rng(N + d)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, 2, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    _full_case(oracle, x, "bf16", 0.05, 0.15)


@pytest.mark.timeout(300)
def test_many_long_heads(oracle):
    # 32 (batch x head) problems of 128 blocks: the launch order of the dK/dV kernel in which every
    # XCD takes whole heads one after the other (chosen from 32 problems and 128 blocks on), with a
    # ragged tail; all heads against the oracle
    B, H, N, d = 4, 8, 128 * 64 - 17, 64
    rng = np.random.default_rng(4128)
    x = {k: wl.round_to_bf16(rng.standard_normal((B, H, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    _full_case(oracle, x, "bf16", 0.05, 0.10)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("T,d,tail", [(150, 128, 23), (128, 64, 0), (200, 64, 63)])
def test_key_blocks_that_nearly_every_query_block_selects(oracle, T, d, tail):
    # a few key blocks whose pooled key points along the direction shared by every query: their
    # column lists hold (nearly) all T query tiles, so the column-wise backward kernel walks them in
    # the longest walks the kernel can be given (its launch order puts them first)
    N = 64 * T - tail
    rng = np.random.default_rng(T + d)
    u = rng.standard_normal(d).astype(np.float32)
    u /= np.linalg.norm(u)
    x = {k: rng.standard_normal((1, 2, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["Q"] += 1.5 * u
    hot = [3, 4, T // 2, T - 1]
    for j in hot:
        x["K"][:, :, 64 * j:64 * (j + 1)] += 4.0 * u
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    x = {k: wl.round_to_bf16(v) for k, v in x.items()}
    Mc = oracle.build_mask(x["Q"], x["K"], 0.08, 0.2)
    cnt = (Mc == 1).sum(-2)
    assert (cnt[0, :, hot] >= T - 2).all() and (cnt >= 64).sum() >= 2 * len(hot)
    _full_case(oracle, x, "bf16", 0.08, 0.2)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,d,H,phi,bq,k_l", [(35, 64, 3, 0, 64, 0.2), (36, 64, 3, 1, 64, 0.2), (37, 128, 2, 0, 64, 0.2),
                                               (49, 64, 5, 0, 128, 0.2), (61, 128, 1, 0, 64, 0.95), (73, 64, 3, 1, 256, 0.1),
                                               (23, 64, 3, 0, 64, 0.2), (24, 128, 2, 1, 64, 0.2), (40, 64, 34, 0, 64, 0.2)])
def test_column_lists_cut_into_pieces(oracle, dtype, T, d, H, phi, bq, k_l):
    # a list longer than twelve is walked in pieces (from 24 blocks on, with floats from 36 and few entries in all), by
    # workgroups of their own and a second launch that adds the sums, or (34 heads) by one workgroup: lists of T,
    # T - 1, .. entries whose last piece is one entry, a full piece or between, key blocks without any, a ragged last
    # block, no marginal block; the same bits on every call
    N = 64 * T - 11
    rng = np.random.default_rng(T + d)
    u = rng.standard_normal(d).astype(np.float32)
    u /= np.linalg.norm(u)
    x = {k: rng.standard_normal((1, H, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["Q"] += 1.5 * u
    for j in (2, T // 2, T - 1):
        x["K"][:, :, 64 * j:64 * (j + 1)] += 4.0 * u
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    if dtype == "bf16":
        x = {k: wl.round_to_bf16(v) for k, v in x.items()}
    k_h = 4.2 / T
    Mc = oracle.build_mask(x["Q"], x["K"], k_h, k_l, bq=bq)
    assert (Mc == 1).sum(-2).max() * (bq // 64) >= T - 2
    _full_case(oracle, x, dtype, k_h, k_l, phi=phi, bq=bq)
    first, again = (run_gpu(x, dtype, k_h, k_l, phi=phi, bq=bq) for _ in range(2))
    assert all(np.array_equal(first[n], again[n]) for n in ("dQ", "dK", "dV", "dW"))


@pytest.mark.parametrize("T,d,k_h,phi,bq,k_l", [(23, 64, 0.1, 0, 64, 0.2), (24, 64, 0.1, 0, 64, 0.2), (25, 128, 0.05, 1, 64, 0.2),
                                                (48, 128, 0.1, 0, 128, 0.2), (66, 64, 0.25, 1, 64, 0.75), (146, 128, 0.05, 0, 64, 0.1),
                                                (200, 64, 0.02, 0, 256, 0.1), (256, 64, 0.04, 1, 64, 0.1)])
def test_gradients_of_a_head_among_few_and_many(T, d, k_h, phi, bq, k_l):
    # pieces of long lists are workgroups of their own among one or two heads and one workgroup's among forty; the
    # gradients of a head are the same bits in every call.  Lists of T, T - 1, .. entries and of lengths between
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    N, H = T * 64 - 5, 64
    u = torch.randn(d, generator=g, device="cuda")
    u /= u.norm()
    x = [torch.randn(1, H, N, d, generator=g, device="cuda") for _ in range(4)]
    # queries lean towards u more and more along the sequence, so the more key block j leans, the longer its list
    x[0] += 3.0 * torch.linspace(0, 1, N, device="cuda")[:, None] * u
    for j, c in ((2, 4.0), (T // 2, 1.0), (T // 3, 0.5), (T - 1, 2.0), (T // 4, 0.25)):
        x[1][:, :, 64 * j:64 * (j + 1)] += c * u
    x = [t.bfloat16() for t in x]
    W = (0.02 * torch.randn(d, d, generator=g, device="cuda")).bfloat16()

    def grads(H):
        Q, K, V, dO = (t[:, :H].contiguous() for t in x)
        p = sla.make_params(1, H, N, d, k_h, k_l, torch.bfloat16, phi=phi, bq=bq)
        Mc, luts, _ = sla.sla_build_mask(p, Q, K)
        ptr = sla.lut_views(p, luts)["col_ptr"][0, 0]
        O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
        need = sla.sla_sizes(p).ws_backward_bytes   # (the pieces' sums lie at its end)
        ws = torch.full((need + 65536,), 0x5a, dtype=torch.uint8, device="cuda")
        g = sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, workspace=ws[:need])[:3]
        assert bool((ws[need:] == 0x5a).all())
        return (ptr[1:] - ptr[:-1]).max().item(), g

    longest, many = grads(H)
    assert longest >= min(T // 2 + 2, T - 4)   # cut, if anything is
    for few in (1, 2, 7):
        for a, b in zip(grads(few)[1], many):
            assert torch.equal(a, b[:, :few])


def test_a_head_alone_above_the_longest_cut_lists():
    # from 257 blocks on nothing is cut: one head gives the bits that it gives among twenty
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    N, d = 257 * 64 - 5, 64
    x = [torch.randn(1, 20, N, d, generator=g, device="cuda").bfloat16() for _ in range(4)]
    x[1][:, :, 640:704] += 0.5   # a long list
    W = (0.02 * torch.randn(d, d, generator=g, device="cuda")).bfloat16()

    def grads(H):
        Q, K, V, dO = (t[:, :H].contiguous() for t in x)
        p = sla.make_params(1, H, N, d, 0.02, 0.1, torch.bfloat16)
        Mc, luts, _ = sla.sla_build_mask(p, Q, K)
        O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
        return sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO)[:3]

    for a, b in zip(grads(1), grads(20)):
        assert torch.equal(a[:, 0], b[:, 0])


@pytest.mark.parametrize("name", ["small_bf16", "small_bf16_d64", "small_fp32"])
def test_token_major_tensors(oracle, name):
    # [B,N,H,d] tensors: the same kernels walk the same values with another row pitch, so every
    # result equals the [B,H,N,d] call's bit for bit; one of the two is checked against the oracle
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(replace(w, B=2))
    a = run_gpu(x, w.dtype, w.k_h, w.k_l)
    b = run_gpu(x, w.dtype, w.k_h, w.k_l, token_major=True)
    for k in a:
        assert np.array_equal(a[k], b[k]), f"{k} differs between the two memory orders"
    Mc, s, f, g = _oracle_all(oracle, x, w.k_h, w.k_l, 0)
    assert np.array_equal(b["Mc"], Mc)
    for k in ("O", "dQ", "dK", "dV", "dW"):
        _compare(k, b[k], (f if k == "O" else g)[k], TOL[w.dtype])


@pytest.mark.parametrize("name", ["small_bf16", "small_fp32"])
def test_slices_of_a_fused_projection(oracle, name):
    # Q, K, V as views into one [B,N,3,H,d] tensor, dO / O and the gradients laid out the same way
    from paper_2509_24006_amd import binding as sla
    w = wl.WORKLOADS[name]
    x = wl.make_inputs(w)
    B, H, N, d = x["Q"].shape
    tdt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    dev = torch.device("cuda:0")
    qkv = torch.empty((B, N, 3, H, d), dtype=tdt, device=dev)
    gout = torch.empty((B, N, 3, H, d), dtype=tdt, device=dev)   # dO in slot 0
    for s_, k in enumerate(("Q", "K", "V")):
        qkv[:, :, s_] = torch.from_numpy(x[k]).to(dev).to(tdt).transpose(1, 2)
    gout[:, :, 0] = torch.from_numpy(x["dO"]).to(dev).to(tdt).transpose(1, 2)
    view = lambda t, s_: t[:, :, s_].permute(0, 2, 1, 3)          # [B,H,N,d], strides (3NHd, d, 3Hd, 1)
    Q, K, V, dO = view(qkv, 0), view(qkv, 1), view(qkv, 2), view(gout, 0)
    p = sla.make_params(B, H, N, d, w.k_h, w.k_l, tdt, layout=sla.SLA_STRIDED, strides=tuple(Q.stride()[:3]))
    W = torch.from_numpy(x["Proj"]).to(dev).to(tdt)
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)
    O, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts)
    dqkv = torch.zeros_like(qkv)
    out = (view(dqkv, 0), view(dqkv, 1), view(dqkv, 2), torch.empty((d, d), dtype=torch.float32, device=dev))
    sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, out=out)
    torch.cuda.synchronize()
    ref = run_gpu(x, w.dtype, w.k_h, w.k_l)
    f64 = lambda t: t.detach().double().cpu().numpy()
    assert np.array_equal(Mc.cpu().numpy(), ref["Mc"])
    for k, got in (("O", O), ("dQ", out[0]), ("dK", out[1]), ("dV", out[2]), ("dW", out[3])):
        assert np.array_equal(f64(got), ref[k]), f"{k} differs from the packed call"


@pytest.mark.parametrize("k_h", [1.0, 0.0])
@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 64), ("bf16", 128)])
def test_rows_far_apart_read_nothing_between_them(wide_tiles, dtype, d, k_h):
    # tokens 512 MB + 4 KB apart, NaN everywhere else: the offsets of the rows that the block does not
    # have pass 2^32 and come back into the range of the tensor, 32 KB and more behind a row of it.
    # Results equal the packed call's bit for bit (same arithmetic, another row pitch)
    from paper_2509_24006_amd import binding as sla
    tdt, esz = (torch.float32, 4) if dtype == "fp32" else (torch.bfloat16, 2)
    N, step = 3, ((1 << 29) + 4096) // esz
    rng = np.random.default_rng(d)
    x = {k: wl.round_to_bf16(rng.standard_normal((1, 1, N, d)).astype(np.float32)) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = wl.round_to_bf16((rng.standard_normal((d, d)) * 0.05).astype(np.float32))
    buf = torch.full(((N - 1) * step + 8 * d,), float("nan"), device="cuda", dtype=tdt)
    view = lambda i: buf.as_strided((1, 1, N, d), (step, step, step, 1), i * d)
    Q, K, V, dO, O, dQ, dK, dV = (view(i) for i in range(8))
    for t, k in ((Q, "Q"), (K, "K"), (V, "V"), (dO, "dO")):
        t.copy_(torch.from_numpy(x[k]))
    W = torch.from_numpy(x["Proj"]).cuda().to(tdt)
    dW = torch.empty((d, d), dtype=torch.float32, device="cuda")
    for bq in (64, 128):
        ref = run_gpu(x, dtype, k_h, 0.0, bq=bq)
        p = sla.make_params(1, 1, N, d, k_h, 0.0, tdt, bq=bq, layout=sla.SLA_STRIDED, strides=(step, step, step))
        Mc, luts, _ = sla.sla_build_mask(p, Q, K)
        _, saved = sla.sla_forward(p, Q, K, V, W, Mc, luts, O=O)
        sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, out=(dQ, dK, dV, dW))
        torch.cuda.synchronize()
        for k, got in (("O", O), ("dQ", dQ), ("dK", dK), ("dV", dV), ("dW", dW)):
            assert np.array_equal(got.double().cpu().numpy(), ref[k]), f"{k} differs from the packed call (bq = {bq})"


def test_classify_given_scores_with_ties(oracle):
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(0)
    T = 130
    p = sla.make_params(1, 3, T * 64, 64, 0.1, 0.2, torch.float32)
    s = rng.integers(-2, 3, size=(1, 3, T, T)).astype(np.float32)     # heavy ties
    s[0, 0, 0] = 0.0
    s[0, 0, 1, ::2] = -0.0
    s[0, 1] = rng.standard_normal((T, T)).astype(np.float32)
    nh, nl = oracle.counts(T, 0.1, 0.2)
    ref = oracle.classify(s, nh, nl)
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(Mc.cpu().numpy(), ref)
    v = {k: t.cpu().numpy() for k, t in sla.lut_views(p, luts).items()}
    check_luts(ref, v["row_idx"], v["col_ptr"], v["col_rows"], v["ind"], v["ind_t"], v["col_order"])


@pytest.mark.parametrize("T,bq", [(65, 64), (128, 64), (129, 64), (192, 128), (193, 192), (256, 64), (257, 64),
                                  (384, 128), (385, 64), (512, 64), (513, 192), (640, 256), (641, 256), (832, 64),
                                  (833, 128), (1024, 256), (1025, 256), (1216, 128), (1217, 256), (1408, 256),
                                  (1409, 256), (1728, 256), (1729, 256), (2048, 256), (2049, 256), (3072, 256)])
def test_classification_and_tables_at_the_edges_of_the_row_lengths(oracle, T, bq):
    # whole numbers, so the comparison is exact: one row of ties only, one of two values, one of
    # small integers, the rest distinct (where the threshold search ends early)
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(T)
    p = sla.make_params(1, 2, T * 64, 64, 0.04, 0.1, torch.bfloat16, bq=bq)
    z = sla.sla_sizes(p)
    s = rng.standard_normal((1, 2, z.Tq, z.T)).astype(np.float32)
    s[0, 0, 0] = 0.25
    s[0, 0, 1] = np.where(np.arange(z.T) % 3 == 0, 1.0, -1.0)
    s[0, 1, 0] = rng.integers(-4, 5, size=z.T)
    nh, nl = oracle.counts(z.T, 0.04, 0.1)
    ref = oracle.classify(s, nh, nl)
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(Mc.cpu().numpy(), ref)
    v = {k: t.cpu().numpy() for k, t in sla.lut_views(p, luts).items()}
    check_luts(per_tile(ref, bq // 64, z.T), v["row_idx"], v["col_ptr"], v["col_rows"], v["ind"], v["ind_t"],
               v["col_order"])


@pytest.mark.parametrize("T,bq,hot,k_h", [(65, 64, 23, 0.4), (130, 64, 24, 0.24), (130, 64, 22, 0.24), (130, 64, 10, 0.2),
                                          (130, 64, 0, 0.19), (200, 128, 12, 0.14), (193, 192, 30, 0.25), (130, 64, 0, 1.0)])
def test_column_lists_short_and_long_in_one_tile(oracle, T, bq, hot, k_h):
    # lists of up to 12 rows of a 64-row tile are written by a lane each, longer ones by the wave, all
    # 64 by the wave where 24 columns and more are long: `hot` columns that every row selects (22, 23,
    # 24 in a tile), the rest of a row's n_h at random (without hot ones: about 12 rows a list)
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(T + hot)
    p = sla.make_params(1, 2, T * 64, 64, k_h, 0.0, torch.bfloat16, bq=bq)
    z = sla.sla_sizes(p)
    s = rng.standard_normal((1, 2, z.Tq, z.T)).astype(np.float32)
    s[..., 3:3 + hot] += 8.0
    nh, nl = oracle.counts(z.T, k_h, 0.0)
    ref = oracle.classify(s, nh, nl)
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(Mc.cpu().numpy(), ref)
    v = {k: t.cpu().numpy() for k, t in sla.lut_views(p, luts).items()}
    check_luts(per_tile(ref, bq // 64, z.T), v["row_idx"], v["col_ptr"], v["col_rows"], v["ind"], v["ind_t"],
               v["col_order"])


@pytest.mark.parametrize("T,H,bq,hot,k_h", [(256, 3, 256, 23, 0.14), (257, 2, 256, 24, 0.24), (321, 2, 64, 22, 0.14),
                                            (577, 2, 256, 10, 1.0), (1025, 2, 256, 24, 0.1), (1100, 15, 256, 23, 0.05),
                                            (2496, 1, 256, 24, 0.03), (2497, 1, 256, 24, 0.03)])
def test_column_tables_by_four_eight_and_sixteen_waves(oracle, T, H, bq, hot, k_h):
    # up to four row tiles, more of them, more than sixteen with few heads (15 heads of 18 tiles: eight waves);
    # the last two: classification with 39 and 48 entries of a row per lane
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(T + hot)
    p = sla.make_params(1, H, T * 64, 64, k_h, 0.0, torch.bfloat16, bq=bq)
    z = sla.sla_sizes(p)
    s = rng.standard_normal((1, H, z.Tq, z.T)).astype(np.float32)
    s[..., 3:3 + hot] += 8.0
    ref = oracle.classify(s, *oracle.counts(z.T, k_h, 0.0))
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(Mc.cpu().numpy(), ref)
    v = {k: t.cpu().numpy() for k, t in sla.lut_views(p, luts).items()}
    check_luts(per_tile(ref, bq // 64, z.T), v["row_idx"], v["col_ptr"], v["col_rows"], v["ind"], v["ind_t"],
               v["col_order"])


@pytest.mark.parametrize("bq,N", [(128, 130 * 64), (192, 130 * 64 - 40), (256, 33 * 64)])
def test_classify_given_scores_with_ties_and_larger_query_blocks(oracle, bq, N):
    # rectangular score matrices (one row per block of bq queries), heavy ties; N is chosen so that
    # the last query block has fewer tiles than the others
    from paper_2509_24006_amd import binding as sla
    rng = np.random.default_rng(bq)
    p = sla.make_params(1, 3, N, 64, 0.1, 0.2, torch.float32, bq=bq)
    z = sla.sla_sizes(p)
    s = rng.integers(-2, 3, size=(1, 3, z.Tq, z.T)).astype(np.float32)
    s[0, 0, 0] = 0.0
    s[0, 0, 1, ::2] = -0.0
    s[0, 1] = rng.standard_normal((z.Tq, z.T)).astype(np.float32)
    nh, nl = oracle.counts(z.T, 0.1, 0.2)
    ref = oracle.classify(s, nh, nl)
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(Mc.cpu().numpy(), ref)
    v = {k: t.cpu().numpy() for k, t in sla.lut_views(p, luts).items()}
    check_luts(per_tile(ref, bq // 64, z.T), v["row_idx"], v["col_ptr"], v["col_rows"], v["ind"], v["ind_t"],
               v["col_order"])


@pytest.mark.parametrize("T,d,k_h,k_l,bq", [(18, 64, 0.1, 0.1, 64), (71, 64, 0.05, 0.45, 64), (300, 128, 0.05, 0.10, 64),
                                            (300, 128, 0.05, 0.85, 64), (41, 64, 0.1, 0.2, 128), (9, 128, 0.0, 0.0, 64),
                                            (33, 64, 0.5, 0.5, 64)])
def test_accumulation_line_by_every_method(oracle, T, d, k_h, k_l, bq):
    # Alg. 1's accumulation line alone, by the matrix-core product the library uses and by the three
    # forms the paper describes (one addition per block, pre-aggregation, Four Russians tables),
    # on random bf16 states and the mask of random scores: each against the oracle's plain sum.
    # Densities from every block marginal to none; a tile count that is no multiple of 4 or 64.
    from paper_2509_24006_amd import binding as sla
    B, H, N = 1, 2, T * 64 - 5
    rng = np.random.default_rng(T + d)
    p = sla.make_params(B, H, N, d, k_h, k_l, torch.bfloat16, bq=bq)
    z = sla.sla_sizes(p)
    assert z.T == T
    s = rng.standard_normal((B, H, z.Tq, T)).astype(np.float32)
    Mc, luts = sla.sla_classify_scores(p, torch.from_numpy(s).cuda())
    h = wl.round_to_bf16(rng.standard_normal((B, H, T, d * d + d)).astype(np.float32))
    ref = oracle.accumulate(h, per_tile(Mc.cpu().numpy(), bq // 64, T))
    hd = torch.from_numpy(h).cuda().to(torch.bfloat16)
    for method, name in ((sla.SLA_AGG_GEMM, "product"), (sla.SLA_AGG_ADD, "additions"),
                         (sla.SLA_AGG_PREAGG, "pre-aggregation"), (sla.SLA_AGG_FOUR_RUSSIANS, "four russians")):
        Hm, Zm = sla.sla_aggregate_states(p, method, luts, hd)
        torch.cuda.synchronize()
        print(f" {name}:", flush=True)
        _compare("H", Hm.double().cpu().numpy(), ref[..., :d * d], TOL["bf16"])
        # the vector part leaves in float; pre-aggregation subtracts two long float sums
        _compare("Z", Zm.double().cpu().numpy(), ref[..., d * d:], 1e-4 if method == sla.SLA_AGG_PREAGG else 1e-5)


@pytest.mark.parametrize("T", [64, 65, 96, 127, 128, 129, 256, 257, 385])
@pytest.mark.parametrize("d", [64, 128])
def test_state_sums_at_the_edges_of_the_row_tiles(T, d):
    # 32 or 64 output rows a wave, 64-column tiles in runs per XCD, several heads (the runs are rotated);
    # bound: the sums are float (T additions), the matrix part is rounded to bf16 once
    from paper_2509_24006_amd import binding as sla
    H = 3
    p = sla.make_params(1, H, T * 64, d, 0.1, 0.2, torch.bfloat16)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    sc = torch.randn(1, H, T, T, generator=g, device="cuda")
    h = torch.randn(1, H, T, d * d + d, generator=g, device="cuda").bfloat16()
    Mc, luts = sla.sla_classify_scores(p, sc)
    Hm, Zm = sla.sla_aggregate_states(p, sla.SLA_AGG_GEMM, luts, h)
    ref = torch.matmul((Mc == 0).double(), h.double())
    mag = torch.matmul((Mc == 0).double(), h.double().abs()) * T * 2.0 ** -24
    assert bool(((Hm.double() - ref[..., :d * d]).abs() <= ref[..., :d * d].abs() * 2.0 ** -8 + mag[..., :d * d]).all())
    assert bool(((Zm.double() - ref[..., d * d:]).abs() <= mag[..., d * d:]).all())


@pytest.mark.parametrize("T,H,bq", [(65, 140, 64), (97, 129, 64), (130, 100, 128)])
def test_scores_are_the_same_with_tiles_of_either_size(T, H, bq):
    # many heads in one call take tiles of 64 x 64 scores, a few of them tiles of 32 x 32: the same bits
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    Q, K = (torch.randn(1, H, T * 64 - 9, 64, generator=g, device="cuda").bfloat16() for _ in range(2))
    mk = lambda h: sla.make_params(1, h, T * 64 - 9, 64, 0.1, 0.1, torch.bfloat16, bq=bq)
    Mc, _, ws = sla.sla_build_mask(mk(H), Q, K)
    scores = sla.mask_ws_views(mk(H), ws)["scores"]
    for h in (0, H // 2, H - 1):
        m1, _, w1 = sla.sla_build_mask(mk(1), Q[:, h:h + 1].contiguous(), K[:, h:h + 1].contiguous())
        assert torch.equal(sla.mask_ws_views(mk(1), w1)["scores"][0, 0], scores[0, h])
        assert torch.equal(m1[0, 0], Mc[0, h])


@pytest.mark.parametrize("N,d,bq,dtype", [(1, 64, 64, torch.bfloat16), (1015, 64, 64, torch.bfloat16),
                                          (1728, 64, 128, torch.bfloat16), (800, 128, 64, torch.bfloat16),
                                          (833, 64, 256, torch.float32), (430, 128, 64, torch.float32)])
def test_short_masks_with_the_pooling_in_their_launch(N, d, bq, dtype):
    # 257 heads are pooled by a kernel of its own, one head by the mask kernel: the same bits
    from paper_2509_24006_amd import binding as sla
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    Q, K = (torch.randn(1, 257, N, d, generator=g, device="cuda").to(dtype) for _ in range(2))
    mk = lambda h: sla.make_params(1, h, N, d, 0.2, 0.2, dtype, bq=bq)
    Mc, luts, ws = sla.sla_build_mask(mk(257), Q, K)
    ref = {**sla.mask_ws_views(mk(257), ws), **sla.lut_views(mk(257), luts), "Mc": Mc}
    for h in (0, 100, 256):
        m1, l1, w1 = sla.sla_build_mask(mk(1), Q[:, h:h + 1], K[:, h:h + 1])
        for k, x in {**sla.mask_ws_views(mk(1), w1), **sla.lut_views(mk(1), l1), "Mc": m1}.items():
            assert torch.equal(x.flatten(0, 1)[0], ref[k].flatten(0, 1)[h]), k


def test_forward_without_saved_matches(oracle):
    from paper_2509_24006_amd import binding as sla
    from tests.gpu_util import to_dev, f64
    w = wl.WORKLOADS["small_bf16"]
    x = wl.make_inputs(w)
    p = sla.make_params(w.B, w.H, w.N, w.d, w.k_h, w.k_l, torch.bfloat16)
    Q, K, V, W = (to_dev(x[k], "bf16") for k in ("Q", "K", "V", "Proj"))
    Mc, luts, _ = sla.sla_build_mask(p, Q, K)
    O1, _ = sla.sla_forward(p, Q, K, V, W, Mc, luts)
    O2, sv = sla.sla_forward(p, Q, K, V, W, Mc, luts, need_saved=False)
    torch.cuda.synchronize()
    assert sv is None and torch.equal(O1, O2)


def test_calls_follow_the_given_stream(oracle):
    # every kernel of a call is enqueued on the stream handed in: the same results on a side
    # stream (default priority) as on the current one, with no host synchronisation in between
    from paper_2509_24006_amd import binding as sla
    w = wl.WORKLOADS["small_bf16"]
    x = wl.make_inputs(w)
    ref = run_gpu(x, "bf16", w.k_h, w.k_l)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = run_gpu(x, "bf16", w.k_h, w.k_l)
    torch.cuda.synchronize()
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


@pytest.mark.parametrize("seed", range(24))
def test_random_small_problems(oracle, seed):
    # a seeded draw over storage type, head size, batch, heads, (ragged) length, k_h, k_l, feature
    # map and memory order
    rng = np.random.default_rng(1000 + seed)
    dtype = str(rng.choice(["bf16", "fp32"], p=[0.7, 0.3]))
    d = int(rng.choice([64, 128])) if dtype == "bf16" else 64
    B, H = int(rng.integers(1, 3)), int(rng.integers(1, 4))
    N = int(rng.choice([rng.integers(1, 200), rng.integers(200, 1500), 64 * rng.integers(1, 20),
                        64 * rng.integers(1, 20) + 1]))
    k_h = float(rng.choice([0.0, 0.05, 0.1, 0.3, 0.5, 1.0]))
    k_l = float(rng.choice([0.0, 0.1, 0.3, 0.9]))
    phi, tm = int(rng.integers(0, 2)), bool(rng.integers(0, 2))
    x = {k: rng.standard_normal((B, H, N, d)).astype(np.float32) for k in ("Q", "K", "V", "dO")}
    x["Proj"] = (rng.standard_normal((d, d)) * 0.05).astype(np.float32)
    if dtype == "bf16":
        x = {k: wl.round_to_bf16(v) for k, v in x.items()}
    print(f"{dtype} d={d} B={B} H={H} N={N} k_h={k_h} k_l={k_l} phi={phi} token_major={tm}", flush=True)
    Mc, s, f, g = _oracle_all(oracle, x, k_h, k_l, phi)
    r = run_gpu(x, dtype, k_h, k_l, phi, token_major=tm)
    assert np.array_equal(r["scores"], s) and np.array_equal(r["Mc"], Mc)
    check_luts(r["Mc"], r["row_idx"], r["col_ptr"], r["col_rows"], r["ind"], r["ind_t"], r["col_order"])
    # sequences of a few blocks at most: a key block of one or a few keys makes most rows' dS
    # cancel exactly, see _compare; only the gradients of such draws get the floor
    short = N < 200
    # no critical block at all (bf16): dQ and dK are the linear branch's alone, an order of magnitude
    # smaller than with a sparse part, and dQ^phi = (dO^l H_i^T - D^l Z_i^T) / den is a difference of
    # nearly equal terms when few blocks are marginal; the H_i saved in bf16 bounds its error
    # relative to the terms (1.5e-2 of the result for one marginal block per row), so the error is
    # measured against a gradient of at least floor_rms per element there too
    lin_only = dtype == "bf16" and int((Mc == 1).sum()) == 0
    for k in ("O", "Os", "Ol", "dQ", "dK", "dV", "dW"):
        floor = 0.05 if (k in ("dQ", "dK", "dV", "dW") and short) or (k in ("dQ", "dK") and lin_only) else 0.0
        _compare(k, r[k], (f if k in f else g)[k], TOL[dtype], floor_rms=floor,
                 block_tol=None if (k == "dW" or short) else BLOCK_TOL[dtype])


def test_a_captured_step_replays_to_the_eager_results():
    # mask + forward + backward captured into one HIP graph (no allocation, no memset node, no host
    # synchronisation inside the calls); every replay, with eager calls and synchronisations in
    # between, gives what the eager calls gave
    from paper_2509_24006_amd import binding as sla
    w = wl.WORKLOADS["small_bf16"]
    x = wl.make_inputs(w)
    B, H, N, d = x["Q"].shape
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(a).to(dev).to(torch.bfloat16)
    Q, K, V, W, dO = t(x["Q"]), t(x["K"]), t(x["V"]), t(x["Proj"]), t(x["dO"])
    p = sla.make_params(B, H, N, d, w.k_h, w.k_l, torch.bfloat16)
    z = sla.sla_sizes(p)
    u8 = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=dev)
    Mc = torch.empty((B, H, z.T, z.T), dtype=torch.int8, device=dev)
    luts, ws_m, ws_f, ws_b, saved = (u8(n) for n in (z.luts_bytes, z.ws_mask_bytes, z.ws_forward_bytes,
                                                    z.ws_backward_bytes, z.saved_bytes))
    O = torch.empty_like(Q)
    out = (torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V),
           torch.empty((d, d), dtype=torch.float32, device=dev))

    def step():
        sla.sla_build_mask(p, Q, K, workspace=ws_m, Mc=Mc, luts=luts)
        sla.sla_forward(p, Q, K, V, W, Mc, luts, O=O, saved=saved, workspace=ws_f)
        sla.sla_backward(p, Q, K, V, W, Mc, luts, saved, dO, workspace=ws_b, out=out)

    results = lambda: [a.clone() for a in (Mc, O) + out]
    step()
    torch.cuda.synchronize()
    ref = results()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for rep in range(3):
        for a in (Mc, O) + out:
            a.zero_()
        luts.zero_()
        saved.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref, results()):
            assert torch.equal(a, b), f"replay {rep} differs from the eager result"
        step()   # eager work between the replays
        torch.cuda.synchronize()
