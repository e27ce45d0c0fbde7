"""linattn_verify_grouped (generation with the three-branch form) on the GPU against the CPU oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
from parity import STATE_TOL, TOL, check, dev, host
from paper_2406_07368_amd import binding, workloads

pytestmark = pytest.mark.gpu

IO = {"f32": torch.float32, "bf16": torch.bfloat16}
C = 64


def make_state(rng, B, H, d, Kc, io, fill):
    """A state as a prefix would leave it: non-negative S (sums of positive features times values of either sign
    are of either sign, but z is positive), history and an open group with `fill[b]` rows in use."""
    S = (rng.standard_normal((B, H, d, d)) * 3).astype(np.float32)
    z = (np.abs(rng.standard_normal((B, H, d))) * 5 + 1).astype(np.float32)
    hist = workloads.round_to_io(rng.standard_normal((B, H, Kc - 1, d)), io)
    kwin = workloads.round_to_io(rng.standard_normal((B, H, C, d)), io)
    vwin = workloads.round_to_io(rng.standard_normal((B, H, C, d)), io)
    return S, z, hist, kwin, vwin, np.asarray(fill, dtype=np.int32)


def to_gpu(state, io):
    dt = IO[io]
    S, z, hist, kwin, vwin, fill = state
    H = S.shape[1]
    return dev(S), dev(z), dev(hist, dt), dev(kwin, dt), dev(vwin, dt), torch.from_numpy(np.repeat(fill[:, None], H, axis=1)).cuda()


def compare_state(got, want, io, what, fill_in):
    """S, z to the bar; history and the rows in use of the open group bit for bit (rows at or beyond fill are not
    part of the state)."""
    check(host(got[0]), want[0], STATE_TOL, what + " S")
    check(host(got[1]), want[1], STATE_TOL, what + " z")
    assert np.array_equal(host(got[2]), workloads.round_to_io(want[2], io).astype(np.float64)), what + " hist"
    assert np.array_equal(got[5].cpu().numpy(), np.repeat(want[5][:, None], got[5].shape[1], axis=1)), what + " fill (per head)"
    for b, n in enumerate(want[5]):
        assert np.array_equal(host(got[3])[b, :, :n], want[3][b, :, :n]), what + f" kwin, batch row {b}"
        assert np.array_equal(host(got[4])[b, :, :n], want[4][b, :, :n]), what + f" vwin, batch row {b}"


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kk,Kc,fill", [(1, 3, (0, 17)), (1, 1, (63, 62)), (2, 3, (62, 10)), (3, 2, (63, 40)), (4, 3, (30, 61)), (5, 5, (59, 60)), (8, 2, (0, 63)),
                                        (13, 8, (50, 55)), (16, 3, (47, 48)), (16, 4, (63, 5)), (6, 1, (20, 63))])
def test_verify_grouped_matches_oracle(io, d, kk, Kc, fill):
    """Groups that stay open, groups that are completed by the kept drafts, drafts beyond the end of the group.
    bf16 with four or more drafts runs on the matrix cores, everything else on the vector ALUs."""
    B, H = 2, 3
    rng = np.random.default_rng(6000 + kk + d + Kc)
    state = make_state(rng, B, H, d, Kc, io, fill)
    q, k, v = (workloads.round_to_io(rng.standard_normal((B, H, kk, d)), io) for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    n_commit = np.array([kk, kk // 2], dtype=np.int32)
    want = oracle.verify_grouped(q, k, v, w, C, *state, n_commit=n_commit, alpha=0.8, eps=1e-3)
    gs = to_gpu(state, io)
    dt = IO[io]
    out = binding.verify_grouped(dev(q, dt), dev(k, dt), dev(v, dt), dev(w), gs, 0.8, torch.from_numpy(n_commit).cuda(), 1e-3)
    torch.cuda.synchronize()
    check(host(out), want[0], TOL[io], "out")
    compare_state(gs, want[1:], io, f"kk={kk} fill={fill}", fill)


def test_nothing_kept_leaves_everything_untouched():
    B, H, d, Kc, kk = 3, 2, 128, 3, 6
    rng = np.random.default_rng(6100)
    state = make_state(rng, B, H, d, Kc, "bf16", (5, 60, 63))
    q, k, v = (workloads.round_to_io(rng.standard_normal((B, H, kk, d)), "bf16") for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    gs = to_gpu(state, "bf16")
    before = [t.clone() for t in gs]
    bf = torch.bfloat16
    out = binding.verify_grouped(dev(q, bf), dev(k, bf), dev(v, bf), dev(w), gs, 1.0, torch.zeros(B, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    want = oracle.verify_grouped(q, k, v, w, C, *state, n_commit=np.zeros(B, dtype=np.int32))
    check(host(out), want[0], TOL["bf16"], "out")
    for a, b in zip(gs, before):
        assert torch.equal(a, b)


@pytest.mark.parametrize("io,d,block", [("bf16", 128, 1), ("bf16", 64, 7), ("f32", 64, 16), ("bf16", 128, 16)])
def test_generation_reproduces_the_grouped_prefill(io, d, block):
    """A sequence fed through verify_grouped from an empty state, block by block with everything kept, against the
    whole-sequence oracle; then the same after a GPU prefill of the first 128 tokens."""
    B, H, Kc, L = 2, 2, 3, 200
    rng = np.random.default_rng(6200 + d + block)
    q, k, v = (workloads.round_to_io(rng.standard_normal((B, H, L, d)), io) for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    want = oracle.prefill_grouped(q, k, v, w, C, alpha=1.0, eps=1e-3)
    dt = IO[io]
    gq, gk, gv, gw = dev(q, dt), dev(k, dt), dev(v, dt), dev(w)
    starts = [(0, binding.grouped_state(B, H, d, Kc, dt))]
    if io == "bf16":
        _, st = binding.prefill_grouped(gq[:, :, :128].contiguous(), gk[:, :, :128].contiguous(), gv[:, :, :128].contiguous(), gw, 1.0, None, 1e-3)
        starts.append((128, binding.grouped_state(B, H, d, Kc, dt, prefill_state=st)))
    for t_start, gs in starts:
        outs = []
        for t0 in range(t_start, L, block):
            sl = slice(t0, min(t0 + block, L))
            outs.append(binding.verify_grouped(gq[:, :, sl].contiguous(), gk[:, :, sl].contiguous(), gv[:, :, sl].contiguous(), gw, gs, 1.0, None, 1e-3))
        torch.cuda.synchronize()
        check(host(torch.cat(outs, dim=2)), want[0][:, :, t_start:], TOL[io], f"outputs from token {t_start}")
        assert gs[5].cpu().tolist() == [[L % C] * H] * B
        # completed groups + the open group's rows = the running sum of the whole sequence
        S_open = np.einsum("bhti,bhtc->bhic", oracle.phi(host(gs[3])[:, :, :L % C]), host(gs[4])[:, :, :L % C])
        check(host(gs[0]) + S_open, want[1], TOL[io], "S")


def test_whole_model_shape_one_token():
    """B32 H32 d128, one token per head (the decode step the bench times), open groups of different lengths."""
    B, H, d, Kc = 32, 32, 128, 3
    rng = np.random.default_rng(6300)
    fill = (np.arange(B) * 5) % C
    state = make_state(rng, B, H, d, Kc, "bf16", fill)
    q, k, v = (workloads.round_to_io(rng.standard_normal((B, H, 1, d)), "bf16") for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    bf = torch.bfloat16
    gs = to_gpu(state, "bf16")
    out = binding.verify_grouped(dev(q, bf), dev(k, bf), dev(v, bf), dev(w), gs, 1.0)
    torch.cuda.synchronize()
    rows = [0, 7, 13, 31]                                          # fill 0, 35, 1 (65 % 64), 27; row 13 of 5*13 = 65 -> 1
    sub = tuple(a[rows] for a in state)
    want = oracle.verify_grouped(q[rows], k[rows], v[rows], w, C, *sub)
    check(host(out)[rows], want[0], TOL["bf16"], "out")
    check(host(gs[0])[rows], want[1], STATE_TOL, "S")
    assert gs[5].cpu().numpy()[rows, 0].tolist() == want[6].tolist()


@pytest.mark.parametrize("d,kk", [(64, 1), (128, 1), (128, 2), (128, 3)])
@pytest.mark.parametrize("phi", ["elu1", "relu"])
def test_completion_against_64_bits_and_with_rows_that_are_not_finite(d, kk, phi):
    """A group of bf16 rows fills up: S and z to the rounding of fp32 sums (64 products per element, exact; bound: 64 roundings of 2^-24
    of the largest partial sum, measured below 1e-7 in the 2-norm).  Infinities and NaN in keys and values reach exactly the
    elements that the sums themselves give them."""
    B, H, Kc = 3, 2, 3
    torch.manual_seed(d + kk)
    w = torch.randn(H, d, Kc, device="cuda")
    q, k, v = (torch.randn(B, H, kk, d, device="cuda").to(torch.bfloat16) for _ in range(3))
    for bad in (False, True):
        st = binding.grouped_state(B, H, d, Kc)
        st[0].normal_(std=30.0)
        st[1].uniform_(50.0, 90.0)
        st[3].normal_()
        st[4].normal_()
        st[5].fill_(64 - kk)
        if bad:
            st[4][0, 0, 7, 3] = float("inf")
            st[4][0, 1, 60, d - 1] = float("nan")
            st[4][1, 0, 0, 0] = float("-inf")
            st[3][1, 1, 9, 5] = float("inf")
            st[3][2, 0, 11, 33] = float("nan")
            st[3][2, 1, 12, 40] = float("-inf")
        rk = torch.cat([st[3][:, :, :64 - kk], k], 2).double()
        rv = torch.cat([st[4][:, :, :64 - kk], v], 2).double()
        f = rk.clamp(min=0) if phi == "relu" else torch.where(rk > 0, rk + 1, rk.exp())
        if phi == "relu":
            f = torch.where(rk.isnan(), torch.zeros_like(f), f)     # the map max(x, 0) takes a NaN to 0
        S = st[0].double() + (f[..., :, None] * rv[..., None, :]).sum(2)
        z = st[1].double() + f.sum(2)
        binding.verify_grouped(q, k, v, w, st, eps=1e-3, phi=phi)
        torch.cuda.synchronize()
        for got, want in ((st[0], S), (st[1], z)):
            assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
            ok = want.isfinite()
            err = (got.double() - want)[ok].norm() / want[ok].norm()
            assert err < 2e-7, float(err)
        assert int(st[5].sum()) == 0


@pytest.mark.parametrize("d,kk", [(64, 1), (128, 2)])
@pytest.mark.parametrize("low,high", [(-87.0, -84.0), (-78.0, -69.0), (-104.0, -88.0), (-70.0, -60.0)])
def test_completion_with_features_near_the_end_of_the_range(d, kk, low, high):
    """Keys whose exponentials are 1e-26 to 1e-46: what S gets of a group of them is off by what the exponential's argument is rounded to
    (|k| roundings of 2^-24), the products' sums (64) and features below the smallest normal number, not by the bf16 terms they are
    multiplied as."""
    B, H, Kc = 2, 3, 3
    torch.manual_seed(d + kk)
    w = torch.randn(H, d, Kc, device="cuda")
    q, v = (torch.randn(B, H, kk, d, device="cuda").to(torch.bfloat16) for _ in range(2))
    st = binding.grouped_state(B, H, d, Kc)
    keys = (torch.rand(B, H, 64, d, device="cuda") * (high - low) + low).to(torch.bfloat16)
    k = keys[:, :, 64 - kk:].contiguous()
    st[3].copy_(keys)
    st[4].normal_()
    st[5].fill_(64 - kk)
    rv = torch.cat([st[4][:, :, :64 - kk], v], 2).double()
    f = keys.double().exp()
    S = (f[..., :, None] * rv[..., None, :]).sum(2)
    most = (f[..., :, None] * rv.abs()[..., None, :]).sum(2)        # of the same sums without cancellation
    binding.verify_grouped(q, k, v, w, st, eps=1e-3)
    torch.cuda.synchronize()
    err = (st[0].double() - S).abs()
    lost = (torch.where(f < 1.01 * 2.0 ** -126, f, 0.0)[..., :, None] * rv.abs()[..., None, :]).sum(2)
    assert (err <= (-low + 64) * 2.0 ** -24 * most + lost + 64 * 2.0 ** -148).all(), float((err / most.clamp(min=1e-300)).max())
