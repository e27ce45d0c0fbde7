"""The sizes of the paper's FLASH experiment on the GPU against the CPU oracle, through the C ABI: a masked
depthwise convolution of up to 63 taps (Sec. 4.1) in both prefill forms, and the three-branch form in groups of
256 tokens (Sec. 5 "Settings")."""
import numpy as np
import pytest
import torch

import oracle
from parity import TOL, check, check_unfloored, dev, host
from paper_2406_07368_amd import binding, workloads
from test_gpu_prefill import IO, same_pattern, small_case

pytestmark = pytest.mark.gpu


def run(q, k, v, w, state, io, chunk=64, eps=0.0, alpha=None, alias_hist=False):
    dt = IO[io]
    st = None if state is None else (dev(state[0]), dev(state[1]), dev(state[2], dt))
    if alias_hist:
        # the caller's history buffer is updated in place: hist_out is hist_in
        B, H, L, d = q.shape
        Kc = w.shape[2]
        gq, gk, gv = dev(q, dt), dev(k, dt), dev(v, dt)
        desc = binding.make_desc(B, H, d, Kc, chunk, dt, eps, L=L)
        out = torch.empty_like(gq)
        nb = binding.linattn_workspace_bytes(desc, L)
        ws = torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")
        binding.linattn_prefill(desc, L, gq, gk, gv, dev(w), st[0], st[1], st[2], out, st[0], st[1], st[2], ws, nb)
        S, z, h = st
    else:
        out, (S, z, h) = binding.prefill(dev(q, dt), dev(k, dt), dev(v, dt), dev(w), st, chunk, eps, grouped_alpha=alpha)
    torch.cuda.synchronize()
    return host(out), host(S), host(z), host(h)


def compare(got, want, io, what):
    e = check(got[0], want[0], TOL[io], what + " out")
    check(got[1], want[1], TOL[io], what + " S")
    check(got[2], want[2], TOL[io], what + " z")
    assert np.array_equal(got[3], want[3]), what + " hist"
    return e


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,Kc,with_state", [(1, 63, True), (40, 9, False), (62, 63, True), (63, 63, False), (64, 33, True),
                                             (130, 63, True), (300, 63, False), (300, 17, True)])
def test_long_conv_kernels_in_the_token_level_prefill(io, d, L, Kc, with_state):
    """More taps than the attention kernels gather themselves: sequences shorter and longer than the window, with
    and without a history of Kc - 1 rows."""
    q, k, v, w, state = small_case(7000 + L + d + Kc, 2, 3, L, d, Kc, io, with_state)
    args = () if state is None else state
    want = oracle.prefill_recurrent(q, k, v, w, *args, eps=1e-3)
    compare(run(q, k, v, w, state, io, 256, 1e-3), want, io, f"L={L} Kc={Kc}")


@pytest.mark.parametrize("L", [20, 200])
def test_long_conv_history_updated_in_place(L):
    """hist_out may be hist_in, also when the new history is part old rows, part new ones (L < Kc - 1)."""
    io, d, Kc = "bf16", 128, 63
    q, k, v, w, state = small_case(7100 + L, 2, 2, L, d, Kc, io, True)
    want = oracle.prefill_recurrent(q, k, v, w, *state)
    compare(run(q, k, v, w, state, io, alias_hist=True), want, io, f"in place, L={L}")


def test_long_conv_on_a_segmented_sequence_and_in_token_major_layout():
    """Few heads, long sequence (the attention kernel cuts the sequence into segments) with 63 taps; and the same
    call on [B,L,H,d] tensors."""
    B, H, L, d, Kc = 1, 2, 2100, 128, 63
    q, k, v, w, state = small_case(7200, B, H, L, d, Kc, "bf16", True)
    want = oracle.prefill_recurrent(q, k, v, w, *state)
    compare(run(q, k, v, w, state, "bf16", 256), want, "bf16", "segmented")
    dt = torch.bfloat16
    tq, tk, tv = (dev(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), dt).transpose(1, 2) for a in (q, k, v))
    st = (dev(state[0]), dev(state[1]), dev(state[2], dt))
    out, (S, z, h) = binding.prefill(tq, tk, tv, dev(w), st, 256)
    torch.cuda.synchronize()
    assert out.stride() == tq.stride()
    compare((host(out), host(S), host(z), host(h)), want, "bf16", "token-major")


def test_long_conv_leaks_nothing_from_later_tokens():
    io, d, Kc, L = "bf16", 128, 63, 200
    q, k, v, w, _ = small_case(7300, 1, 2, L, d, Kc, io, False)
    base = run(q, k, v, w, None, io)[0]
    rng = np.random.default_rng(7301)
    for t in (0, 61, 62, 63, 130):
        q2, k2, v2 = q.copy(), k.copy(), v.copy()
        for a in (q2, k2, v2):
            a[:, :, t + 1:] = workloads.round_to_io(a[:, :, t + 1:] + 4.0 * rng.standard_normal(a[:, :, t + 1:].shape), io)
        got = run(q2, k2, v2, w, None, io)[0]
        assert np.array_equal(got[:, :, :t + 1], base[:, :, :t + 1]), f"leak into tokens <= {t}"


@pytest.mark.parametrize("io,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("L,Kc,with_state", [(1, 3, False), (255, 63, True), (256, 5, False), (257, 63, True), (600, 63, False)])
def test_three_branch_form_in_groups_of_256(io, d, L, Kc, with_state):
    q, k, v, w, state = small_case(7400 + L + d + Kc, 2, 2, L, d, Kc, io, with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 256, alpha=0.7, eps=1e-3, **args)
    compare(run(q, k, v, w, state, io, 256, 1e-3, alpha=0.7), want, io, f"groups of 256, L={L} Kc={Kc}")


@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [(10, 10, 1100, 128, 5, True),     # 100 heads: two segments of 3 and 2 groups
                                                    (8, 32, 600, 128, 3, True),      # 256 heads: no segments, 3 groups each
                                                    (8, 32, 300, 64, 8, False),
                                                    (1, 3, 2100, 64, 2, True)])      # 9 segments of one group
def test_three_branch_form_in_groups_of_256_launch_plans(B, H, L, d, Kc, with_state):
    """bf16 rows on the matrix cores: every way the sequence can be laid out on the chip (segments of several groups,
    of one group, none at all), with the state handed back after the last token."""
    q, k, v, w, state = small_case(7450 + B + L, B, H, L, d, Kc, "bf16", with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 256, alpha=1.0, eps=1e-3, **args)
    compare(run(q, k, v, w, state, "bf16", 256, 1e-3, alpha=1.0), want, "bf16", f"B{B} H{H} L{L} d{d}")


@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [(1, 1, 257, 64, 9, False), (1, 1, 257, 128, 17, True), (1, 3, 511, 64, 18, True),
                                                   (2, 2, 513, 128, 49, True), (1, 4, 1000, 128, 50, False), (2, 5, 800, 64, 63, True),
                                                   (6, 8, 1030, 128, 63, True), (1, 4, 2100, 128, 40, True)])
@pytest.mark.parametrize("in_place", [False, True])
def test_long_conv_in_the_launch_of_the_prefix_sum(B, H, L, d, Kc, with_state, in_place):
    """Groups of 256, several segments, a conv of one tile a workgroup: it runs beside the prefix sum (every number of contraction
    steps, ragged last tiles, a history or none); with the history updated in place, and with two tiles a workgroup (48 heads of
    1030 tokens), in a launch of its own.  Out is one rounding of the sum in either, and the two agree to the bit."""
    if in_place and not with_state:
        pytest.skip("no history to update")
    q, k, v, w, state = small_case(7470 + L + Kc, B, H, L, d, Kc, "bf16", with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 256, alpha=1.0, eps=1e-3, **args)
    got = run(q, k, v, w, state, "bf16", 256, 1e-3, alpha=1.0)
    compare(got, want, "bf16", f"B{B} H{H} L{L} d{d} Kc{Kc}")
    if in_place:
        dt = torch.bfloat16
        S, z, h = dev(state[0]), dev(state[1]), dev(state[2], dt)
        desc = binding.make_desc(B, H, d, Kc, 256, dt, 1e-3, L=L)
        nb = binding.linattn_workspace_bytes(desc, L)
        ws = torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")
        out = torch.empty(B, H, L, d, dtype=dt, device="cuda")
        binding.linattn_prefill_grouped(desc, L, 1.0, dev(q, dt), dev(k, dt), dev(v, dt), dev(w), S, z, h, out, S, z, h, ws, nb)
        torch.cuda.synchronize()
        for a, b in zip(got, (out, S, z, h)):
            assert np.array_equal(a, host(b))


@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [(1, 1, 1, 128, 3, True), (1, 2, 31, 64, 63, False), (1, 2, 33, 128, 1, True),
                                                   (1, 3, 65, 64, 8, True), (1, 5, 255, 128, 63, True), (1, 4, 256, 64, 4, True),
                                                   (1, 3, 545, 128, 5, False), (1, 8, 1000, 64, 3, True), (1, 8, 1000, 128, 63, True),
                                                   (2, 12, 600, 64, 63, True), (4, 8, 700, 128, 7, True), (1, 8, 4090, 64, 2, True),
                                                   (16, 8, 130, 128, 3, True), (16, 8, 129, 64, 63, True)])
@pytest.mark.parametrize("phi", ["elu1", "relu"])
def test_groups_of_256_shared_by_workgroups(B, H, L, d, Kc, with_state, phi):
    """Few groups: 8, 4 or 2 workgroups share one (queries), and the state after the last token is another's work.  Against the
    oracle, token-major rows to the bit, and -- sequences of one group, whose state and history updated in place keep one
    workgroup per group -- against the other kernel: S, z and the history to the bit, the outputs to two roundings."""
    io, dt = "bf16", torch.bfloat16
    q, k, v, w, state = small_case(7480 + L + Kc, B, H, L, d, Kc, io, with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    with oracle.feature_map(phi):
        want = oracle.prefill_grouped(q, k, v, w, 256, alpha=0.7, eps=0.05, **args)
    st = None if state is None else (dev(state[0]), dev(state[1]), dev(state[2], dt))
    out, new = binding.prefill(dev(q, dt), dev(k, dt), dev(v, dt), dev(w), st, 256, 0.05, phi=phi, grouped_alpha=0.7)
    torch.cuda.synchronize()
    got = [host(x) for x in (out, *new)]
    compare(got, want, io, f"B{B} H{H} L{L} d{d} Kc{Kc} {phi}")
    tq, tk, tv = (dev(np.ascontiguousarray(x.transpose(0, 2, 1, 3)), dt).transpose(1, 2) for x in (q, k, v))
    out2, new2 = binding.prefill(tq, tk, tv, dev(w), st, 256, 0.05, phi=phi, grouped_alpha=0.7)
    torch.cuda.synchronize()
    for x, y in zip(got, (out2, *new2)):
        assert np.array_equal(x, host(y))
    if with_state and L <= 256 and phi == "elu1":
        S, z, h = (x.clone() for x in st)
        desc = binding.make_desc(B, H, d, Kc, 256, dt, 0.05, L=L)
        nb = binding.linattn_workspace_bytes(desc, L)
        ws = torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")
        o = torch.empty(B, H, L, d, dtype=dt, device="cuda")
        binding.linattn_prefill_grouped(desc, L, 0.7, dev(q, dt), dev(k, dt), dev(v, dt), dev(w), S, z, h, o, S, z, h, ws, nb)
        torch.cuda.synchronize()
        for x, y in zip(got[1:], (S, z, h)):
            assert np.array_equal(x, host(y))
        err = np.abs(got[0] - host(o))
        # one rounding of the output either way, the weights' rounding (2 ** -9 of a value) taken at another tile's maximum
        assert (err <= 2.0 ** -7 * (np.abs(host(o)) + np.abs(v).max())).all()


@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [(1, 1, 257, 128, 3, True), (1, 3, 513, 64, 63, False), (1, 8, 1000, 128, 63, True),
                                                   (4, 8, 768, 64, 4, True), (1, 22, 1030, 128, 63, True), (1, 2, 8200, 128, 5, True)])
def test_parts_of_a_segment_in_the_first_pass(B, H, L, d, Kc, with_state):
    """Groups of 256, few segments: 4 or 2 workgroups share one in the first pass, with slots of their own behind the rest of the
    workspace.  A workspace without room for these is enough, with whole segments; and nothing is written behind either."""
    dt = torch.bfloat16
    q, k, v, w, state = small_case(7492 + L + Kc, B, H, L, d, Kc, "bf16", with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 256, alpha=0.7, eps=1e-3, **args)
    desc = binding.make_desc(B, H, d, Kc, 256, dt, 1e-3, L=L)
    full = binding.linattn_workspace_bytes(desc, L)
    whole = B * H * (-(-L // 256) * (d * d + d) * 4 + 8 * d * 2)
    assert full > whole
    st = (None, None, None) if state is None else (dev(state[0]), dev(state[1]), dev(state[2], dt))
    got = []
    for nb in (full, whole):
        ws = torch.full((nb + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        out = torch.empty(B, H, L, d, dtype=dt, device="cuda")
        S, z = torch.empty(B, H, d, d, device="cuda"), torch.empty(B, H, d, device="cuda")
        h = torch.empty(B, H, Kc - 1, d, dtype=dt, device="cuda")
        binding.linattn_prefill_grouped(desc, L, 0.7, dev(q, dt), dev(k, dt), dev(v, dt), dev(w), *st, out, S, z, h, ws, nb)
        torch.cuda.synchronize()
        assert (ws[nb:] == 0xA5).all()
        got.append([host(x) for x in (out, S, z, h)])
        compare(got[-1], want, "bf16", f"B{B} H{H} L{L} d{d} Kc{Kc} workspace {nb}")
    for x, y in zip(got[0][1:], got[1][1:]):               # fp32 sums over L tokens in another order
        assert np.abs(x - y).max(initial=0) <= L * 2.0 ** -24 * np.abs(y).max(initial=0)
    with pytest.raises(binding.LinattnError):
        binding.linattn_prefill_grouped(desc, L, 0.7, dev(q, dt), dev(k, dt), dev(v, dt), dev(w), *st, out, S, z, h, ws, whole - 1)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [1, 40, 64, 100])        # workgroups per group: 8, 8, 8, 4; of 300 tokens 8, 4, 2, 1
@pytest.mark.parametrize("L", [64, 300])
def test_key_tiles_whose_logits_are_all_minus_infinity(d, heads, L):
    """Keys of -inf against positive queries have no weight.  A wave that meets nothing but such a tile hands on zeros: against
    160 or more heads, whose groups have one workgroup each and whose waves see the first tile before."""
    dt = torch.bfloat16
    g = torch.Generator().manual_seed(7491 + d)
    q, k, v = (torch.randn((1, 1, L, d), generator=g) * d ** -0.5 for _ in range(3))
    k[:, :, 32:64] = -float("inf")
    w = torch.randn((1, d, 3), generator=g) * 0.3
    def call(B):
        a = [x.expand(B, 1, L, d).contiguous().to(dt).cuda() for x in (q.abs() + 0.01, k, v)]
        out, (S, z, h) = binding.prefill_grouped(*a, w.cuda(), group=256)
        torch.cuda.synchronize()
        return [host(x)[:1] for x in (out, S, z, h)]
    got, want = call(heads), call(320)
    assert all(np.isfinite(x).all() for x in got)
    for x, y in zip(got[1:], want[1:]):
        # fp32 sums over L tokens, in the same order where there is one group
        assert np.array_equal(x, y) if L <= 256 else np.abs(x - y).max() <= L * 2.0 ** -24 * np.abs(y).max()
    # one rounding of the output either way, the weights' rounding (2 ** -9 of a value) taken at another tile's maximum
    assert (np.abs(got[0] - want[0]) <= 2.0 ** -7 * (np.abs(want[0]) + v.abs().max().item())).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [1, 40, 100])            # workgroups per group of 300 tokens: 8, 4, 1 (of 64 heads 2)
@pytest.mark.parametrize("Kc", [1, 2, 3, 4, 5, 6, 7, 8])
def test_values_that_are_not_finite_reach_the_same_outputs_with_a_group_shared(d, heads, Kc):
    """An infinity or a NaN in the values, inside a group, at its end (the next group's first taps see it) and in its last rows:
    infinities and NaN come out where the kernel of one workgroup per group has them, whose conv takes no row beyond its taps but for
    those of a tap count it was not built for."""
    dt, L = torch.bfloat16, 300
    g = torch.Generator().manual_seed(7493 + d + Kc)
    q, k, v = (torch.randn((3, 1, L, d), generator=g) * (d ** -0.5 if i < 2 else 1.0) for i in range(3))
    v[0, :, 17, 3] = v[1, :, 254, d - 1] = v[2, :, 290, 8] = float("inf")
    v[0, :, 200, 40], v[2, :, 100, 9] = float("nan"), -float("inf")
    w = torch.randn((1, d, Kc), generator=g).abs() * 0.3 + 0.1
    def call(B, one):
        a = [x[one:one + 1].expand(B, 1, L, d).contiguous().to(dt).cuda() for x in (q, k, v)]
        out, _ = binding.prefill_grouped(*a, w.cuda(), group=256)
        torch.cuda.synchronize()
        return host(out)[:1]
    for one in range(3):
        got, want = call(heads, one), call(320, one)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))


def test_three_branch_form_in_groups_of_256_details():
    """Nothing before the first group and eps = 0 (the linear branch is absent there, no division by zero reaches
    the output); the other feature map; token-major tensors; peaked softmax weights; no leak from later tokens."""
    io, dt, d = "bf16", torch.bfloat16, 128
    q, k, v, w, _ = small_case(7460, 1, 4, 700, d, 3, io, False)
    want = oracle.prefill_grouped(q, k, v, w, 256, alpha=1.0, eps=0.0)
    base = run(q, k, v, w, None, io, 256, 0.0, alpha=1.0)
    compare(base, want, io, "eps = 0")
    with oracle.feature_map("relu"):
        want = oracle.prefill_grouped(q, k, v, w, 256, alpha=0.5, eps=0.05)
    out, (S, z, h) = binding.prefill(dev(q, dt), dev(k, dt), dev(v, dt), dev(w), None, 256, 0.05, phi="relu", grouped_alpha=0.5)
    torch.cuda.synchronize()
    compare((host(out), host(S), host(z), host(h)), want, io, "relu")
    tq, tk, tv = (dev(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), dt).transpose(1, 2) for a in (q, k, v))
    out, (S, z, h) = binding.prefill(tq, tk, tv, dev(w), None, 256, 0.0, grouped_alpha=1.0)
    torch.cuda.synchronize()
    assert np.array_equal(host(out), base[0]), "token-major layout"
    q3, k3, v3, w3, _ = small_case(7461, 2, 2, 500, d, 3, io, False, scale=2.5)        # logits in the tens
    want = oracle.prefill_grouped(q3, k3, v3, w3, 256, alpha=0.0)
    compare(run(q3, k3, v3, w3, None, io, 256, alpha=0.0), want, io, "peaked weights")
    rng = np.random.default_rng(7462)
    for t in (0, 100, 255, 256, 600):
        q2, k2, v2 = q.copy(), k.copy(), v.copy()
        for a in (q2, k2, v2):
            a[:, :, t + 1:] = workloads.round_to_io(a[:, :, t + 1:] + 4.0 * rng.standard_normal(a[:, :, t + 1:].shape), io)
        got = run(q2, k2, v2, w, None, io, 256, 0.0, alpha=1.0)[0]
        assert np.array_equal(got[:, :, :t + 1], base[0][:, :, :t + 1]), f"leak into tokens <= {t}"


@pytest.mark.parametrize("d", [64, 128])
def test_three_branch_form_in_groups_of_64_with_63_taps(d):
    """The matrix-core kernel of the three-branch form followed by the long convolution."""
    q, k, v, w, state = small_case(7500 + d, 2, 3, 333, d, 63, "bf16", True)
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=1.0, eps=1e-3, S0=state[0], z0=state[1], hist0=state[2])
    compare(run(q, k, v, w, state, "bf16", 64, 1e-3, alpha=1.0), want, "bf16", f"groups of 64, 63 taps, d={d}")


def test_fp32_rows_of_128_in_groups_of_256_are_refused():
    q, k, v, w, _ = small_case(7600, 1, 1, 10, 128, 3, "f32", False)
    with pytest.raises(binding.LinattnError) as ei:
        run(q, k, v, w, None, "f32", 256, alpha=1.0)
    assert ei.value.status == 5


@pytest.mark.parametrize("name", ["flash_L1024", "flash_L4096", "flash_L8192"])
def test_flash_shaped_workload_every_head(name):
    """B1 H8 d128 bf16, groups of 256, 63 taps, at full length: the token-level form (which does not depend on
    the group size) and the three-branch form in groups of 256, all heads against the oracle."""
    wl = workloads.CONFIGS[name]
    q, k, v, w = workloads.prefill_tensors(wl)
    gq, gk, gv, gw = q.cuda(), k.cuda(), v.cuda(), w.cuda()
    out, (S, z, h) = binding.prefill(gq, gk, gv, gw, None, wl.chunk)
    gout, (gS, gz, gh) = binding.prefill_grouped(gq, gk, gv, gw, 1.0, group=wl.chunk)
    torch.cuda.synchronize()
    hq, hk, hv = host(q), host(k), host(v)
    want = oracle.prefill_recurrent(hq, hk, hv, w.numpy())
    e1 = compare((host(out), host(S), host(z), host(h)), want, "bf16", name)
    p1 = check_unfloored(host(out), want[0], TOL["bf16"], name + " out")
    gwant = oracle.prefill_grouped(hq, hk, hv, w.numpy(), wl.chunk, alpha=1.0)
    e2 = compare((host(gout), host(gS), host(gz), host(gh)), gwant, "bf16", name + " three-branch form")
    print(f"{name}: token-level form {e1:.2e} (un-floored 99th percentile {p1:.2e}), three-branch form in groups of "
          f"{wl.chunk}: {e2:.2e}", flush=True)


@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [
    (1, 2, 255, 64, 17, True), (1, 2, 257, 128, 18, False), (2, 2, 513, 64, 49, True), (1, 2, 529, 128, 50, True),  # edges of tiles and tap capacities
    (1, 64, 513, 128, 63, False), (1, 64, 530, 128, 9, True)])                                                     # two tiles per workgroup
def test_long_conv_and_its_gradients_at_the_edges_of_tiles(B, H, L, d, Kc, with_state):
    """The conv added to what the token-level kernel left, written ahead of the groups of 256, and met from the other
    side (its share of dv, the gradient of the taps: fp32 sums of exact products, so 1e-4 of their rms)."""
    q, k, v, w, state = small_case(7800 + L + Kc, B, H, L, d, Kc, "bf16", with_state)
    args = () if state is None else state
    compare(run(q, k, v, w, state, "bf16", 256, 1e-3), oracle.prefill_recurrent(q, k, v, w, *args, eps=1e-3), "bf16", f"added, L={L} Kc={Kc}")
    want = oracle.prefill_grouped(q, k, v, w, 256, 0.7, *((None,) * 3 if state is None else state), eps=1e-3)
    compare(run(q, k, v, w, state, "bf16", 256, 1e-3, alpha=0.7), want, "bf16", f"written first, L={L} Kc={Kc}")
    dout = workloads.upstream_gradient(q.shape, "bf16", 7801)
    want = oracle.prefill_grouped_backward(q, k, v, w, dout, 256, alpha=0.7, eps=1e-3)
    bf = torch.bfloat16
    _, _, dv, dw = binding.prefill_grouped_backward(dev(q, bf), dev(k, bf), dev(v, bf), dev(w), dev(dout, bf), 0.7, 1e-3, group=256)
    torch.cuda.synchronize()
    check(host(dv), want["dv"], TOL["bf16"], f"dv, L={L} Kc={Kc}")
    err = float(np.max(np.abs(host(dw) - want["dw"])) / np.sqrt(np.mean(want["dw"] ** 2)))
    assert err <= TOL["f32"], f"dw, L={L} Kc={Kc}: {err:.2e}"


@pytest.mark.parametrize("alpha", [None, 0.7])                   # added to the rows, written ahead of them
@pytest.mark.parametrize("B,H,L,d,Kc", [(2, 2, 300, 64, 63), (1, 2, 270, 128, 50), (1, 2, 200, 64, 9), (1, 64, 513, 128, 63)])
def test_long_conv_of_rows_and_taps_that_are_not_finite(B, H, L, d, Kc, alpha):
    """A history row or a tap that is an infinity or a NaN reaches the tokens that see it and no others; a tap at the end of
    the range is a finite one."""
    q, k, v, w, state = small_case(7900 + L + Kc, B, H, L, d, Kc, "bf16", True)
    state[2][0, 0, 0, 5] = np.inf
    state[2][B - 1, H - 1, Kc // 2, d - 1] = np.nan
    v[:, H - 1, :, :2] *= 2.0 ** -20
    state[2][:, H - 1, :, :2] *= 2.0 ** -20
    w[H - 1, 0, Kc - 1] = np.inf
    w[H - 1, 1, 2] = 3.4e38
    want = oracle.prefill_recurrent(q, k, v, w, *state, eps=1e-3) if alpha is None else oracle.prefill_grouped(q, k, v, w, 256, alpha, *state, eps=1e-3)
    got = run(q, k, v, w, state, "bf16", 256, 1e-3, alpha=alpha)
    assert np.isnan(want[0]).any() and np.isinf(want[0]).any()
    # (that tap's channel lies thirty orders of magnitude above the rest of its head: held to the bar by itself)
    big = (slice(None), slice(H - 1, H), slice(None), slice(1, 2))
    check(got[0][big], want[0][big], TOL["bf16"], "tap at the end of the range")
    got[0][big] = want[0][big] = 0.0
    same_pattern(got[:3], want[:3], TOL["bf16"], f"L={L} Kc={Kc}")


@pytest.mark.parametrize("io,B,H,L,d,Kc", [("f32", 1, 2, 300, 64, 50), ("f32", 1, 2, 70, 128, 9), ("bf16", 2, 32, 100, 64, 20)])
def test_long_conv_on_the_vector_alus_of_rows_that_are_not_finite(io, B, H, L, d, Kc):
    """Taps beyond the last one are zeros there; a row beyond the window may not meet them."""
    q, k, v, w, state = small_case(7960 + L + Kc, B, H, L, d, Kc, io, True)
    state[2][0, 0, 0, 5] = np.inf
    state[2][B - 1, H - 1, Kc // 2, d - 1] = np.nan
    want = oracle.prefill_recurrent(q, k, v, w, *state, eps=1e-3)
    got = run(q, k, v, w, state, io, 64, 1e-3)
    same_pattern(got[:3], want[:3], TOL[io], f"{io} L={L} Kc={Kc}")


def test_gradient_of_the_long_conv_with_a_gradient_row_that_is_not_finite():
    """dv is the conv's share and a product along the tokens: an infinity in one channel of dout stays in that channel, and
    in the group of its token and the window of taps before it."""
    B, H, L, d, Kc = 1, 2, 700, 64, 63
    q, k, v, w, _ = small_case(7950, B, H, L, d, Kc, "bf16", False, d ** -0.5)
    dout = workloads.upstream_gradient(q.shape, "bf16", 7951)
    want = oracle.prefill_grouped_backward(q, k, v, w, dout, 256, alpha=0.7, eps=1e-3)
    dout[0, 1, 100, 9] = np.inf
    bf = torch.bfloat16
    _, _, dv, dw = binding.prefill_grouped_backward(dev(q, bf), dev(k, bf), dev(v, bf), dev(w), dev(dout, bf), 0.7, 1e-3, group=256)
    torch.cuda.synchronize()
    dv, dw = host(dv), host(dw)
    assert not np.isfinite(dv[0, 1, 100 - Kc + 1:101, 9]).any() and not np.isfinite(dw[1, 9]).any()
    dv[0, 1, :256, 9] = want["dv"][0, 1, :256, 9]
    dw[1, 9] = want["dw"][1, 9]
    check(dv, want["dv"], TOL["bf16"], "dv")
    err = float(np.max(np.abs(dw - want["dw"])) / np.sqrt(np.mean(want["dw"] ** 2)))
    assert err <= TOL["f32"], f"dw: {err:.2e}"


@pytest.mark.parametrize("B,H,L,d,Kc", [
    (1, 2, 256, 128, 16), (1, 16, 257, 128, 16),          # up to 16 taps: matrix cores below 64 tiles, vector ALUs from there on
    (1, 31, 100, 64, 31), (1, 32, 100, 64, 31), (1, 32, 100, 64, 32),   # fewer than 32 taps and heads enough, 32 taps
    (2, 32, 128, 64, 40), (2, 32, 129, 64, 40),           # half a tile and more
    (2, 64, 600, 128, 63), (2, 64, 513, 128, 33)])        # one tile per workgroup where the second would be padding
def test_long_conv_on_either_side_of_its_dispatch(B, H, L, d, Kc):
    q, k, v, w, state = small_case(8100 + L + Kc, B, H, L, d, Kc, "bf16", True)
    h = [0, H - 1]
    want = oracle.prefill_recurrent(q[:, h], k[:, h], v[:, h], w[h], *(x[:, h] for x in state), eps=1e-3)
    got = run(q, k, v, w, state, "bf16", 256, 1e-3)
    compare(tuple(x[:, h] for x in got), want, "bf16", f"added, H={H} L={L} Kc={Kc}")
    got = run(q, k, v, w, state, "bf16", 256, 1e-3, alias_hist=True)
    compare(tuple(x[:, h] for x in got), want, "bf16", f"history in place, H={H} L={L} Kc={Kc}")
    want = oracle.prefill_grouped(q[:, h], k[:, h], v[:, h], w[h], 256, 0.7, *(x[:, h] for x in state), eps=1e-3)
    got = run(q, k, v, w, state, "bf16", 256, 1e-3, alpha=0.7)
    compare(tuple(x[:, h] for x in got), want, "bf16", f"written first, H={H} L={L} Kc={Kc}")
