"""linattn_prefill on the GPU against the CPU oracle (through the C ABI)."""
import numpy as np
import pytest
import torch

import oracle
from parity import TOL, check, check_unfloored, dev, host
from paper_2406_07368_amd import binding, workloads

pytestmark = pytest.mark.gpu

IO = {"f32": torch.float32, "bf16": torch.bfloat16}


def small_case(seed, B, H, L, d, Kc, io, with_state, scale=1.0):
    rng = np.random.default_rng(seed)
    q, k, v = (workloads.round_to_io(rng.standard_normal((B, H, L, d)) * scale, io) for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    state = None
    if with_state:
        S0 = (rng.standard_normal((B, H, d, d)) * 3.0).astype(np.float32)
        z0 = (np.abs(rng.standard_normal((B, H, d))) * 5.0 + 1.0).astype(np.float32)
        h0 = workloads.round_to_io(rng.standard_normal((B, H, Kc - 1, d)), io)
        state = (S0, z0, h0)
    return q, k, v, w, state


def run_gpu(q, k, v, w, state, io, chunk=64, eps=0.0):
    dt = IO[io]
    st = None if state is None else (dev(state[0]), dev(state[1]), dev(state[2], dt))
    out, (S, z, h) = binding.prefill(dev(q, dt), dev(k, dt), dev(v, dt), dev(w), st, chunk, eps)
    torch.cuda.synchronize()
    return host(out), host(S), host(z), host(h)


def compare(got, want, io, what=""):
    tol = TOL[io]
    e = check(got[0], want[0], tol, what + " out")
    check(got[1], want[1], tol, what + " S")
    check(got[2], want[2], tol, what + " z")
    assert np.array_equal(got[3], want[3]), what + " hist"
    return e


def test_config1_fp32_against_brute_force_quadratic():
    """B1 H4 L256 d64, all fp32, Kc 3: every output against the definition, to 1e-4."""
    wl = workloads.CONFIGS["cfg1_fp32_tiny"]
    q, k, v, w = workloads.prefill_inputs(wl)
    want = oracle.prefill_quadratic(q, k, v, w)
    got = run_gpu(q, k, v, w, None, "f32", wl.chunk)
    compare(got, want, "f32", "config 1")


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("d,chunk", [(64, 64), (128, 64), (128, 128), (64, 128)])
@pytest.mark.parametrize("L,Kc,with_state", [(1, 3, False), (63, 3, True), (64, 1, False), (65, 5, True),
                                             (200, 3, False), (333, 8, True), (512, 2, True)])
def test_prefill_matches_oracle_small(io, d, chunk, L, Kc, with_state):
    """Several tiles and a ragged tail, with and without an incoming state."""
    B, H = 2, 3
    q, k, v, w, state = small_case(1000 + L + d + Kc, B, H, L, d, Kc, io, with_state)
    args = () if state is None else state
    want = oracle.prefill_recurrent(q, k, v, w, *args, eps=1e-3)
    got = run_gpu(q, k, v, w, state, io, chunk, eps=1e-3)
    compare(got, want, io, f"L={L} d={d} C={chunk}")


@pytest.mark.parametrize("d,chunk,L,Kc,with_state", [(128, 64, 2100, 5, True), (64, 128, 4099, 3, False),
                                                     (128, 128, 3000, 8, True), (64, 64, 1024, 2, True)])
def test_few_heads_long_sequence_is_segmented(d, chunk, L, Kc, with_state):
    """B*H far below the number of compute units: the sequence axis is cut into segments whose start
    states come from a first pass and a prefix sum; results must not change."""
    B, H = 1, 2
    desc = binding.make_desc(B, H, d, Kc, chunk, torch.bfloat16, L=L)
    assert binding.linattn_workspace_bytes(desc, L) > 0
    q, k, v, w, state = small_case(2000 + L, B, H, L, d, Kc, "bf16", with_state)
    args = () if state is None else state
    want = oracle.prefill_recurrent(q, k, v, w, *args)
    got = run_gpu(q, k, v, w, state, "bf16", chunk)
    compare(got, want, "bf16", f"segmented L={L}")


def test_state_outputs_may_alias_state_inputs():
    """S_out/z_out/hist_out pointing at S_in/z_in/hist_in, with and without segments."""
    for (B, H, L, d, chunk, Kc) in ((2, 3, 200, 128, 64, 3), (1, 2, 2100, 64, 64, 4), (1, 1, 2, 128, 64, 5)):
        q, k, v, w, state = small_case(77 + L, B, H, L, d, Kc, "bf16", True)
        want = oracle.prefill_recurrent(q, k, v, w, *state)
        dt = torch.bfloat16
        S, z, h = dev(state[0]), dev(state[1]), dev(state[2], dt)
        out = torch.empty((B, H, L, d), dtype=dt, device="cuda")
        desc = binding.make_desc(B, H, d, Kc, chunk, dt, L=L)
        nbytes = binding.linattn_workspace_bytes(desc, L)
        ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
        binding.linattn_prefill(desc, L, dev(q, dt), dev(k, dt), dev(v, dt), dev(w), S, z, h, out, S, z, h, ws, nbytes)
        torch.cuda.synchronize()
        compare((host(out), host(S), host(z), host(h)), want, "bf16", f"aliased L={L}")


def test_config2_full():
    """GPT-2-small shape, B4 H12 L1024 d64 bf16: every head against the recurrent oracle."""
    wl = workloads.CONFIGS["cfg2_gpt2_small"]
    q, k, v, w = workloads.prefill_inputs(wl)
    want = oracle.prefill_recurrent(q, k, v, w)
    got = run_gpu(q, k, v, w, None, "bf16", wl.chunk)
    compare(got, want, "bf16", "config 2")


def _full_size_every_head(name, L=None, token_major=False, heads_per_call=32):
    """The workload at full size on the GPU; the oracle follows every head from the same inputs, a block of heads
    at a time (all host threads; whole workload: seconds)."""
    wl = workloads.CONFIGS[name]
    if L is not None:
        wl = wl.small(L=L)
    q, k, v, w = workloads.prefill_tensors(wl)
    gq, gk, gv = q.cuda(), k.cuda(), v.cuda()
    if token_major:   # [B,L,H,d] in memory, seen as [B,H,L,d]
        gq, gk, gv = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (gq, gk, gv))
    out, (S, z, h) = binding.prefill(gq, gk, gv, w.cuda(), None, wl.chunk)
    assert out.stride() == gq.stride()
    torch.cuda.synchronize()
    del gq, gk, gv
    out, S, z, h = out.cpu(), S.cpu(), z.cpu(), h.cpu()
    worst, worst_p99 = 0.0, 0.0
    for b in range(wl.B):
        for h0 in range(0, wl.H, heads_per_call):
            sl = (slice(b, b + 1), slice(h0, min(h0 + heads_per_call, wl.H)))
            want = oracle.prefill_recurrent(host(q[sl]), host(k[sl]), host(v[sl]), w[sl[1]].numpy())
            got = (host(out[sl]), host(S[sl]), host(z[sl]), host(h[sl]))
            worst = max(worst, compare(got, want, "bf16", f"{name} batch row {b} heads {h0}.."))
            worst_p99 = max(worst_p99, check_unfloored(got[0], want[0], TOL["bf16"], f"{name} batch row {b} heads {h0}.. out"))
    print(f"{name}{' token-major' if token_major else ''}: {wl.B * wl.H} heads, worst out error {worst:.2e}, "
          f"99th percentile of the un-floored error {worst_p99:.2e}", flush=True)
    return worst


def test_config3_full_size_every_head():
    """LLaMA-2-7B layer shape B8 H32 L4096 d128 bf16 at full size; all 256 heads against the oracle."""
    _full_size_every_head("cfg3_llama7b_prefill")


def test_config3_full_size_token_major_every_head():
    """The same workload with q, k, v, out laid out [B,L,H,d] (what a projection GEMM writes and
    what bench.py times); all 256 heads against the oracle."""
    _full_size_every_head("cfg3_llama7b_prefill", token_major=True)


def test_config5_long_context_every_head():
    """B1 H32 L65536 d128, chunk 128, Kc 5 at full length; all 32 heads against the oracle."""
    _full_size_every_head("cfg5_long_context", heads_per_call=16)


def test_workspace_does_not_grow_with_length():
    wl = workloads.CONFIGS["cfg5_long_context"]
    sizes = []
    for L in (8192, 16384, 32768, 65536):
        desc = binding.make_desc(wl.B, wl.H, wl.d, wl.conv_k, wl.chunk, torch.bfloat16, L=L)
        sizes.append(binding.linattn_workspace_bytes(desc, L))
    assert len(set(sizes)) == 1


@pytest.mark.parametrize("io,d,chunk", [("bf16", 128, 64), ("bf16", 64, 128), ("f32", 64, 64)])
def test_split_invariance_on_gpu(io, d, chunk):
    """prefill(L) == prefill(L1) then prefill(L - L1) from the handed-over state (to rounding)."""
    B, H, L, Kc = 1, 4, 300, 3
    q, k, v, w, _ = small_case(55, B, H, L, d, Kc, io, False)
    full = run_gpu(q, k, v, w, None, io, chunk)
    for L1 in (1, 64, 130):
        a = run_gpu(q[:, :, :L1], k[:, :, :L1], v[:, :, :L1], w, None, io, chunk)
        st = (a[1].astype(np.float32), a[2].astype(np.float32), a[3].astype(np.float32))
        b = run_gpu(q[:, :, L1:], k[:, :, L1:], v[:, :, L1:], w, st, io, chunk)
        tol = 1e-5 if io == "f32" else 1.2e-2
        check(np.concatenate([a[0], b[0]], axis=2), full[0], tol, f"split {L1} out")
        check(b[1], full[1], tol, f"split {L1} S")
        check(b[2], full[2], tol, f"split {L1} z")
        assert np.array_equal(b[3], full[3])


@pytest.mark.parametrize("io,d", [("bf16", 128), ("f32", 64)])
def test_empty_sequence_copies_the_state_through(io, d):
    B, H, Kc = 2, 2, 3
    q, k, v, w, state = small_case(56, B, H, 0, d, Kc, io, True)
    got = run_gpu(q, k, v, w, state, io)
    assert got[0].shape[2] == 0
    for g, s in zip(got[1:], state):
        assert np.array_equal(g, s.astype(np.float64))


@pytest.mark.parametrize("io,d,chunk", [("bf16", 128, 64), ("bf16", 128, 128), ("f32", 64, 64)])
def test_no_leak_from_later_tokens_on_gpu(io, d, chunk):
    """Changing tokens after t (finite values) leaves outputs up to t bit-identical, inside a
    group and across groups."""
    B, H, L, Kc = 1, 2, 200, 3
    q, k, v, w, _ = small_case(57, B, H, L, d, Kc, io, False)
    base = run_gpu(q, k, v, w, None, io, chunk)[0]
    rng = np.random.default_rng(570)
    for t in (0, 17, 63, 64, 130, 198):
        q2, k2, v2 = q.copy(), k.copy(), v.copy()
        for a in (q2, k2, v2):
            a[:, :, t + 1:] = workloads.round_to_io(a[:, :, t + 1:] + 4.0 * rng.standard_normal(a[:, :, t + 1:].shape), io)
        got = run_gpu(q2, k2, v2, w, None, io, chunk)[0]
        assert np.array_equal(got[:, :, :t + 1], base[:, :, :t + 1]), f"leak into tokens <= {t}"
        assert not np.array_equal(got[:, :, t + 1:], base[:, :, t + 1:])


def test_prefill_is_deterministic():
    B, H, L, d, Kc = 2, 8, 700, 128, 3
    q, k, v, w, _ = small_case(58, B, H, L, d, Kc, "bf16", False)
    a = run_gpu(q, k, v, w, None, "bf16")
    b = run_gpu(q, k, v, w, None, "bf16")
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_strided_token_major_layout(io):
    """q, k, v, out stored as [B, L, H, d] (the layout a fused QKV projection leaves behind)."""
    B, H, L, d, Kc = 2, 4, 150, 64, 3
    dt = IO[io]
    q, k, v, w, _ = small_case(59, B, H, L, d, Kc, io, False)
    want = oracle.prefill_recurrent(q, k, v, w)
    tq, tk, tv = (dev(np.ascontiguousarray(a.transpose(0, 2, 1, 3)), dt) for a in (q, k, v))   # [B,L,H,d]
    out = torch.empty_like(tq)
    S = torch.empty((B, H, d, d), device="cuda")
    z = torch.empty((B, H, d), device="cuda")
    h = torch.empty((B, H, Kc - 1, d), device="cuda", dtype=dt)
    desc = binding.make_desc(B, H, d, Kc, 64, dt, strides=(L * H * d, d, H * d))
    nbytes = binding.linattn_workspace_bytes(desc, L)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    binding.linattn_prefill(desc, L, tq, tk, tv, dev(w), None, None, None, out, S, z, h, ws, nbytes)
    torch.cuda.synchronize()
    got = (host(out).transpose(0, 2, 1, 3), host(S), host(z), host(h))
    compare(got, want, io, "token-major")


def test_prefill_then_verify_equals_longer_prefill():
    """Sec. 5.3 (a shared prefix is computed once): prefill(P) -> verify(k) == last k rows of prefill(P + k)."""
    B, H, d, Kc, P, kk = 2, 4, 128, 3, 190, 8
    q, k, v, w, _ = small_case(60, B, H, P + kk, d, Kc, "bf16", False)
    dt = torch.bfloat16
    _, state = binding.prefill(dev(q[:, :, :P], dt), dev(k[:, :, :P], dt), dev(v[:, :, :P], dt), dev(w))
    out = binding.verify(dev(q[:, :, P:], dt), dev(k[:, :, P:], dt), dev(v[:, :, P:], dt), dev(w), state)
    torch.cuda.synchronize()
    want = oracle.prefill_recurrent(q, k, v, w)
    check(host(out), want[0][:, :, P:], TOL["bf16"], "verify after prefill")
    check(host(state[0]), want[1], TOL["bf16"], "S")
    check(host(state[1]), want[2], TOL["bf16"], "z")
    assert np.array_equal(host(state[2]), want[3])


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("L", [40, 300])
def test_a_wait_that_gives_up_shows_as_nan(grouped, L):
    """The waves of a bf16 prefill workgroup wait for each other with bounded polling.  With the limit set so that
    every wait gives up at once (from the host; the kernel still runs to its end), nothing that was computed from
    operands that were not waited for may come back as a number: every output row, S and z are NaN, the history
    (a copy of input rows) is exact.  Back at the default limit the same call is correct again."""
    B, H, d, Kc = 2, 4, 128, 3
    q, k, v, w, _ = small_case(61, B, H, L, d, Kc, "bf16", False)
    dt = torch.bfloat16
    args = (dev(q, dt), dev(k, dt), dev(v, dt), dev(w))
    alpha = 0.5 if grouped else None
    prev = binding.linattn_set_wait_limit(-1)
    try:
        assert prev == 1 << 20
        out, (S, z, h) = binding.prefill(*args, grouped_alpha=alpha)
        torch.cuda.synchronize()
    finally:
        assert binding.linattn_set_wait_limit(0) == -1
    assert torch.isnan(out).all() and torch.isnan(S).all() and torch.isnan(z).all()
    assert np.array_equal(host(h), v[:, :, L - (Kc - 1):])
    out, (S, z, h) = binding.prefill(*args, grouped_alpha=alpha)
    torch.cuda.synchronize()
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=alpha) if grouped else oracle.prefill_recurrent(q, k, v, w)
    compare((host(out), host(S), host(z), host(h)), want, "bf16", "default limit")


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("B,H,L,d,Kc,with_state", [
    (1, 2, 31, 64, 3, True), (1, 4, 33, 128, 8, False), (1, 4, 512, 64, 5, True),      # quadratic kernel, edges of its tiles
    (1, 4, 545, 64, 3, True), (2, 8, 289, 128, 4, True), (1, 40, 257, 64, 8, True),    # token form: segmented walk, quadratic, segmented
    (8, 40, 97, 64, 3, False), (3, 100, 65, 128, 1, True)])                            # token form: one workgroup per head
def test_fp32_rows_on_either_side_of_the_dispatch(grouped, B, H, L, d, Kc, with_state):
    """The fp32 kernels (quadratic, segmented, whole heads) against the oracle; the three-branch form is quadratic at all of
    these sizes.  S and z updated in place take the walk, whole heads at a time."""
    q, k, v, w, state = small_case(6200 + L + d, B, H, L, d, Kc, "f32", with_state)
    args = {} if state is None else dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=0.7, eps=1e-2, **args) if grouped else oracle.prefill_recurrent(q, k, v, w, eps=1e-2, **args)
    gq, gk, gv, gw = dev(q), dev(k), dev(v), dev(w)
    desc = binding.make_desc(B, H, d, Kc, 64, torch.float32, 1e-2, L=L)
    need = binding.linattn_workspace_bytes(desc, L)
    ws = torch.full((max(need, 16) // 4,), float("nan"), device="cuda")
    for in_place in (False, True) if with_state else (False,):
        st = (None, None, None) if state is None else tuple(dev(x) for x in state)
        res = st if in_place else (torch.full((B, H, d, d), float("nan"), device="cuda"), torch.full((B, H, d), float("nan"), device="cuda"),
                                   torch.full((B, H, Kc - 1, d), float("nan"), device="cuda"))
        out = torch.full_like(gq, float("nan"))
        if grouped:
            binding.linattn_prefill_grouped(desc, L, 0.7, gq, gk, gv, gw, *st, out, *res, ws, need)
        else:
            binding.linattn_prefill(desc, L, gq, gk, gv, gw, *st, out, *res, ws, need)
        torch.cuda.synchronize()
        compare((host(out), *(host(x) for x in res)), want, "f32", f"grouped={grouped} L={L} d={d} in place={in_place}")


@pytest.mark.parametrize("form", ["tokens", "grouped"])
@pytest.mark.parametrize("B,H,L,d", [(8, 16, 1100, 128), (8, 8, 1531, 128), (5, 8, 1100, 128),   # 2, 4, 6 segments
                                     (7, 12, 1197, 64), (1, 32, 1100, 128), (1, 4, 1000, 64), (1, 3, 520, 128),
                                     (1, 11, 1000, 128), (1, 12, 1000, 128)])             # eight segments, six
def test_segments_summed_in_the_full_pass_or_by_the_prefix_sum(form, B, H, L, d):
    """A new sequence of few segments adds their increments up in the full pass; handed zeros as its state the same
    sequence takes the prefix sum.  Same order of additions; the segments differ up to 1024 tokens only."""
    q, k, v, w, _ = small_case(3100 + L + H, B, H, L, d, 3, "bf16", False, d ** -0.5)
    bf = torch.bfloat16
    args = (dev(q, bf), dev(k, bf), dev(v, bf), dev(w))
    zeros = (torch.zeros((B, H, d, d), device="cuda"), torch.zeros((B, H, d), device="cuda"),
             torch.zeros((B, H, 2, d), dtype=bf, device="cuda"))
    if form == "tokens":
        one, two = binding.prefill(*args), binding.prefill(*args, zeros)
    else:
        one, two = binding.prefill_grouped(*args, 1.0), binding.prefill_grouped(*args, 1.0, zeros)
    torch.cuda.synchronize()
    for a, b in zip((one[0], *one[1]), (two[0], *two[1])):
        if L > 1024:
            assert torch.equal(a, b)
        else:                                        # increments of other segments: fp32 sums and one rounding apart
            assert (a.float() - b.float()).norm() <= TOL["bf16"] * b.float().norm()
    h = slice(H - 1, H)
    if form == "tokens":
        want = oracle.prefill_recurrent(q[:, h], k[:, h], v[:, h], w[h])
    else:
        want = oracle.prefill_grouped(q[:, h], k[:, h], v[:, h], w[h], 64, alpha=1.0)
    check(host(one[0][:, h]), want[0], TOL["bf16"], "out")
    check(host(one[1][0][:, h]), want[1], TOL["bf16"], "S")


NON_FINITE = [(2, 4, 130, 64, 3), (2, 4, 130, 128, 4),           # quadratic kernel
              (1, 4, 1700, 64, 3), (1, 3, 1700, 128, 5),         # segmented walk
              (8, 40, 130, 64, 2), (3, 100, 129, 128, 8)]        # one workgroup per head


def same_pattern(got, want, tol, what):
    """NaN and infinities exactly where the oracle has them, the rest to the tolerance."""
    for g, w, name in zip(got, want, ("out", "S", "z")):
        assert np.array_equal(np.isnan(g), np.isnan(w)), f"{what} {name}: NaN elsewhere"
        inf = np.isinf(w)
        assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], w[inf]), f"{what} {name}: infinities elsewhere"
        ok = np.isfinite(w)
        check(np.where(ok, g, 0.0), np.where(ok, w, 0.0), tol, f"{what} {name}")


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("B,H,L,d,Kc", NON_FINITE)
@pytest.mark.parametrize("which", ["q", "k"])
def test_fp32_nan_in_q_or_k_reaches_what_it_should(which, B, H, L, d, Kc, grouped):
    q, k, v, w, state = small_case(6300 + L + d, B, H, L, d, Kc, "f32", True)
    x = q if which == "q" else k
    x[0, 1, 45, 7] = np.nan
    x[B - 1, H - 1, L - 2, d - 1] = np.nan
    args = dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=0.7, eps=1e-2, **args) if grouped else oracle.prefill_recurrent(q, k, v, w, eps=1e-2, **args)
    st = tuple(dev(x) for x in state)
    gq, gk, gv, gw = dev(q), dev(k), dev(v), dev(w)
    out, new = (binding.prefill_grouped(gq, gk, gv, gw, 0.7, st, 1e-2) if grouped else binding.prefill(gq, gk, gv, gw, st, 64, 1e-2))
    torch.cuda.synchronize()
    got = (host(out), host(new[0]), host(new[1]))
    assert np.isnan(want[0]).any()
    same_pattern(got, want, TOL["f32"], f"NaN in {which}")


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("B,H,L,d,Kc", NON_FINITE)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_fp32_value_row_that_is_not_finite_stays_out_of_earlier_tokens(value, B, H, L, d, Kc, grouped):
    """No output depends on a later token, whatever that token holds: masked keys and taps that do not exist may not enter
    with weight zero.  One such value in the middle of a tile, one near the end, one in the oldest row of the history."""
    q, k, v, w, state = small_case(6400 + L + d, B, H, L, d, Kc, "f32", True)
    def call():
        st = tuple(dev(x) for x in state)
        gq, gk, gv, gw = dev(q), dev(k), dev(v), dev(w)
        out, new = (binding.prefill_grouped(gq, gk, gv, gw, 0.7, st, 1e-2) if grouped else binding.prefill(gq, gk, gv, gw, st, 64, 1e-2))
        torch.cuda.synchronize()
        return out, host(out), host(new[0]), host(new[1])
    clean = call()[0].clone()
    v[0, 1, 45, 7] = value
    v[B - 1, H - 1, L - 2, d - 1] = value
    state[2][B - 1, H - 1, 0, 5] = value
    args = dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=0.7, eps=1e-2, **args) if grouped else oracle.prefill_recurrent(q, k, v, w, eps=1e-2, **args)
    out, *got = call()
    assert torch.equal(out[0, 1, :45], clean[0, 1, :45])
    same_pattern(got, want, TOL["f32"], f"{value} in v")


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("B,H,d_v", [(1100, 60, 64), (550, 60, 128)])
def test_fp32_more_heads_than_a_grid_axis_counts(grouped, B, H, d_v):
    """B H (d_v / d) beyond 65535: the descriptor takes B H up to 2^24."""
    if grouped and d_v != 64:
        return                                                   # the three-branch form takes d_v = d only
    L, d, Kc = 3, 64, 3
    rng = np.random.default_rng(6500)
    q, k, v = (rng.standard_normal((B, H, L, n)).astype(np.float32) for n in (d, d, d_v))
    w = workloads.conv_weights(rng, H, d_v, Kc)
    if grouped:
        out, _ = binding.prefill_grouped(dev(q), dev(k), dev(v), dev(w), 0.7, None, 1e-2, want_state=False)
    else:
        out, _ = binding.prefill(dev(q), dev(k), dev(v), dev(w), None, 64, 1e-2, want_state=False)
    torch.cuda.synchronize()
    out = host(out)
    for b in (slice(0, 2), slice(B - 2, B)):
        if grouped:
            want = oracle.prefill_grouped(q[b], k[b], v[b], w, 64, alpha=0.7, eps=1e-2)
        else:
            want = oracle.prefill_recurrent(q[b], k[b], v[b], w, eps=1e-2)
        check(out[b], want[0], TOL["f32"], f"B={B} rows {b}")


@pytest.mark.parametrize("form,B,H,L,d,d_v,Kc,segments", [
    ("grouped", 1, 4, 1601, 64, 64, 3, True), ("grouped", 2, 8, 801, 128, 128, 5, True), ("grouped", 1, 40, 577, 64, 64, 8, True),
    ("grouped", 8, 40, 130, 64, 64, 3, False), ("grouped", 3, 100, 129, 128, 128, 8, False),
    ("tokens", 1, 3, 700, 64, 128, 5, True), ("tokens", 2, 4, 513, 64, 128, 8, True), ("tokens", 1, 2, 520, 128, 256, 3, True),
    ("tokens", 8, 40, 70, 64, 128, 4, False)])
def test_fp32_walk_in_segments_or_whole_heads(form, B, H, L, d, d_v, Kc, segments):
    """The walk over an incoming state, which segments get through the workspace (history rows as floats behind the sums):
    the three-branch form beyond its quadratic kernel, and value rows wider than key rows.  A segmented plan leaves its sums in
    the workspace, so a change of the plan does not leave these cases to another kernel unnoticed."""
    rng = np.random.default_rng(6600 + L + d)
    q, k, v = (rng.standard_normal((B, H, L, n)).astype(np.float32) for n in (d, d, d_v))
    w = workloads.conv_weights(rng, H, d_v, Kc)
    state = ((rng.standard_normal((B, H, d, d_v)) * 3.0).astype(np.float32), (np.abs(rng.standard_normal((B, H, d))) * 5.0 + 1.0).astype(np.float32),
             rng.standard_normal((B, H, Kc - 1, d_v)).astype(np.float32))
    args = dict(S0=state[0], z0=state[1], hist0=state[2])
    want = oracle.prefill_grouped(q, k, v, w, 64, alpha=0.7, eps=1e-2, **args) if form == "grouped" else oracle.prefill_recurrent(q, k, v, w, eps=1e-2, **args)
    gq, gk, gv, gw = dev(q), dev(k), dev(v), dev(w)
    desc = binding.make_desc(B, H, d, Kc, 64, torch.float32, 1e-2, L=L, d_v=d_v)
    need = binding.linattn_workspace_bytes(desc, L)
    ws = torch.full((max(need, 16) // 4,), float("nan"), device="cuda")
    for buf in (ws, None) if segments else (ws,):               # no workspace: the same call, not split
        st = tuple(dev(x) for x in state)
        out, res = torch.full_like(gv, float("nan")), tuple(torch.full_like(x, float("nan")) for x in st)
        nbytes = 0 if buf is None else need
        if form == "grouped":
            binding.linattn_prefill_grouped(desc, L, 0.7, gq, gk, gv, gw, *st, out, *res, buf, nbytes)
        else:
            binding.linattn_prefill(desc, L, gq, gk, gv, gw, *st, out, *res, buf, nbytes)
        torch.cuda.synchronize()
        compare((host(out), *(host(x) for x in res)), want, "f32", f"{form} L={L} d={d} d_v={d_v} workspace={nbytes}")
    assert bool(torch.isfinite(ws).any()) == segments


@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("B,H,L,d", [(1, 8, 256, 64), (2, 4, 289, 128), (1, 8, 1200, 64), (2, 16, 400, 128)])   # quadratic kernel, walk
def test_fp32_three_branch_rounds_no_more_than_short_chains_do(B, H, L, d, unit):
    """Rows of d^-1/2 or of unit normals (where the logits' rounding shows).  The bound is what fp32 arithmetic reaches with the
    logits and the local outputs in four chains per row (4.7e-8 to 4.9e-8 and 5.9e-8 to 6.1e-8 at d = 64, 4.9e-8 and 6.6e-8 at
    d = 128, over lengths of 64 to 4000), and 1 % for the draw; one chain each gives 5.2e-8 and 8.1e-8, 5.3e-8 and 9.9e-8."""
    rng = np.random.default_rng(6700 + L)
    scale = 1.0 if unit else d ** -0.5
    q, k = ((rng.standard_normal((B, H, L, d)) * scale).astype(np.float32) for _ in range(2))
    v = rng.standard_normal((B, H, L, d)).astype(np.float32)
    w = (rng.standard_normal((H, d, 3)) * 0.5).astype(np.float32)
    out, _ = binding.prefill_grouped(dev(q), dev(k), dev(v), dev(w), 1.0, None, 0.0, want_state=False)
    want = oracle.prefill_grouped(q, k, v, w, 64)[0]
    err = float(np.linalg.norm(host(out).astype(np.float64) - want) / np.linalg.norm(want))
    assert err <= {64: (4.95e-8, 6.15e-8), 128: (5.0e-8, 6.7e-8)}[d][unit], err


@pytest.mark.parametrize("form", ["tokens", "grouped"])
@pytest.mark.parametrize("B,H,L,d,d_v,Kc,layout,phi", [
    (1, 4, 65, 64, 64, 3, "bhld", "elu1"), (2, 16, 447, 128, 128, 5, "blhd", "elu1"), (1, 36, 448, 128, 128, 1, "bhld", "elu1"),
    (1, 37, 448, 128, 128, 3, "bhld", "elu1"),                                            # 259 groups: one workgroup per head
    (4, 32, 128, 128, 128, 8, "blhd", "relu"), (1, 3, 129, 64, 64, 63, "bhld", "elu1"), (1, 3, 449, 64, 64, 3, "bhld", "elu1"),   # 8 groups: segments
    (3, 5, 300, 64, 128, 4, "blhd", "elu1"), (2, 8, 191, 64, 192, 2, "bhld", "relu"), (1, 2, 64, 64, 64, 3, "bhld", "elu1")])
def test_short_sequences_with_a_workgroup_per_group(form, B, H, L, d, d_v, Kc, layout, phi):
    """A new sequence of 2 to 7 groups: every group's workgroup forms the state before it.  The same sums in the same order as the
    walk over a head, which a call with a state of zeros takes: the same bits, up to seven groups; and the oracle's numbers."""
    if form == "grouped" and d_v != d:
        pytest.skip("value rows as wide as key rows")
    rng = np.random.default_rng(8800 + L + d + Kc)
    q, k = (workloads.round_to_io(rng.standard_normal((B, H, L, d)), "bf16") for _ in range(2))
    v = workloads.round_to_io(rng.standard_normal((B, H, L, d_v)), "bf16")
    w = workloads.conv_weights(rng, H, d_v, Kc)
    bf = torch.bfloat16

    def put(x):
        x = dev(x, bf)
        return x.transpose(1, 2).contiguous().transpose(1, 2) if layout == "blhd" else x
    qd, kd, vd, wd = put(q), put(k), put(v), dev(w)
    zeros = (torch.zeros(B, H, d, d_v, device="cuda"), torch.zeros(B, H, d, device="cuda"), torch.zeros(B, H, Kc - 1, d_v, device="cuda", dtype=bf))
    call = binding.prefill if form == "tokens" else binding.prefill_grouped
    eps = 1e-3 if phi == "relu" else 0.0
    out, st = call(qd, kd, vd, wd, eps=eps, phi=phi)
    out0, st0 = call(qd, kd, vd, wd, state=zeros, eps=eps, phi=phi)
    torch.cuda.synchronize()
    if L <= 448:
        for a, b in zip((out, *st), (out0, *st0)):
            assert torch.equal(a, b)
    if phi == "elu1":
        if form == "tokens":
            want = oracle.prefill_recurrent(q, k, v, w)
        else:
            want = oracle.prefill_grouped(q, k, v, w, 64)
        compare((host(out), host(st[0]), host(st[1]), host(st[2])), want, "bf16", form)


@pytest.mark.parametrize("H,L,Kc,with_state", [(12, 3000, 3, False), (24, 2500, 1, True), (128, 300, 5, True), (255, 300, 8, False)])
def test_fp32_rows_of_64_with_a_workspace_for_half_of_the_segments(H, L, Kc, with_state):
    """The plan asks for up to 1024 segments.  A workspace for the segments of a plan of up to 512 buys these, not none: it is written, to its
    end at most, and the results are the oracle's.  A shorter one is left alone."""
    d = 64
    rng = np.random.default_rng(8900 + L)
    q, k, v = (rng.standard_normal((1, H, L, d)).astype(np.float32) * 0.5 for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    state = (rng.standard_normal((1, H, d, d)).astype(np.float32), np.abs(rng.standard_normal((1, H, d))).astype(np.float32) + 50.0,
             rng.standard_normal((1, H, Kc - 1, d)).astype(np.float32)) if with_state else (None, None, None)
    want = oracle.prefill_recurrent(q, k, v, w, *(state if with_state else ()))
    desc = binding.make_desc(1, H, d, Kc, 64, torch.float32, L=L)
    units = -(-L // 32)
    per = -(-units // min(512 // H, units // 2, 64))
    half = H * (-(-units // per) * (d * d + d) + 8 * d) * 4
    full = binding.linattn_workspace_bytes(desc, L)
    assert half < full
    st = [None if x is None else dev(x) for x in state]
    qd, kd, vd, wd = dev(q), dev(k), dev(v), dev(w)
    for nb, used in ((full, True), (half, True), (half - 16, False)):
        ws = torch.full((full + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        out, S, z = torch.empty(1, H, L, d, device="cuda"), torch.empty(1, H, d, d, device="cuda"), torch.empty(1, H, d, device="cuda")
        h = torch.empty(1, H, Kc - 1, d, device="cuda")
        binding.linattn_prefill(desc, L, qd, kd, vd, wd, *st, out, S, z, h, ws, nb)
        torch.cuda.synchronize()
        assert bool((ws[:nb] != 0xA5).any()) == used and bool((ws[nb:] == 0xA5).all())
        compare((host(out), host(S), host(z), host(h)), want, "f32", f"workspace of {nb}")


@pytest.mark.parametrize("B,H,L,Kc,in_place", [
    (1, 257, 256, 3, True), (2, 150, 289, 1, False), (1, 512, 257, 3, True), (1, 512, 130, 5, False), (1, 513, 300, 3, False),     # three segments, two, whole heads
    (1, 255, 200, 3, True), (1, 170, 450, 8, False), (1, 16, 4100, 3, True), (1, 2, 4200, 5, False)])                              # ... five; up to 64
def test_fp32_rows_of_64_in_up_to_1024_segments(B, H, L, Kc, in_place):
    """Four workgroups per compute unit: against the oracle, from a state that is updated in place, and with the static scratch to the
    bit."""
    d = 64
    rng = np.random.default_rng(8950 + H + L)
    q, k, v = (rng.standard_normal((B, H, L, d)).astype(np.float32) * 0.5 for _ in range(3))
    w = workloads.conv_weights(rng, H, d, Kc)
    S0 = rng.standard_normal((B, H, d, d)).astype(np.float32)
    z0 = np.abs(rng.standard_normal((B, H, d))).astype(np.float32) + 50.0
    h0 = rng.standard_normal((B, H, Kc - 1, d)).astype(np.float32)
    want = oracle.prefill_recurrent(q, k, v, w, S0, z0, h0)
    desc = binding.make_desc(B, H, d, Kc, 64, torch.float32, L=L)
    a = [dev(x) for x in (q, k, v, w)]
    got = []
    for noalloc in (False, True):
        st = [dev(x) for x in (S0, z0, h0)]
        new = st if in_place else [torch.empty_like(x) for x in st]
        out = torch.empty(B, H, L, d, device="cuda")
        if noalloc:
            binding.linattn_prefill_noalloc(desc, L, *a, *st, out, *new)
        else:
            nb = binding.linattn_workspace_bytes(desc, L)
            binding.linattn_prefill(desc, L, *a, *st, out, *new, torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda"), nb)
        torch.cuda.synchronize()
        got.append([host(x) for x in (out, *new)])
        compare(got[-1], want, "f32", f"B{B} H{H} L{L}")
    for x, y in zip(*got):
        assert np.array_equal(x, y)
