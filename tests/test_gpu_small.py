"""The calls around an update at the sizes where they take the launches for small batches, and just beyond: limits of tokens, turns,
trajectories, groups and bytes, streams that start inside a block of tokens, masks at odd addresses.  Expected values as in
tests/test_gpu_large.py."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2605_26646_amd as umas
from oracle import umas_oracle as orc
from tests import arraywise as aw
from tests import parity as P
from tests.test_gpu_large import check_front_arraywise, check_ready_batch_arraywise
from tests.test_gpu_sizes import check_update

pytestmark = pytest.mark.gpu


def sized_graph(seed, n_tokens, n_turns, n_traj, n_models, n_roles, group):
    """A seeded graph of exactly these numbers: turns and trajectories may be empty."""
    rng = np.random.default_rng([31, seed])
    w = wl.make_workload(0)
    w.n_traj, w.n_turns, w.n_roles, w.n_models, w.n_tokens = n_traj, n_turns, n_roles, n_models, n_tokens
    w.traj_turn_off = np.concatenate([[0], np.sort(rng.integers(0, n_turns + 1, n_traj - 1)), [n_turns]]).astype(np.int32)
    w.turn_tok_off = np.concatenate([[0], np.sort(rng.integers(0, n_tokens + 1, n_turns - 1)), [n_tokens]]).astype(np.int64)
    w.turn_role = rng.integers(0, n_roles, n_turns).astype(np.int32)
    w.role_to_model = (np.arange(n_roles) % n_models).astype(np.int32)
    w.turn_pred_off, w.turn_pred = None, None
    density = rng.choice(np.array([0.0, 0.02, 0.5, 1.0], np.float32), n_turns)
    w.tok_mask = (rng.random(n_tokens, dtype=np.float32) < np.repeat(density, np.diff(w.turn_tok_off))).astype(np.uint8) * 7
    w.traj_reward = rng.normal(size=n_traj).astype(np.float32)
    w.traj_group = rng.permutation((np.arange(n_traj) // group).astype(np.int32)) if group else None
    w.role_reward = rng.normal(size=n_traj * n_roles).astype(np.float32) if n_traj * n_roles < 4000 else None
    w.turn_reward = rng.normal(size=n_turns).astype(np.float32)
    w.w_role, w.w_turn, w.w_traj = (rng.random(n_roles).astype(np.float32) for _ in range(3))
    w.value = rng.normal(size=n_tokens).astype(np.float32)
    return w


def route(w, place_mode, shift=0):
    mask = torch.zeros(w.n_tokens + shift, dtype=torch.uint8, device="cuda")
    mask[shift:] = P.to_dev(w.tok_mask)
    return umas.umas_assign_token_rewards(
        n_roles=w.n_roles, n_models=w.n_models, role_to_model=w.role_to_model, traj_turn_off=w.traj_turn_off, turn_role=w.turn_role,
        turn_tok_off=w.turn_tok_off, tok_mask_global=mask[shift:], traj_group=w.traj_group, role_reward=w.role_reward,
        turn_reward=w.turn_reward, traj_reward=w.traj_reward, w_role=w.w_role, w_turn=w.w_turn, w_traj=w.w_traj, place_mode=place_mode,
        norm_eps=w.norm_eps)


@pytest.mark.parametrize("n_tokens,n_turns,n_traj,n_models,n_roles,group", [
    (1, 1, 1, 1, 1, 0), (3, 5, 4, 2, 3, 1), (1023, 1, 1, 1, 1, 0), (4096, 7, 3, 1, 3, 2), (4097, 7, 3, 2, 3, 0), (8191, 512, 40, 3, 5, 3),
    (20000, 2, 1024, 2, 2, 8), (30000, 100, 256, 8, 19, 2), (30000, 100, 258, 4, 4, 2), (65536, 512, 65, 8, 8, 0), (65536, 3, 2, 1, 2, 0),
    (65537, 512, 65, 8, 8, 0), (60000, 513, 65, 4, 4, 5), (50000, 40, 1025, 1, 1, 0)])
@pytest.mark.parametrize("place_mode,shift", [(wl.PLACE_LAST, 0), (wl.PLACE_ALL, 3)])
def test_routing_around_the_limits_of_one_launch(n_tokens, n_turns, n_traj, n_models, n_roles, group, place_mode, shift):
    w = sized_graph(n_tokens + n_turns, n_tokens, n_turns, n_traj, n_models, n_roles, group)
    s = route(w, place_mode, shift)
    adv, ret = umas.umas_advantages(s, P.to_dev(w.value), 0.99, 0.95, 0.9, wl.SEG_TRAJ)
    check_front_arraywise(w, s, adv, ret, place_mode, wl.SEG_TRAJ, 0.99, 0.95, 0.9)


@pytest.mark.parametrize("n_tokens,n_turns,n_traj,n_models", [
    (1, 1, 1, 1), (500, 64, 33, 1), (3000, 65, 64, 2), (9000, 257, 65, 3), (60000, 1024, 256, 4), (200000, 9, 2, 1), (90000, 300, 128, 8),
    (20000, 1025, 256, 4), (20000, 1000, 257, 1), (20000, 1000, 205, 5)])
@pytest.mark.parametrize("share", [0.8, 0.0, None])
def test_ready_batch_around_the_limits_of_one_launch(n_tokens, n_turns, n_traj, n_models, share):
    w = sized_graph(n_tokens + n_turns, n_tokens, n_turns, n_traj, n_models, n_models + 1, 0)
    s = route(w, wl.PLACE_LAST)
    rng = np.random.default_rng(n_tokens)
    keep = None if share is None else (rng.random(n_traj) < share).astype(np.uint8)
    order = None if share is None else rng.permutation(n_traj).astype(np.int32)
    sa = aw.streams(w)
    for M in (1, 7, 300):
        check_ready_batch_arraywise(w, s, sa, np.ones(n_traj, np.uint8) if keep is None else keep,
                                    np.arange(n_traj, dtype=np.int32) if order is None else order, M)
    if share is None:                                    # neither given
        rows, off = umas.umas_ready_batch(s, w.traj_turn_off, 3)
        want_rows, want_off = aw.ready_batch(w, sa, np.ones(n_traj, np.uint8), np.arange(n_traj, dtype=np.int32), 3, False)
        assert np.array_equal(off.cpu().numpy(), want_off) and np.array_equal(rows.cpu().numpy()[:len(want_rows)], want_rows)


@pytest.mark.parametrize("n_tokens,n_turns,n_traj", [(1, 1, 1), (16385, 1, 1), (18000, 2, 1), (65536, 1, 1), (65535, 3, 2), (65537, 3, 2), (50001, 40, 2)])
@pytest.mark.parametrize("seg_mode,gamma,lam,gamma_turn,values", [
    (wl.SEG_TURN, 1.0, 1.0, 1.0, False), (wl.SEG_TURN, 0.99, 0.95, 1.0, True), (wl.SEG_TRAJ, 1.0, 0.9, 0.9, False), (wl.SEG_TRAJ, 0.99, 0.95, 0.9, True)])
def test_scan_of_few_tokens_in_long_segments(n_tokens, n_turns, n_traj, seg_mode, gamma, lam, gamma_turn, values):
    w = sized_graph(n_tokens, n_tokens, n_turns, n_traj, 1, 2, 0)
    if not values:
        w.value = None
    s, adv, ret = P.gpu_front(w, place_mode=wl.PLACE_ALL, seg_mode=seg_mode, gamma=gamma, lam=lam, gamma_turn=gamma_turn)
    check_front_arraywise(w, s, adv, ret, wl.PLACE_ALL, seg_mode, gamma, lam, gamma_turn)


# from 8 388 608 tokens on routing and scan store past the caches: the last block whole, with a wavefront of part of its tokens, with a thread of part of
# its four; turns of a few tokens (blocks of more segments than the 256 that are held beside others; on average less than 17, 17 and more), of some more, of some hundred (several in a
# wavefront's 256 tokens) and long
@pytest.mark.parametrize("n_tokens", [(1 << 23) - 1, 1 << 23, (1 << 23) + 1023, (1 << 23) + 2050])
@pytest.mark.parametrize("n_turns,n_models,seg_mode,gamma_turn,values", [
    (300, 1, wl.SEG_TRAJ, 0.9, True), (40001, 3, wl.SEG_TURN, 1.0, False), (400001, 2, wl.SEG_TRAJ, 0.9, True), (480001, 2, wl.SEG_TURN, 1.0, True), (540001, 2, wl.SEG_TURN, 1.0, True)])
def test_front_end_on_both_sides_of_the_cache(n_tokens, n_turns, n_models, seg_mode, gamma_turn, values):
    w = sized_graph(n_tokens, n_tokens, n_turns, max(n_turns // 3, 1), n_models, n_models + 1, 0)
    by_model = np.argsort(w.role_to_model[w.turn_role], kind="stable")
    starts = np.concatenate([[0], np.cumsum(np.diff(w.turn_tok_off)[by_model])])
    held = [np.searchsorted(starts, min(b + 4096, n_tokens) - 1, side="right") - np.searchsorted(starts, b, side="right") + 1 <= 256 for b in range(0, n_tokens, 4096)]
    assert all(held) if n_turns < 450000 else any(held) and not all(held)
    if not values:
        w.value = None
    s, adv, ret = P.gpu_front(w, place_mode=wl.PLACE_LAST, seg_mode=seg_mode, gamma=0.99, lam=0.95, gamma_turn=gamma_turn)
    check_front_arraywise(w, s, adv, ret, wl.PLACE_LAST, seg_mode, 0.99, 0.95, gamma_turn)


@pytest.mark.parametrize("n_tokens,n_turns,seg_mode,gamma_turn", [(20000, 1, wl.SEG_TURN, 1.0), (49152, 2, wl.SEG_TRAJ, 0.9), (49153, 2, wl.SEG_TRAJ, 0.9), (65536, 2, wl.SEG_TRAJ, 1.0),
                                                                  (5000, 40, wl.SEG_TURN, 1.0), (100000, 3, wl.SEG_TRAJ, 0.9)])
@pytest.mark.parametrize("over", ["adv over the rewards, ret over the values", "ret over the rewards", "adv over the values"])
def test_scan_written_over_its_inputs(n_tokens, n_turns, seg_mode, gamma_turn, over):
    from paper_2605_26646_amd import binding
    w = sized_graph(n_tokens, n_tokens, n_turns, 1, 1, 2, 0)
    w.tok_mask[:] = 1
    s, lib = route(w, wl.PLACE_ALL), umas.load_library()
    value = P.to_dev(w.value)
    want = umas.umas_advantages(s, value, 0.99, 0.95, gamma_turn, seg_mode)
    ws = torch.empty(lib.umas_advantages_workspace_bytes(n_tokens), dtype=torch.uint8, device="cuda")
    for _ in range(10):
        r, v, adv, ret = s.tok_reward.clone(), value.clone(), torch.empty_like(value), torch.empty_like(value)
        out = {"adv over the rewards, ret over the values": (r, v), "ret over the rewards": (adv, r), "adv over the values": (v, ret)}[over]
        fields = {f: getattr(s, f).data_ptr() for f, _ in binding._Streams._fields_}
        st = binding._Streams(**{**fields, "tok_reward": r.data_ptr()})
        status = lib.umas_advantages(binding.C.addressof(st), n_tokens, n_turns, v.data_ptr(), 0.99, 0.95, gamma_turn, seg_mode, out[0].data_ptr(), out[1].data_ptr(),
                                     ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert status == 0, lib.umas_last_error().decode()
        for got, x in zip(out, want):   # float32 maps composed in two orders: the tolerance of the scan's own tests
            assert (got - x).abs().max() <= 1e-5 * max(1.0, float(x.abs().max()))


@pytest.mark.parametrize("n", [1, 7, 8192, 8193, 49153, 65536, 65537])
@pytest.mark.parametrize("density", [0.0, 0.6])
def test_kl_rewards_of_few_tokens(n, density):
    rng = np.random.default_rng(n)
    r = rng.normal(size=n).astype(np.float32)
    logp = rng.uniform(-3.0, 0.0, n).astype(np.float32)
    ref = (logp + 0.1 * rng.standard_normal(n)).astype(np.float32)
    mask = (rng.random(n) < density).astype(np.uint8)
    want, kl_want = orc.kl_penalised_rewards(r, logp, ref, mask, 0.05)
    for in_place in (False, True):
        x = P.to_dev(r)
        got, kl = umas.umas_kl_rewards(x, P.to_dev(logp), P.to_dev(ref), P.to_dev(mask), 0.05, out=x if in_place else None)
        got = got.cpu().numpy()
        assert np.array_equal(got[mask == 0].view(np.uint32), r[mask == 0].view(np.uint32))
        # r - beta * kl in float32: the product and the difference round once each
        assert (np.abs(got - want) <= 2.0 ** -23 * (np.abs(r) + 0.05 * np.abs(logp.astype(np.float64) - ref)) + 1e-30).all()
        # each float32 difference is half a unit in its last place off, their float64 sum is exact to 1e-12
        assert abs(float(kl.cpu()[0]) - kl_want) <= 2.0 ** -24 * (abs(kl_want) + np.abs(logp.astype(np.float64) - ref).max())


@pytest.mark.parametrize("over", ["logp", "logp_ref"])
def test_kl_rewards_written_over_the_log_probs(over):
    n, g = 46000, torch.Generator(device="cuda").manual_seed(1)
    r, logp, ref = (torch.randn(n, device="cuda", generator=g) for _ in range(3))
    mask = (torch.rand(n, device="cuda", generator=g) < 0.8).to(torch.uint8)
    want, want_kl = umas.umas_kl_rewards(r, logp, ref, mask, 0.05)
    for _ in range(20):
        a, b = logp.clone(), ref.clone()
        out, kl = umas.umas_kl_rewards(r, a, b, mask, 0.05, out=a if over == "logp" else b)
        assert torch.equal(out, want)
        assert abs(float(kl) - float(want_kl)) <= 2.0 ** -23 * abs(float(want_kl))   # float64 sums in two orders, rounded once


@pytest.mark.parametrize("rows,d,V", [  # every pair of tile sizes of the two float32 gradient products, 16, 32 and 64 wide
    (1, 1, 1), (60, 33, 100), (255, 64, 512), (1030, 127, 1001), (100, 100, 3000), (100, 512, 8000), (3000, 100, 101), (300, 500, 300),
    (300, 512, 8190), (4001, 512, 60), (4000, 511, 401), (4096, 512, 2100)])
@pytest.mark.parametrize("select", [False, True])
def test_float32_gradient_products_in_every_tile_size(rows, d, V, select):
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    n = rows + 9 if select else rows
    H, W = torch.randn(n, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g) / d ** 0.5
    ids = torch.randint(0, V, (n,), device="cuda", dtype=torch.int32, generator=g)
    adv = torch.randn(n, device="cuda", generator=g)
    sel = torch.randperm(n, device="cuda", generator=g)[:rows].to(torch.int32) if select else None
    dW0 = torch.randn(V, d, device="cuda", generator=g)
    _, logp, dH, dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, None, adv, None, 0, 0.2, accumulate_dW=True, dW=dW0.clone())
    # the same in float64, on-policy: dz = (A / n) (softmax - onehot)
    at = torch.arange(n, device="cuda") if sel is None else sel.long()
    h, w, y = H[at].double(), W.double(), ids[at].long()
    z = h @ w.T
    lp = torch.log_softmax(z, 1)
    dz = torch.exp(lp)
    dz[torch.arange(rows, device="cuda"), y] -= 1.0
    dz *= (adv[at].double() / rows)[:, None]
    want_H, want_lp = torch.zeros(n, d, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    want_H[at], want_lp[at] = dz @ w, lp.gather(1, y[:, None])[:, 0]
    want_W = dW0.double() + dz.T @ h
    # float32 dz and results round once each, the sums are float64: 2^-24 of the terms' magnitudes and of the result, twice that for what comes
    # of the float32 logsumexp and g (a difference in the logsumexp's last place scales every probability of the row)
    lse = torch.logsumexp(z, 1).abs()
    mag = dz.abs() * (4.0 + 4.0 * lse[:, None]) * 2.0 ** -24
    for got, want, bound in ((dH[at], want_H[at], mag @ w.abs()), (dW, want_W, mag.T @ h.abs())):
        assert ((got.double() - want).abs() <= bound + 2.0 ** -23 * want.abs() + 1e-30).all()
    assert (logp.double() - want_lp).abs().max() <= 1e-5 * max(1.0, float(want_lp.abs().max()))
    if select:
        rest = torch.ones(n, dtype=torch.bool, device="cuda")
        rest[at] = False
        assert (dH[rest] == 0).all() and (logp[rest] == 0).all()


@pytest.mark.parametrize("rows,d,V", [(60, 33, 100), (300, 64, 512), (300, 512, 8190), (3000, 100, 101)])
def test_float32_gradient_added_to_the_weights(rows, d, V):
    g = torch.Generator(device="cuda").manual_seed(rows)
    H, W = torch.randn(rows, d, device="cuda", generator=g), torch.randn(V, d, device="cuda", generator=g) / d ** 0.5
    ids = torch.randint(0, V, (rows,), device="cuda", dtype=torch.int32, generator=g)
    adv = torch.randn(rows, device="cuda", generator=g)
    stats, logp, dH, dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, accumulate_dW=True, dW=W.clone())
    for _ in range(5):
        X = W.clone()
        got = umas.umas_ppo_loss_fwd_bwd(H, X, ids, None, None, adv, None, 0, 0.2, accumulate_dW=True, dW=X)
        assert all(torch.equal(a, b) for a, b in zip(got, (stats, logp, dH, dW)))   # the same sums


@pytest.mark.parametrize("rows,V,dead", [(1100, 512, (64, 192)), (1100, 512, (0, 64)), (2000, 2000, (128, 384))])
def test_float32_update_of_vocabulary_that_cannot_be_taken(rows, V, dead):
    """Weights of -infinity on whole parts of the vocabulary: no probability, and nothing for the entropy, as the scoring call has it."""
    g, d = torch.Generator(device="cuda").manual_seed(rows + V), 32
    H, W = torch.randn(rows, d, device="cuda", generator=g).abs() + 0.1, torch.randn(V, d, device="cuda", generator=g) / 8
    W[dead[0]:dead[1]] = 0.0
    W[dead[0]:dead[1], 3] = -float("inf")
    ids = torch.randint(dead[1], V, (rows,), device="cuda", dtype=torch.int32, generator=g)
    lp, _, entropy = umas.umas_policy_logprobs(H, W, ids, None)
    assert entropy.isfinite().all() and (entropy > 0).all()
    stats, logp, _, _ = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, lp, torch.ones(rows, device="cuda"), None, 0, 0.2)
    st = umas.read_stats(stats)[0]
    # float64 sums in two orders, each entropy and log-prob rounded to float32 once
    assert abs(float(st["entropy_mean"]) - float(entropy.double().mean())) <= 2.0 ** -22 * float(entropy.max())
    assert (logp.double() - lp.double()).abs().max() <= 2.0 ** -22 * float(lp.abs().max()) and abs(float(st["loss"]) + 1.0) <= 1e-5


@pytest.mark.parametrize("n,n_sel,shift", [(1, 1, 0), (2, 1, 1), (127, 5, 3), (129, 128, 0), (8300, 3, 2), (8300, 8299, 1), (70000, 50001, 0), (600000, 10, 0), (600000, 480001, 3)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_critic_defines_the_rows_that_are_not_selected(n, n_sel, shift, dtype):
    g = torch.Generator(device="cuda").manual_seed(n_sel)
    d = 72
    H, w = torch.randn(n, d, device="cuda", generator=g).to(dtype), torch.randn(d, device="cuda", generator=g).to(dtype)
    sel = torch.randperm(n, device="cuda", generator=g)[:n_sel].to(torch.int32)
    at = torch.empty(n_sel + shift, dtype=torch.int32, device="cuda")
    at[shift:] = sel                                     # a selection at any multiple of four bytes
    sel, ret, old = at[shift:], torch.randn(n, device="cuda", generator=g), torch.zeros(n, device="cuda")
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    value = umas.umas_values(H, w, 0.5, sel, value=nan(n))
    _, value_new, dH, dw, db = umas.umas_value_loss_fwd_bwd(H, w, 0.5, sel, old, ret, None, 0, 1e9, dH=nan(n, d).to(dtype), value_new=nan(n))
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[sel.long()] = False
    v64 = H[sel.long()].double() @ w.double() + 0.5
    # float32 (bf16 rows) or float64 sums of d products of numbers below 5, rounded once
    assert (value[sel.long()].double() - v64).abs().max() <= d * 25 * 2.0 ** -23
    assert torch.equal(value[rest], torch.zeros_like(value[rest])) and torch.equal(value_new, value)
    assert (dH[rest] == 0).all()
    gr = (v64 - ret[sel.long()].double()) / n_sel
    want = gr[:, None] * w.double()
    eps = 2.0 ** -8 if dtype is torch.bfloat16 else 2.0 ** -22
    assert ((dH[sel.long()].double() - want).abs() <= eps * want.abs() + d * 25 * 2.0 ** -22 / n_sel * w.double().abs()).all()
    kept = nan(n, d).to(dtype)                           # accumulating: other rows keep what they hold
    kept[sel.long()] = 0
    umas.umas_value_loss_fwd_bwd(H, w, 0.5, sel, old, ret, None, 0, 1e9, dH=kept, accumulate_dH=True)
    assert torch.equal(kept[sel.long()], dH[sel.long()]) and kept[rest].isnan().all()


# where rows are cleared in the launch that works on the selected ones, up to 2^20 of them, and where in launches of their own, with a byte a row where it fits
@pytest.mark.parametrize("n,n_sel,d", [(1 << 15, 9, 8), ((1 << 15) + 1, 1 << 15, 16), (1 << 20, 9, 8), ((1 << 20) + 1, (1 << 20) - 77, 16), (1 << 20, 700001, 192),
                                       ((1 << 20) + 1, 400001, 384), (1 << 17, 100001, 640), ((1 << 17) + 1, 9, 640), (2200000, 1900000, 16), (5000, 4001, 2624)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_critic_of_many_rows(n, n_sel, d, dtype):
    g = torch.Generator(device="cuda").manual_seed(n_sel)
    H, w = torch.randn(n, d, device="cuda", generator=g).to(dtype), torch.randn(d, device="cuda", generator=g).to(dtype)
    sel = torch.randperm(n, device="cuda", generator=g)[:n_sel].to(torch.int32)
    ret, old, at = torch.randn(n, device="cuda", generator=g), torch.zeros(n, device="cuda"), sel.long()
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    value = umas.umas_values(H, w, 0.5, sel, value=nan(n))
    _, value_new, dH, _, _ = umas.umas_value_loss_fwd_bwd(H, w, 0.5, sel, old, ret, None, 0, 1e9, dH=nan(n, d).to(dtype), value_new=nan(n))
    # the selected rows alone are the same rows, bit for bit
    _, want_value, want_dH, _, _ = umas.umas_value_loss_fwd_bwd(H[at], w, 0.5, None, old[at], ret[at], None, 0, 1e9)
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[at] = False
    for got in (value, value_new):
        assert torch.equal(got[at], want_value) and (got[rest] == 0).all()
    assert torch.equal(dH[at], want_dH) and (dH[rest] == 0).all()


# the selection as the workgroups that clear read it: in front of, at and behind a multiple of 16 bytes, rounds of 8192 entries, 64 and 128 shares of the rows
@pytest.mark.parametrize("d,dtype", [(512, torch.bfloat16), (512, torch.float32), (1032, torch.bfloat16)])
@pytest.mark.parametrize("n,n_sel", [(127, 3), (8193, 2), (16385, 8192), (20000, 8195), (33000, 32771)])
def test_critic_clears_what_a_shuffled_selection_leaves_out(n, n_sel, d, dtype):
    g = torch.Generator(device="cuda").manual_seed(n)
    H, w = torch.randn(n, d, device="cuda", generator=g).to(dtype), torch.randn(d, device="cuda", generator=g).to(dtype)
    old, ret = torch.zeros(n, device="cuda"), torch.randn(n, device="cuda", generator=g)
    order = torch.randperm(n, device="cuda", generator=g).to(torch.int32)
    for first in range(4):
        sel = order[first:first + n_sel]
        rest = torch.ones(n, dtype=torch.bool, device="cuda")
        rest[sel.long()] = False
        value = umas.umas_values(H, w, 0.5, sel, value=torch.full((n,), float("nan"), device="cuda"))
        _, value_new, dH, _, _ = umas.umas_value_loss_fwd_bwd(H, w, 0.5, sel, old, ret, None, 0, 1e9, dH=torch.full_like(H, float("nan")),
                                                              value_new=torch.full((n,), float("nan"), device="cuda"))
        for got in (value[:, None], value_new[:, None], dH):
            assert (got[rest] == 0).all() and (got[sel.long()] != 0).any(dim=1).all()


# rows of a wavefront around the 64 that its lanes hold at a time, and few
@pytest.mark.parametrize("n_roles", [3, 64])
@pytest.mark.parametrize("n,d,dtype", [(33, 2048, torch.bfloat16), (8191, 512, torch.float32), (18439, 4096, torch.float32), (20493, 8192, torch.bfloat16),
                                       (60001, 1096, torch.bfloat16), (262145, 264, torch.bfloat16), (532481, 8, torch.bfloat16), (530001, 12, torch.float32)])
def test_critic_statistics_and_sums_of_many_rows(n, d, dtype, n_roles):
    g = torch.Generator(device="cuda").manual_seed(n)
    H, w = torch.randn(n, d, device="cuda", generator=g).to(dtype), (torch.randn(d, device="cuda", generator=g) / d ** 0.5).to(dtype)
    ret, old = torch.randn(n, device="cuda", generator=g), torch.randn(n, device="cuda", generator=g)
    role = torch.randint(-1, n_roles + 1, (n,), device="cuda", generator=g).to(torch.int32)      # some have none
    dH0 = (torch.randn(n, d, device="cuda", generator=g) / n).to(dtype)
    stats, V, dH, dw, db = umas.umas_value_loss_fwd_bwd(H, w, 0.5, None, old, ret, role, n_roles, 0.25)
    v64, r64, o64, V = V.double(), ret.double(), old.double(), V.double()
    assert all((V[i:i + 65536] - (H[i:i + 65536].double() @ w.double() + 0.5)).abs().max() <= 2.0 ** -22 * 5 * d ** 0.5 * 5 for i in range(0, n, 65536))
    vc = torch.minimum(torch.maximum(v64, o64 - 0.25), o64 + 0.25)
    lu, lc = (v64 - r64) ** 2, (vc - r64) ** 2
    loss, clipped = 0.5 * torch.maximum(lu, lc), lu < lc
    st = umas.read_value_stats(stats)
    for k in range(1 + n_roles):
        at = role == k - 1 if k else torch.ones_like(clipped)
        count = int(at.sum())
        assert int(st["n_scored"][k]) == count
        if count:                                        # losses are float32, summed in 64 bits; a row at the line may fall either way
            assert abs(float(st["loss"][k]) - float(loss[at].mean())) <= 2.0 ** -19 * float(loss[at].mean())
            assert abs(float(st["clip_frac"][k]) - float(clipped[at].double().mean())) <= 2.0 / count + 1e-6
            assert abs(float(st["value_mean"][k]) - float(v64[at].mean())) <= 2.0 ** -22 * float(v64[at].abs().max())
    near = ((lu - lc).abs() <= 1e-5 * lu) & clipped | ((lu - lc).abs() <= 1e-5 * lu) & (vc != v64)
    gr = torch.where(clipped, 0.0, (v64 - r64) / n)
    eps = 2.0 ** -8 if dtype is torch.bfloat16 else 2.0 ** -21
    for i in range(0, n, 65536):
        want, ok = gr[i:i + 65536, None] * w.double(), ~near[i:i + 65536]
        assert ((dH[i:i + 65536].double() - want).abs() <= eps * want.abs() + 1e-30)[ok].all()
    # dw and db: float32 sums of at most n terms, and what the rows at the line could add
    room = (((v64 - r64).abs() / n)[near]).sum()
    want, size = torch.zeros(d, dtype=torch.float64, device="cuda"), torch.zeros(d, dtype=torch.float64, device="cuda")
    for i in range(0, n, 65536):
        h = H[i:i + 65536].double()
        want += gr[i:i + 65536] @ h
        size += gr[i:i + 65536].abs() @ h.abs()
    assert ((dw.double() - want).abs() <= 2.0 ** -16 * size + 6 * room).all()
    assert abs(float(db) - float(gr.sum())) <= 2.0 ** -16 * float(gr.abs().sum()) + float(room)
    added = umas.umas_value_loss_fwd_bwd(H, w, 0.5, None, old, ret, role, n_roles, 0.25, accumulate_dH=True, dH=dH0.clone())[2]
    for i in range(0, n, 65536):
        term = gr[i:i + 65536, None] * w.double()
        want, ok = dH0[i:i + 65536].double() + term, ~near[i:i + 65536]
        assert ((added[i:i + 65536].double() - want).abs() <= eps * want.abs() + 2.0 ** -21 * term.abs() + 1e-30)[ok].all()


def test_values_of_more_rows_than_32_bits_count():
    """Row 2^32 + 5 is not selected by an entry 5 (the values of 2^32 rows are 17 GB, their rows of 16 bytes, of which three are read, 69 GB)."""
    n, d = (1 << 32) + (1 << 20), 4
    H, value = torch.empty(n, d, device="cuda"), torch.empty(n, device="cuda")
    sel = torch.tensor([5, 70000, (1 << 31) - 1], dtype=torch.int32, device="cuda")
    H[sel.long()] = 1.0
    value.fill_(float("nan"))
    umas.umas_values(H, torch.ones(d, device="cuda"), 0.5, sel, value=value)
    assert torch.equal(value[sel.long()], torch.full((3,), 4.5, device="cuda"))
    value[sel.long()] = 0.0
    assert all((part == 0).all() for part in value.split(1 << 30))
    del H, value
    torch.cuda.empty_cache()


@pytest.mark.parametrize("shape", ["alike", "front", "back", "blocks", "none"])
@pytest.mark.parametrize("n_models", [1, 3])
def test_ready_batch_of_masks_that_are_not_alike(shape, n_models):
    """The guesses at a run's first row and at a turn's trajectory, where the density of scored tokens or of turns says little."""
    n_traj, rng = 3000, np.random.default_rng(5)
    w = sized_graph(11, 500000, 9000, n_traj, n_models, n_models + 1, 0)
    if shape != "alike":                                 # trajectories of very different numbers of turns
        cuts = np.sort(rng.choice([0, 1, 2, 4500, 8999, 9000], n_traj - 1))
        w.traj_turn_off = np.concatenate([[0], cuts, [9000]]).astype(np.int32)
    at = np.arange(w.n_tokens)
    w.tok_mask = {"alike": rng.random(w.n_tokens) < 0.8, "front": at < 7000, "back": at > w.n_tokens - 7000, "blocks": at // 30000 % 3 == 0,
                  "none": at < 0}[shape].astype(np.uint8)
    s = route(w, wl.PLACE_LAST)
    check_ready_batch_arraywise(w, s, aw.streams(w), (rng.random(n_traj) < 0.9).astype(np.uint8), rng.permutation(n_traj).astype(np.int32), 5)


# slices around one entry a lane, around one and four 16-byte vectors a lane, at every boundary of 4 bytes on either side
@pytest.mark.parametrize("lengths", [(0, 1, 2, 3, 5), (63, 64, 65, 66, 67, 68, 71), (255, 256, 257, 260, 263), (1023, 1024, 1025, 1027, 1031, 2111)])
@pytest.mark.parametrize("n_models", [1, 2])
def test_ready_batch_slices_of_these_lengths(lengths, n_models):
    n_traj, rng = 1500, np.random.default_rng(len(lengths))
    w = sized_graph(3, 16, 2 * n_traj, n_traj, n_models, n_models, 0)
    tokens = rng.choice(np.array(lengths), 2 * n_traj)
    w.n_tokens, w.turn_tok_off = int(tokens.sum()), np.concatenate([[0], np.cumsum(tokens)]).astype(np.int64)
    w.traj_turn_off, w.turn_role = np.arange(n_traj + 1, dtype=np.int32) * 2, (np.arange(2 * n_traj) % 2 % n_models).astype(np.int32)
    w.tok_mask, w.value = np.ones(w.n_tokens, np.uint8), None
    if n_models == 1:                                    # one turn of a trajectory is all there is
        w.tok_mask[np.repeat(np.arange(2 * n_traj) % 2 == 1, tokens)] = 0
    s = route(w, wl.PLACE_LAST)
    check_ready_batch_arraywise(w, s, aw.streams(w), (rng.random(n_traj) < 0.8).astype(np.uint8), rng.permutation(n_traj).astype(np.int32), 7)


# chunks of 256 rows, each with slices of dH that are added up before the next chunk's; the last chunk's go with the rest of the update
@pytest.mark.parametrize("n,d,V", [(257, 64, 3000), (600, 1032, 1300)])
@pytest.mark.parametrize("entropy_coef", [0.0, 0.01])
def test_update_with_slices_in_several_chunks(n, d, V, entropy_coef):
    nbytes = umas.ppo_workspace_bytes(n, d, V, torch.bfloat16, 0, minimum=True) + 3 * -(-d // 256) * (256 * 256 * 4)
    check_update(np.random.default_rng(n), n, d, V, select=1.0, entropy_coef=entropy_coef, accumulate=True,
                 workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))


# Few rows, or few in the last block of 256: halves of a block (128 rows) change the scores' tiles and the half of the wavefronts that multiplies
# for dH, steps of 64 rows the length of dW's sums and dH's loads; the vocabulary ends in either half of its last block
@pytest.mark.parametrize("entropy_coef", [0.0, 0.01])
@pytest.mark.parametrize("d,V", [(64, 2048), (72, 2049), (264, 5120 + 128), (512, 1281 + 128)])
@pytest.mark.parametrize("rows", [1, 63, 64, 65, 127, 128, 129, 192, 193, 257, 320, 321, 384, 385])
def test_update_of_rows_that_fill_part_of_a_block(rows, d, V, entropy_coef):
    check_update(np.random.default_rng([rows, d, V]), rows, d, V, select=1.0, entropy_coef=entropy_coef, accumulate=rows % 3 == 0)


# logits that spread far: the block's dz is computed once more, over what the half tiles have left
@pytest.mark.parametrize("rows,d,V", [(100, 64, 2305), (128, 72, 2433), (300, 64, 3000)])
def test_update_of_part_of_a_block_that_is_computed_again(rows, d, V):
    check_update(np.random.default_rng([rows, d, V]), rows, d, V, select=1.0, scale=12.0)


# a head that the caches don't hold, whose weights dH reads past them
@pytest.mark.parametrize("rows", [90, 200])
def test_update_of_few_rows_with_a_large_head(rows):
    check_update(np.random.default_rng(rows), rows, 2048, 66000, select=1.0)


# dW of 1 GiB and more (1.25 below 129 rows), which has a launch of its own up to 256 rows: a column tile of eight columns, a step of 32 rows that is partly
# filled; up to 128 rows the operand comes in halves of its blocks, whose other rows nobody has written; added to in rows that start at 64 bytes and in the middle
@pytest.mark.parametrize("d,V,rows,entropy_coef,accumulate,apart", [
    (4088, 82200, 65, 0.0, False, True), (4088, 82200, 96, 0.0, True, True), (4088, 82200, 97, 0.0, False, True), (4088, 82200, 128, 0.0, True, True),
    (4088, 82200, 100, 0.01, True, True), (4104, 65500, 70, 0.0, True, False), (4104, 65500, 200, 0.01, False, True), (4104, 65500, 256, 0.0, True, True),
    (4104, 65500, 257, 0.0, False, False), (4096, 82200, 99, 0.0, True, True), (2064, 66000, 60, 0.0, True, False)])
def test_update_of_few_rows_with_a_large_gradient(d, V, rows, entropy_coef, accumulate, apart):
    umas.profile_enable(True)
    try:
        check_update(np.random.default_rng(rows), rows, d, V, select=1.0, entropy_coef=entropy_coef, accumulate=accumulate)
        launched = umas.profile_read()
    finally:
        umas.profile_enable(False)
    assert ("k_dw_short" in launched) == apart and ("k_score_keep_narrow" in launched) == (rows <= 128 and entropy_coef == 0)


# rows so wide that dW's lie farther apart than 32-bit offsets of a tile's pieces reach (a product of the two overflows from 4.33 million columns on), and
# the widest that are not; in a launch of its own and beside dH; a vocabulary block that is whole and one that is not
@pytest.mark.parametrize("rows,accumulate", [(130, False), (130, True), (40, True)])
@pytest.mark.parametrize("d", [1 << 22, 4400008])
def test_update_of_very_wide_rows(rows, d, accumulate):
    V, g = 259, torch.Generator(device="cuda").manual_seed(rows)
    H = torch.randn(rows, d, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, d, device="cuda", generator=g) / d ** 0.5 / 64).bfloat16()
    ids, adv = torch.randint(0, V, (rows,), device="cuda", generator=g, dtype=torch.int32), torch.randn(rows, device="cuda", generator=g)
    dW0 = torch.randn(V, d, device="cuda", generator=g) / rows if accumulate else None
    dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, accumulate_dW=accumulate, dW=dW0.clone() if accumulate else None)[3]
    z = sum(H[:, i:i + 65536].double() @ W[:, i:i + 65536].double().T for i in range(0, d, 65536))
    dz = torch.softmax(z, 1) - torch.nn.functional.one_hot(ids.long(), V)
    dz *= adv.double()[:, None] / rows
    for i in range(0, d, 65536):
        h = H[:, i:i + 65536].double()
        want, size = dz.T @ h, dz.abs().T @ h.abs()
        got = dW[:, i:i + 65536].double()
        if accumulate:
            want, size = want + dW0[:, i:i + 65536].double(), size + 2.0 ** -16 * dW0[:, i:i + 65536].double().abs()
        # probability and scaled row are bf16, 2^-9 each.  A logit, below 5/64, is a float32 sum of d / 32 products that may each lose 2^-23 of it:
        # less than 2^-9, and the logsumexp as much.  (With logits of unit size, 64 times that, three quarters of 2^-7 were not enough.)
        worst = float(((got - want).abs() / size).max())
        assert worst <= 2.0 ** -7, (i, worst)


# New log-probs written over the old ones: these are gone when the surrogate looks at them, as if none were given.  One launch for the rows would
# read some of them first; more rows than one launch takes, for comparison
@pytest.mark.parametrize("rows", [60, 300, 2100])
def test_update_that_writes_the_new_log_probs_over_the_old_ones(rows):
    rng = np.random.default_rng(rows)
    n, d, V = rows + rows // 4, 64, 700
    H, W = (P.to_dev(wl.round_to_bf16(rng.normal(size=s).astype(np.float32)), torch.bfloat16) for s in ((n, d), (V, d)))
    ids, sel = P.to_dev(rng.integers(0, V, n).astype(np.int32)), P.to_dev(np.sort(rng.choice(n, rows, replace=False)).astype(np.int32))
    adv, old, role = P.to_dev(rng.normal(size=n).astype(np.float32)), P.to_dev(rng.normal(size=n).astype(np.float32)), P.to_dev(rng.integers(0, 2, n).astype(np.int32))
    want = umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, None, adv, role, 2, 0.2)
    got = umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, old, adv, role, 2, 0.2, logp_new=old)
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    assert (got[3] - want[3]).norm() <= 1e-4 * want[3].norm()        # atomic order of the one-hot rows
    a, b = umas.read_stats(got[0]), umas.read_stats(want[0])
    assert all(np.allclose(a[k], b[k], rtol=1e-6, atol=1e-9) for k in a.dtype.names)
