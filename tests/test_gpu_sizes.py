"""Sizes at which the update's dispatch changes: edges of tiles, slices and workspaces, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import umas_oracle as orc
from tests import parity as P
import paper_2605_26646_amd as umas

pytestmark = pytest.mark.gpu


def check_update(rng, n, d, V, *, select=0.8, workspace=None, shift_dH=0, entropy_coef=0.0, accumulate=False, scale=1.0, **kw):
    """One update of random rows against the oracle, every entry within the bounds that the arithmetic gives."""
    H = wl.round_to_bf16((rng.normal(size=(n, d)) / np.sqrt(d) * 3).astype(np.float32))
    W = wl.round_to_bf16((scale * rng.normal(size=(V, d))).astype(np.float32))
    ids = rng.integers(0, V, size=n).astype(np.int32)
    sel = np.sort(rng.choice(n, size=max(1, int(select * n)), replace=False)).astype(np.int32)
    rng.shuffle(sel)
    adv = rng.normal(size=n).astype(np.float32)
    logp_o, lse_o, ent_o = orc.score(H, W, ids, sel)
    # a logit more than 50 above the taken token's: the row's block is flagged and its dz computed from the logits once more
    assert scale == 1.0 or logp_o[sel].min() < -50 - np.log(V)
    logp_old = np.zeros(n, np.float32)
    logp_old[sel] = (logp_o[sel] + 0.05 * rng.normal(size=len(sel))).astype(np.float32)
    _, g_o = orc.ppo_loss(logp_o, logp_old, adv, ent_o, sel, np.zeros(n, np.int32), 0, 0.2)
    k_ent = entropy_coef / len(sel)
    if k_ent:
        dH_o, dW_o = orc.lm_head_backward_entropy(H, W, ids, lse_o, ent_o, g_o, entropy_coef, len(sel), sel)
    else:
        dH_o, dW_o = orc.lm_head_backward(H, W, ids, lse_o, g_o, sel)
    buf = torch.empty(n * d + 8, dtype=torch.bfloat16, device="cuda")
    dW0 = (0.01 * rng.normal(size=(V, d))).astype(np.float32) if accumulate else None
    stats, logp_new, dH, dW = umas.umas_ppo_loss_fwd_bwd(
        P.to_dev(H, torch.bfloat16), P.to_dev(W, torch.bfloat16), P.to_dev(ids), P.to_dev(sel), P.to_dev(logp_old), P.to_dev(adv),
        None, 0, 0.2, entropy_coef=entropy_coef, dH=buf[shift_dH:shift_dH + n * d].view(n, d), workspace=workspace,
        accumulate_dW=accumulate, dW=P.to_dev(dW0) if accumulate else None, **kw)
    what = f"n={n} d={d} V={V}"
    assert int(umas.read_stats(stats)["n_scored"][0]) == len(sel), what
    assert np.abs(logp_new.cpu().numpy()[sel] - logp_o[sel]).max() <= 2e-2, what
    dH_g = dH.float().cpu().numpy()
    assert not dH_g[np.setdiff1d(np.arange(n), sel)].any(), what
    dz = P.oracle_dz(H, W, ids, lse_o, g_o, sel, ent_o, k_ent)
    bound_h, bound_w = P.bf16_gradient_bounds(H, W, dz, dH_o, dW_o, sel, ids, lse_o, g_o)
    P.close_bounded(dH_g, dH_o, bound_h, 1e-2, "dH, " + what)
    if accumulate:
        bound_w = bound_w + 2.0 ** -23 * (np.abs(dW0) + np.abs(dW_o))
    P.close_bounded(dW.cpu().numpy() - (dW0 if accumulate else 0), dW_o, bound_w, 1e-2, "dW, " + what)


# one to several row tiles, one and several column tiles (ragged ones too), slices of one vocabulary block and of several,
# a last slice that is short and a last vocabulary block that is nearly empty
@pytest.mark.parametrize("n,d,V", [(1, 64, 513), (30, 8, 1283), (320, 264, 2561), (650, 64, 9000), (400, 1032, 5121)])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("entropy_coef", [0.0, 0.01])
def test_update_with_dh_cut_along_the_vocabulary(n, d, V, accumulate, entropy_coef):
    check_update(np.random.default_rng(n + d), n, d, V, accumulate=accumulate, entropy_coef=entropy_coef)


@pytest.mark.parametrize("n,d,V", [(320, 264, 2561), (650, 64, 9000)])
def test_update_with_dh_cut_along_the_vocabulary_and_flagged_blocks(n, d, V):
    check_update(np.random.default_rng(n), n, d, V, scale=10.0)


# workspaces between the smallest and the recommended one: no room for slices, room in the scoring pass's place (many rows
# in small chunks), room for two
@pytest.mark.parametrize("n,d,V,extra_tiles", [(300, 64, 3000, 0), (300, 64, 3000, 2), (1500, 64, 20000, 0), (700, 128, 5000, 5)])
def test_update_with_room_for_few_slices(n, d, V, extra_tiles):
    n_sel = max(1, int(0.8 * n))
    nbytes = umas.ppo_workspace_bytes(n_sel, d, V, torch.bfloat16, 0, minimum=True) + extra_tiles * (256 * 256 * 4)
    check_update(np.random.default_rng(n), n, d, V, workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))


def test_update_with_dh_at_an_address_that_is_not_a_multiple_of_eight():
    check_update(np.random.default_rng(5), 300, 64, 3000, shift_dH=2)


def updates(n, d, V, calls, **kw):
    """dH and logp_new of the same update for every (bytes of workspace or None, entries by which dH is shifted)."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    H = torch.randn(n, d, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(V, d, device="cuda", generator=gen) / d ** 0.5).bfloat16()
    ids = torch.randint(0, V, (n,), device="cuda", generator=gen, dtype=torch.int32)
    adv = torch.randn(n, device="cuda", generator=gen)
    out = []
    for nbytes, shift in calls:
        buf = torch.empty(n * d + 8, dtype=torch.bfloat16, device="cuda")
        ws = None if nbytes is None else torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        _, logp, dH, _ = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, dH=buf[shift:shift + n * d].view(n, d),
                                                    workspace=ws, **kw)
        out.append((dH.clone(), logp))
    return out


# from 256 tiles of 256 x 256 on (rows x hidden size) every row of dH is one sum over the vocabulary, with every workspace that
# holds chunks of 128 tiles: the same bits.  Smaller chunks are summed over slices: two sums of V + 1 terms in float32 in
# different orders, rounded to bf16
@pytest.mark.parametrize("n,d,V,rows", [(31 * 256 + 1, 2048, 8000, 4096), (65280 + 1, 256, 1500, 32768)])
@pytest.mark.parametrize("entropy_coef", [0.0, 0.01])
def test_large_updates_do_not_depend_on_the_workspace(n, d, V, rows, entropy_coef):
    sized = lambda r: umas.ppo_workspace_bytes(n, d, V, torch.bfloat16, 0, minimum=True) + (r - 256) * 2 * (-(-V // 256) * 256 + d)
    calls = [(None, 0), (sized(rows), 0), (sized(rows + 512) - 256, 0), (sized(6 * rows // 5 // 256 * 256), 0), (None, 2),
             (sized(256), 0), (sized(rows // 2), 0)]
    (first, logp), *others = updates(n, d, V, calls, entropy_coef=entropy_coef)
    assert first.float().abs().max() > 0
    for dH, lp in others[:4]:
        assert torch.equal(dH, first) and torch.equal(lp, logp)
    # dz has magnitudes of |A| <= 6 over n and, with the bonus, entropy_coef |log p| over n; those of a row sum to twice that
    dz = 2 * (6 + entropy_coef * 30) / n
    for dH, lp in others[4:]:
        bound = 2.0 ** -7 * first.float().abs() + (V + 1) * 2.0 ** -23 * dz * 6 / d ** 0.5
        assert torch.equal(lp, logp) and ((dH.float() - first.float()).abs() <= bound).all()


# with an entropy bonus the logits are kept where the workspace has room for them: all rows at once, chunks of at least 128 tiles of
# dH (rows x hidden size), and fewer rows only when they are the whole selection; else, and for hidden sizes below 768, they are computed
# twice.  The same bits
@pytest.mark.parametrize("n,d,V,fits", [(32 * 256 - 3, 2048, 700, {0: 1, 256: 0, 15 * 256: 0, 16 * 256: 2, 31 * 256: 2, 32 * 256: 1}),
                                        (700, 776, 3001, {0: 1, 256: 0}), (700, 264, 3001, {0: 0, 256: 0})])
def test_kept_logits_and_logits_computed_twice_give_the_same(n, d, V, fits):
    pad = lambda x: -(-x // 256) * 256
    gen = torch.Generator(device="cuda").manual_seed(n)
    H = torch.randn(n, d, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(V, d, device="cuda", generator=gen) / d ** 0.5).bfloat16()
    ids = torch.randint(0, V, (n,), device="cuda", generator=gen, dtype=torch.int32)
    adv = torch.randn(n, device="cuda", generator=gen)
    sliced = pad(n) // 256 * (pad(d) // 256) < 256
    results = {}
    for fit, chunks in fits.items():
        ws = None
        if fit:
            nbytes = umas.ppo_workspace_bytes(n, d, V, torch.bfloat16, 0, minimum=True) + fit * (4 * pad(V) + 2 * pad(d)) - 512 * (pad(V) + pad(d))
            ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(255)     # old contents: NaN
        umas.profile_enable(True)
        try:
            stats, logp, dH, dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, entropy_coef=0.01, workspace=ws)
            names = umas.profile_read()
        finally:
            umas.profile_enable(False)
        assert names.get("k_score_logits", (0, 0))[1] == chunks and ("k_dz_tiles" in names) == (chunks == 0), (fit, names)
        results[fit] = umas.read_stats(stats)["loss"][0], logp, dH, dW
    first, *others = results.values()
    for loss, logp, dH, dW in others:
        assert loss == first[0] and torch.equal(logp, first[1])
        assert sliced or torch.equal(dH, first[2])
        # dW: the same products, added up over one chunk or several (float32)
        assert float((dW - first[3]).norm()) <= 2.0 ** -20 * float(first[3].norm())
        assert float((dH.float() - first[2].float()).norm()) <= 2.0 ** -8 * float(first[2].float().norm())


# the same through a selection: two chunks of kept logits, the second of which begins in the middle of the selection, against one
@pytest.mark.parametrize("accumulate", [False, True])
def test_chunks_of_kept_logits_through_a_selection(accumulate):
    n, n_sel, d, V, n_roles, k = 10000, 32 * 256 - 3, 2048, 700, 3, 0.01
    gen = torch.Generator(device="cuda").manual_seed(7)
    H = torch.randn(n, d, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(V, d, device="cuda", generator=gen) / d ** 0.5).bfloat16()
    ids = torch.randint(0, V, (n,), device="cuda", generator=gen, dtype=torch.int32)
    adv = torch.randn(n, device="cuda", generator=gen)
    role = torch.randint(0, n_roles, (n,), device="cuda", generator=gen, dtype=torch.int32)
    sel = torch.randperm(n, device="cuda", generator=gen)[:n_sel].to(torch.int32)
    base = torch.randn(V, d, device="cuda", generator=gen)
    results = []
    for fit, chunks in ((0, 1), (16 * 256, 2)):
        ws = None
        if fit:
            nbytes = umas.ppo_workspace_bytes(n_sel, d, V, torch.bfloat16, n_roles, minimum=True) + fit * (4 * 768 + 2 * d) - 512 * (768 + d)
            ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(255)
        dW, dH, logp_new = base.clone(), torch.full_like(H, float("nan")), torch.full((n,), float("nan"), device="cuda")
        umas.profile_enable(True)
        try:
            stats, *_ = umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, None, adv, role, n_roles, 0.2, entropy_coef=k, accumulate_dW=accumulate,
                                                   dW=dW, dH=dH, logp_new=logp_new, workspace=ws)
            assert umas.profile_read()["k_score_logits"][1] == chunks
        finally:
            umas.profile_enable(False)
        results.append((umas.read_stats(stats), logp_new, dH, dW - base if accumulate else dW))
    (stats, logp_new, dH, dW), (stats_2, logp_2, dH_2, dW_2) = results
    assert np.array_equal(stats, stats_2) and torch.equal(logp_new, logp_2) and torch.equal(dH, dH_2)
    # float64: dz = p (adv / n + k / n (log p + entropy)) - adv / n at the taken token, on-policy (ratio 1)
    x, y, a = H[sel.long()].double(), ids[sel.long()].long(), adv[sel.long()].double()[:, None] / n_sel
    z = x @ W.double().T
    log_p = torch.log_softmax(z, 1)
    p = log_p.exp()
    dz = p * (a + k / n_sel * (log_p - (p * log_p).sum(1, keepdim=True)))
    dz.scatter_add_(1, y[:, None], -a)
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[sel.long()] = False
    assert not logp_new[rest].any() and not dH[rest].any()
    # as in test_rows_beyond_a_panel: roundings of the logits' sums; two roundings to bf16 in every product
    bound = 4 * d ** 0.5 * 2.0 ** -24 * float((x[:256].abs() @ W.double().abs().T).max())
    assert float((logp_new[sel.long()].double() - log_p.gather(1, y[:, None])[:, 0]).abs().max()) <= bound
    # dW added to old values and these taken away again: three roundings of 2^-24 of the old values
    over = 3 * 2.0 ** -24 * float(base.double().norm()) if accumulate else 0.0
    for got, want, slack in ((dH[sel.long()], dz @ W.double(), 0.0), (dW, dz.T @ x, over), (dW_2, dz.T @ x, over)):
        assert float((got.double() - want).norm()) <= 2.0 ** -8 * float(want.norm()) + slack


@pytest.mark.parametrize("n,d,V", [(300, 64, 3000), (700, 1288, 5121)])
def test_updates_do_not_depend_on_the_address_of_dh(n, d, V):
    (a, _), (b, _), (c, _) = updates(n, d, V, [(None, 0), (None, 2), (None, 4)])
    assert torch.equal(a, b) and torch.equal(a, c)


@pytest.mark.parametrize("entropy_coef", [0.0, 0.01])
def test_an_update_allocates_what_its_coefficient_needs(entropy_coef):
    n, d, V = 3000, 776, 5000
    H, W = torch.zeros(n, d, dtype=torch.bfloat16, device="cuda"), torch.zeros(V, d, dtype=torch.bfloat16, device="cuda")
    ids, adv = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.ones(n, device="cuda")
    out = dict(dW=torch.empty(V, d, device="cuda"), dH=torch.empty_like(H), logp_new=torch.empty(n, device="cuda"), stats=torch.empty(64, dtype=torch.uint8, device="cuda"))
    plain, bonus = (umas.ppo_workspace_bytes(n, d, V, torch.bfloat16, 0, entropy_bonus=b) for b in (False, True))
    assert bonus > plain + (24 << 20)
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, entropy_coef=entropy_coef, **out)
    used = torch.cuda.max_memory_allocated() - before
    assert 0 <= used - (bonus if entropy_coef else plain) <= 4 << 20          # the allocator's rounding


# chunks of the update: as few as the workspace allows, from the smallest one (256 rows a chunk) to the recommended one (even
# chunks of at most 65 536 rows), and never more rows than fit
@pytest.mark.parametrize("dt,n,fit", [("bf16", 131072, None), ("bf16", 131073, None), ("bf16", 5000, 1792), ("bf16", 5000, 256), ("bf16", 3000, 2816),
                                      ("bf16", 700, 700), ("f32", 4097, None), ("f32", 4000, 1300), ("f32", 300, 300)])
def test_update_runs_in_as_few_chunks_as_the_workspace_allows(dt, n, fit):
    d, V, dtype, cap = 8, 40, torch.bfloat16 if dt == "bf16" else torch.float32, 65536 if dt == "bf16" else 4096
    row = 2 * (256 + 256) if dt == "bf16" else 4 * V
    pad = lambda rows: -(-rows // 256) * 256
    if fit is None:
        nbytes, chunks = umas.ppo_workspace_bytes(n, d, V, dtype, 0), -(-n // cap)
    else:
        nbytes = umas.ppo_workspace_bytes(n, d, V, dtype, 0, minimum=True) + pad(row * (pad(fit) if dt == "bf16" else fit)) - row * 256
        chunks = 1 if fit >= n else -(-n // (fit // 256 * 256))
    H, W = torch.randn(n, d, device="cuda").to(dtype), torch.randn(V, d, device="cuda").to(dtype)
    ids, adv = torch.randint(0, V, (n,), device="cuda", dtype=torch.int32), torch.randn(n, device="cuda")
    umas.profile_enable(True)
    try:
        umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        launches = umas.profile_read()["k_gemm_dh_dw" if dt == "bf16" else "k_dw_f32"][1]
    finally:
        umas.profile_enable(False)
    assert launches == chunks


def check_scores(rng, n_sel, d, V, select, static):
    n = n_sel + 7 if select else n_sel
    H = wl.round_to_bf16((rng.normal(size=(n, d)) / np.sqrt(d) * 3).astype(np.float32))
    W = wl.round_to_bf16(rng.normal(size=(V, d)).astype(np.float32))
    ids = rng.integers(0, V, size=n).astype(np.int32)
    sel = rng.permutation(n)[:n_sel].astype(np.int32)
    ids[sel[-1]] = V + 1 if n_sel > 1 else V - 1
    good = sel[ids[sel] < V]
    logp_o, lse_o, ent_o = orc.score(H, W, np.minimum(ids, V - 1), sel)
    fn = umas.umas_policy_logprobs_static if static else umas.umas_policy_logprobs
    out = [x.cpu().numpy() for x in fn(P.to_dev(H, torch.bfloat16), P.to_dev(W, torch.bfloat16), P.to_dev(ids), P.to_dev(sel) if select else None)]
    # products are exact in float32: a logit carries d 2^-24 of the sum of its terms' magnitudes, a logsumexp no more
    bound = (d + 64) * 2.0 ** -24 * (np.abs(H[sel]).astype(np.float64) @ np.abs(W).T.astype(np.float64)).max() + 1e-5
    for name, x, o in zip(("logp", "lse", "entropy"), out, (logp_o, lse_o, ent_o)):
        rows = sel if name == "lse" else good
        assert np.abs(x[rows] - o[rows]).max() <= (3 if name == "entropy" else 2) * bound, (name, n_sel, d, V)
    assert not out[0][np.setdiff1d(np.arange(n), good)].any() and not out[2][np.setdiff1d(np.arange(n), good)].any()


# the three scoring kernels for few rows: edges of their row counts, hidden sizes below, at and above a multiple of what
# eight wavefronts share (512), the last one the register-resident kernel takes and the first it does not; vocabularies
# smaller than one block of 16, than the device's workgroups, and with a last block that is nearly empty
@pytest.mark.parametrize("d,V", [(8, 5), (200, 257), (512, 4097), (520, 3000), (2048, 1030), (2056, 700), (4096, 2500), (4104, 300)])
@pytest.mark.parametrize("n_sel", [1, 16, 17, 33, 64, 65, 128, 129])
def test_scoring_of_few_rows(n_sel, d, V):
    check_scores(np.random.default_rng(n_sel + d), n_sel, d, V, select=n_sel % 2 == 1, static=n_sel in (16, 33, 65))


# Logits that are not finite: a NaN or +inf logit makes the row's sums NaN, a -inf logit adds nothing to them (its place in the
# entropy, 0 * inf, is NaN).  Few rows against the same rows among 129, which the tiles score, and against float64: one
# vocabulary entry to a place of the register-resident kernel (V <= 4096) and many, first and last ones of a block of 16,
# hidden sizes that fill eight wavefronts' pieces and that leave some of them without columns.
@pytest.mark.parametrize("d,V", [(512, 5), (64, 1000), (512, 4096), (520, 4112), (1088, 4097), (64, 151936)])
@pytest.mark.parametrize("n_sel", [1, 16, 17, 32, 33, 64, 65])
def test_logits_that_are_not_finite(n_sel, d, V):
    rng = np.random.default_rng(n_sel + d + V)
    H = rng.normal(size=(n_sel, d)).astype(np.float32) / np.sqrt(d).astype(np.float32)
    H[:, -1] = 0.5 + np.abs(H[:, -1])                                # a weight of -inf there is a logit of -inf
    H, W = wl.round_to_bf16(H), wl.round_to_bf16(rng.normal(size=(V, d)).astype(np.float32))
    ids = rng.integers(1, V - 1, size=n_sel).astype(np.int32)
    at = np.unique([0, 16 * ((V - 1) // 32), V - 1])                 # none of them is a taken token
    ids = np.where(np.isin(ids, at), 1, ids).astype(np.int32)
    more = np.arange(129) % n_sel
    inf = np.float32(np.inf)
    for what, h_row, w_at, x in (("NaN weight, last", None, at[-1:], np.nan), ("NaN weight, first", None, at[:1], np.nan),
                                 ("NaN row", n_sel // 2, [], np.nan), ("-inf logits", None, at, -inf), ("inf logit", None, at[1:2], inf)):
        Hx, Wx = H.copy(), W.copy()
        if h_row is not None:
            Hx[h_row] = x
        Wx[w_at, -1] = x
        dev = [P.to_dev(Hx, torch.bfloat16), P.to_dev(Wx, torch.bfloat16), P.to_dev(ids)]
        few = [a.cpu().numpy() for a in umas.umas_policy_logprobs(*dev)]
        idx = P.to_dev(more.astype(np.int64))
        tiles = [a.cpu().numpy()[:n_sel] for a in umas.umas_policy_logprobs(dev[0][idx].contiguous(), dev[1], dev[2][idx].contiguous())]
        keep = np.setdiff1d(np.arange(V), w_at)
        z = H.astype(np.float64) @ W[keep].T.astype(np.float64)
        lse = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
        zy = np.einsum("nk,nk->n", H.astype(np.float64), W[ids].astype(np.float64))
        bad = np.full(n_sel, what in ("NaN weight, last", "NaN weight, first", "inf logit"))
        if h_row is not None:
            bad[h_row] = True
        # exact products: a logit carries d 2^-24 of its terms' magnitudes, the sum of V exponentials (V + 64) 2^-24 of itself at most
        lim = (2 * d * (np.abs(H).astype(np.float64) @ np.abs(W).T.astype(np.float64)).max() + 64 + V / 16) * 2.0 ** -24 + 1e-5
        for name, a, b, want in zip(("logp", "lse"), few, tiles, (zy - lse, lse)):
            assert np.array_equal(np.isnan(a), bad) and np.array_equal(np.isnan(b), bad), (what, name, a, b)
            assert (np.abs(a - want)[~bad] <= lim).all() and (np.abs(a - b)[~bad] <= 2 * lim).all(), (what, name)
        assert np.array_equal(np.isnan(few[2]), np.isnan(tiles[2])), what
        assert np.isnan(few[2]).all() if what == "-inf logits" else np.array_equal(np.isnan(few[2]), bad), what


# enough rows for the merge that does not split a row's tiles over the workgroup, and one less
@pytest.mark.parametrize("n_sel", [19999, 20000])
def test_scoring_of_many_rows(n_sel):
    check_scores(np.random.default_rng(n_sel), n_sel, 64, 700, select=False, static=False)


# more rows than a panel of the logit kernels holds (32 tiles of 8192 columns): two panels of 24 and of 9 tiles, three of 24
@pytest.mark.parametrize("n,V", [(8193, 600), (16641, 1300)])
@pytest.mark.parametrize("entropy_coef", [None, 0.0, 0.01])
def test_rows_beyond_a_panel(n, V, entropy_coef):
    d = 8192
    gen = torch.Generator(device="cuda").manual_seed(n)
    H = torch.randn(n, d, device="cuda", generator=gen).bfloat16()
    W = (0.02 * torch.randn(V, d, device="cuda", generator=gen)).bfloat16()
    ids = torch.randint(0, V, (n,), device="cuda", generator=gen, dtype=torch.int32)
    z = H.double() @ W.double().T
    p = torch.softmax(z, 1)
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, ids.long()[:, None])[:, 0] - lse
    entropy = lse - (p * z).sum(1)
    # float32 sums of d products in any order: a random walk of d roundings of the terms' size, four deviations
    bound = 4 * d ** 0.5 * 2.0 ** -24 * float((H[:256].double().abs() @ W.double().abs().T).max())
    if entropy_coef is None:
        for got, want in zip(umas.umas_policy_logprobs(H, W, ids), (logp, lse, entropy)):
            assert float((got.double() - want).abs().max()) <= bound
        return
    adv = torch.randn(n, device="cuda", generator=gen)
    _, logp_new, dH, dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, None, None, adv, None, 0, 0.2, entropy_coef=entropy_coef)
    assert float((logp_new.double() - logp).abs().max()) <= bound
    k = entropy_coef / n                                             # on-policy: ratio 1, g = -adv / n
    dz = p * (adv.double()[:, None] / n + k * (z - (lse - entropy)[:, None]))
    dz.scatter_add_(1, ids.long()[:, None], -adv.double()[:, None] / n)
    # every product carries two roundings to bf16 (2^-8 together at most), random in sign
    for got, want in ((dH, dz @ W.double()), (dW, dz.T @ H.double())):
        assert float((got.double() - want).norm() / want.norm()) <= 2.0 ** -8


# the one-hot rows of dW: one group of 128 rows spread over many workgroups, several groups over a few, every row the same
# token and every row another; and statistics per role when a wavefront holds one role, many, and roles outside the range
@pytest.mark.parametrize("n,n_tokens", [(1, 1), (127, 1), (129, 129), (700, 3), (5000, 400)])
def test_one_hot_rows_and_statistics_per_role(n, n_tokens):
    rng = np.random.default_rng(n)
    d, V, n_roles = 72, 512, 64
    H = wl.round_to_bf16(rng.normal(size=(n, d)).astype(np.float32) / 4)
    W = wl.round_to_bf16(rng.normal(size=(V, d)).astype(np.float32) / 4)
    ids = rng.integers(0, n_tokens, size=n).astype(np.int32)
    role = np.where(np.arange(n) % 256 < 64, 5, rng.integers(-1, n_roles + 1, size=n)).astype(np.int32)
    adv = rng.normal(size=n).astype(np.float32)
    logp_o, lse_o, ent_o = orc.score(H, W, ids)
    logp_old = (logp_o + 0.1 * rng.normal(size=n)).astype(np.float32)
    inside = np.where((role >= 0) & (role < n_roles), role, n_roles)
    st_o, g_o = orc.ppo_loss(logp_o, logp_old, adv, ent_o, None, inside, n_roles + 1, 0.2)
    dH_o, dW_o = orc.lm_head_backward(H, W, ids, lse_o, g_o)
    stats, _, dH, dW = umas.umas_ppo_loss_fwd_bwd(P.to_dev(H, torch.bfloat16), P.to_dev(W, torch.bfloat16), P.to_dev(ids), None,
                                                  P.to_dev(logp_old), P.to_dev(adv), P.to_dev(role), n_roles, 0.2)
    sg = umas.read_stats(stats)
    assert np.array_equal(sg["n_scored"], st_o[:1 + n_roles, 4].astype(np.int64))
    for j, name in enumerate(("loss", "clip_frac", "entropy_mean", "approx_kl")):
        o = st_o[:1 + n_roles, j]
        # log-probs within 1e-5 move a row's ratio, and a row on the clip boundary by its whole share
        lim = 2.0 / np.maximum(st_o[:1 + n_roles, 4], 1) if name == "clip_frac" else 1e-4 * np.maximum(np.abs(o), 1)
        assert (np.abs(sg[name] - o) <= lim).all(), name
    bound_h, bound_w = P.bf16_gradient_bounds(H, W, P.oracle_dz(H, W, ids, lse_o, g_o, np.arange(n)), dH_o, dW_o, np.arange(n), ids, lse_o, g_o)
    P.close_bounded(dH.float().cpu().numpy(), dH_o, bound_h, 1e-2, "dH")
    P.close_bounded(dW.cpu().numpy(), dW_o, bound_w, 1e-2, "dW")


# the critic's update on both sides of the size from which dH is cleared only where no selected row lies (48 MiB of selected
# rows), with selections that are nearly everything, half and shuffled; more rows than the partial sums have bytes; every
# wavefront of the last workgroup busy and one; the widest rows
@pytest.mark.parametrize("n,n_sel,d,dt", [(1, 1, 8, "bf16"), (70, 5, 8192, "bf16"), (6200, 3071, 8192, "bf16"), (3073, 3072, 8192, "bf16"),
                                          (6209, 3073, 4096, "f32"), (3200000, 3145729, 8, "bf16"), (130001, 98305, 260, "f32"),
                                          (500, 0, 64, "bf16")])
def test_critic_update_clears_the_rows_that_are_not_selected(n, n_sel, d, dt):
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    H = torch.randn(n, d, device="cuda", generator=gen).to(dtype)
    w = (torch.randn(d, device="cuda", generator=gen) / np.sqrt(d)).to(dtype)
    sel = torch.randperm(n, device="cuda", generator=gen)[:n_sel].to(torch.int32)
    R = torch.randn(n, device="cuda", generator=gen)
    dH = torch.full((n, d), 7.0, device="cuda", dtype=dtype)
    value_new = torch.full((n,), 7.0, device="cuda")
    stats, V, dH, dw, db = umas.umas_value_loss_fwd_bwd(H, w, 0.25, sel, torch.zeros(n, device="cuda"), R, None, 0, 1e9,
                                                        dH=dH, value_new=value_new)
    sl = sel.long()
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[sl] = False
    assert not dH[rest].any() and not V[rest].any()
    s = umas.read_value_stats(stats)
    assert int(s["n_scored"][0]) == n_sel
    if n_sel == 0:
        assert not dw.any() and not db.any()
        return
    Hd, wd = H[sl].double(), w.double()
    V_o = Hd @ wd + 0.25
    err_V = (d + 8) * 2.0 ** -24 * (Hd.abs() @ wd.abs() + 1)          # a float32 dot product of exact products
    assert ((V[sl].double() - V_o).abs() <= err_V).all()
    g = (V_o - R[sl].double()) / n_sel                                # the clip range is wide: every row keeps its gradient
    err_g = (err_V + 2.0 ** -22 * (V_o - R[sl].double()).abs()) / n_sel
    rnd = 2.0 ** -8 if dt == "bf16" else 2.0 ** -23
    want = g[:, None] * wd[None, :]
    assert ((dH[sl].double() - want).abs() <= rnd * want.abs() + 2 * err_g[:, None] * wd.abs()[None, :] + 1e-38).all()
    # sums of float32 terms: a wavefront's rows, four wavefronts, then the workgroups; 2^-24 of the magnitudes per addition
    adds = n_sel / min((n_sel + 3) // 4, 256) + 64
    lim = (err_g[:, None] * Hd.abs()).sum(0) + adds * 2.0 ** -24 * (g.abs()[:, None] * Hd.abs()).sum(0)
    assert ((dw.double() - (g[:, None] * Hd).sum(0)).abs() <= lim).all()
    assert abs(float(db) - float(g.sum())) <= float(err_g.sum() + adds * 2.0 ** -24 * g.abs().sum())
    assert abs(float(s["loss"][0]) - float(0.5 * (V_o - R[sl].double()).square().mean())) <= 1e-5 * (1 + float(V_o.square().mean()))


# the float32 products: edges of the 32-entry tiles and of the 16 k of a round, hidden and vocabulary sizes that are not
# multiples of four, K parts that get nothing, the 64 x 64 tiles (V / 64 x d / 64 >= 256) and what just misses them, two
# chunks of rows, and scoring with statistics of many parts, of two and of one
@pytest.mark.parametrize("n,d,V", [(1, 1, 1), (3, 5, 2), (33, 31, 33), (40, 16, 129), (17, 130, 700), (200, 64, 512), (70, 100, 4097),
                                   (90, 1022, 1030), (1100, 1024, 1023), (4500, 24, 77)])
@pytest.mark.parametrize("entropy_coef", [0.0, 0.05])
def test_float32_products(n, d, V, entropy_coef):
    rng = np.random.default_rng(n + d)
    H = rng.normal(size=(n, d)).astype(np.float32)
    H /= np.sqrt(np.mean(H.astype(np.float64) ** 2, 1, keepdims=True)).astype(np.float32)
    W = (rng.normal(size=(V, d)) / np.sqrt(d)).astype(np.float32)
    ids = rng.integers(0, V, size=n).astype(np.int32)
    sel = rng.permutation(n)[:max(1, n - n // 5)].astype(np.int32)
    ids[sel[-1]] = V if len(sel) > 1 else 0
    good = sel[ids[sel] < V]
    safe = np.minimum(ids, V - 1)
    adv = rng.normal(size=n).astype(np.float32)
    adv[ids >= V] = 0                                                  # a row without a valid id has no gradient
    logp_o, lse_o, ent_o = orc.score(H, W, safe, sel)
    dev = [P.to_dev(x) for x in (H, W, ids, sel)]
    full = [x.cpu().numpy() for x in umas.umas_policy_logprobs(*dev)]
    alone = [x.cpu().numpy() for x in umas.umas_policy_logprobs_static(*dev)]
    nbytes = umas.ppo_workspace_bytes(len(sel), d, V, torch.float32, 0, minimum=True)
    for a, b, o, rows in zip(full, alone, (logp_o, lse_o, ent_o), (good, sel, good)):
        # float64 sums, one rounding to float32 (log V + |z| bounds every quantity that is subtracted)
        assert np.abs(a[rows] - o[rows]).max() <= 2.0 ** -22 * (np.abs(lse_o[sel]).max() + 1)
        assert np.abs(a - b).max() <= 2.0 ** -22 * (np.abs(lse_o[sel]).max() + 1)
    logp_old = np.zeros(n, np.float32)
    logp_old[sel] = (logp_o[sel] + 0.01 * rng.normal(size=len(sel))).astype(np.float32)
    _, g_o = orc.ppo_loss(logp_o, logp_old, adv, ent_o, sel, np.zeros(n, np.int32), 0, 0.2)
    if entropy_coef:
        dH_o, dW_o = orc.lm_head_backward_entropy(H, W, safe, lse_o, ent_o, g_o, entropy_coef, len(sel), good)
    else:
        dH_o, dW_o = orc.lm_head_backward(H, W, safe, lse_o, g_o, sel)
    dW0 = (0.01 * rng.normal(size=(V, d))).astype(np.float32)
    for workspace in (None, torch.empty(nbytes, dtype=torch.uint8, device="cuda")):
        stats, logp_new, dH, dW = umas.umas_ppo_loss_fwd_bwd(*dev, P.to_dev(logp_old), P.to_dev(adv), None, 0, 0.2, workspace=workspace,
                                                             entropy_coef=entropy_coef, accumulate_dW=True, dW=P.to_dev(dW0))
        assert int(umas.read_stats(stats)["n_scored"][0]) == len(sel)
        dH_g, dW_g = dH.cpu().numpy(), dW.cpu().numpy()
        # dz is rounded to float32 (its g carries the rounding of a ratio, 1e-6 of it), each result once more
        scale_h = np.abs(dH_o).max() + 1e-12
        assert np.abs(dH_g - dH_o).max() <= 1e-5 * scale_h, (n, d, V)
        assert np.abs(dW_g - dW0 - dW_o).max() <= 1e-5 * (np.abs(dW_o).max() + 1e-12) + 2.0 ** -23 * (np.abs(dW0) + np.abs(dW_o)).max(), (n, d, V)


# float32 scoring with room for the statistics of one, two, five, six and all parts of the vocabulary, on both sides of the
# numbers of rows from which tiles are taken without room, with room for two parts and for six
@pytest.mark.parametrize("n", [1, 256, 257, 512, 768, 769, 1280, 1281])
def test_float32_scoring_with_room_for_few_parts(n):
    rng = np.random.default_rng(n)
    d, V = 36, 2100
    H, W = rng.normal(size=(n, d)).astype(np.float32), (rng.normal(size=(V, d)) / 6).astype(np.float32)
    ids = rng.integers(0, V, size=n).astype(np.int32)
    want = orc.score(H, W, ids)
    dev = [P.to_dev(x) for x in (H, W, ids)]
    for parts in (0, 1, 2, 5, 6, 17):
        out = umas.umas_policy_logprobs(*dev, workspace=torch.empty(max(256, 40 * n * parts), dtype=torch.uint8, device="cuda"))
        for x, o in zip(out, want):
            assert np.abs(x.cpu().numpy() - o).max() <= 2.0 ** -22 * (np.abs(want[1]).max() + 1), (n, parts)


def test_group_numbers_in_order_counted_and_sorted_give_the_same_streams():
    rng = np.random.default_rng(11)
    n_traj, n_roles = 513, 3
    same = rng.permutation(np.arange(n_traj) // 4)                     # the partition; its members lie anywhere
    order = np.argsort(same, kind="stable")
    reward = rng.random(n_traj).astype(np.float32)
    kw = dict(n_roles=n_roles, n_models=1, role_to_model=np.zeros(n_roles, np.int32), traj_turn_off=np.arange(n_traj + 1) * n_roles,
              turn_role=np.tile(np.arange(n_roles), n_traj), turn_tok_off=np.arange(n_traj * n_roles + 1) * 5,
              tok_mask_global=torch.ones(n_traj * n_roles * 5, dtype=torch.uint8, device="cuda"))

    def scalars(group, r):
        return umas.umas_assign_token_rewards(traj_group=group.astype(np.int32), traj_reward=r, **kw).turn_scalar.cpu().numpy().reshape(n_traj, n_roles)

    counted = scalars(same, reward)
    assert np.abs(counted).max() > 0.5
    assert np.array_equal(counted, scalars(same * 10 ** 7 + 3, reward))                    # sorted
    assert np.array_equal(counted[order], scalars(same[order], reward[order]))             # in order
    assert np.array_equal(counted, scalars(same.max() - same, reward))


# one segment as long as the stream: a single range, ranges of one tile that cannot be cut and the first that can, and the
# sizes at which ranges grow from one tile to two
@pytest.mark.parametrize("n", [1, 1023, 1025, 17407, 17408, 40001, 2 * 512 * 1024 - 1, 2 * 512 * 1024 + 5])
@pytest.mark.parametrize("with_value", [False, True])
def test_scan_of_one_segment(n, with_value):
    from scipy.signal import lfilter
    rng = np.random.default_rng(n)
    gamma, lam = 0.99, 0.95
    reward = rng.normal(size=n).astype(np.float32)
    value = rng.normal(size=n).astype(np.float32) if with_value else None
    st = umas.umas_assign_token_rewards(n_roles=1, n_models=1, role_to_model=[0], traj_turn_off=[0, 1], turn_role=[0], turn_tok_off=[0, n],
                                        tok_mask_global=torch.ones(n, dtype=torch.uint8, device="cuda"))
    st.tok_reward.copy_(P.to_dev(reward))
    adv, ret = umas.umas_advantages(st, None if value is None else P.to_dev(value), gamma, lam)
    v = np.zeros(n) if value is None else value.astype(np.float64)
    delta = reward.astype(np.float64) + gamma * np.append(v[1:], 0.0) - v
    want = lfilter([1.0], [1.0, -gamma * lam], delta[::-1])[::-1]
    # the smallest workspace that is accepted (ranges of 8192 tokens, 32 + 40 bytes each) and one that holds ranges of three tiles
    lib, cs = umas.load_library(), st._c()
    for chunk in (8192, 3072):
        ranges = -(-n // chunk)
        ws = torch.empty(-(-32 * ranges // 256) * 256 + -(-40 * ranges // 256) * 256, dtype=torch.uint8, device="cuda")
        adv2, ret2 = torch.empty_like(adv), torch.empty_like(ret)
        rc = lib.umas_advantages(ctypes.addressof(cs), n, 1, None if value is None else (v_dev := P.to_dev(value)).data_ptr(), gamma, lam, 1.0, 0,
                                 adv2.data_ptr(), ret2.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0 and (adv2 - adv).abs().max().item() <= 2e-5 and (ret2 - ret).abs().max().item() <= 2e-5
    # a float32 recurrence that forgets with 0.94 a token: some 17 terms of |delta| <= 10 carry 2^-24 each, folds a few times as many
    assert np.abs(adv.cpu().numpy() - want).max() <= 2e-5
    assert np.abs(ret.cpu().numpy() - want - v).max() <= 2e-5


# block sums (1024 tokens each) times groups at, below and above the number from which their statistics take a launch of
# their own (256), and a last block of one token
@pytest.mark.parametrize("n,n_roles", [(1, 3), (1025, 3), (85 * 1024, 3), (86 * 1024, 3), (255 * 1024 + 1, 1), (257 * 1024, 1), (4 * 1024, 64), (5 * 1024, 64)])
def test_whitening_statistics(n, n_roles):
    rng = np.random.default_rng(n)
    adv = (3 + rng.normal(size=n)).astype(np.float32)
    mask = (rng.random(n) < 0.8).astype(np.uint8)
    role = rng.integers(0, n_roles, size=n).astype(np.int32)
    out = umas.umas_whiten_advantages(P.to_dev(adv), P.to_dev(mask), P.to_dev(role), np.array([0, n]), n_roles, umas.WHITEN_MODEL_ROLE).cpu().numpy()
    a64 = adv.astype(np.float64)
    off = np.array([0, n])
    want = orc.whiten_advantages(a64, mask, role, off, n_roles, orc.WHITEN_MODEL_ROLE)
    bound = P.whiten_bounds(a64, mask, role, off, n_roles, True)
    assert not out[mask == 0].any()
    assert (np.abs(out - want) <= bound).all()


# a wavefront's 256 tokens hold one group, two, a few, many, in lanes of one group and of several; whole wavefronts and a last one of 1, 3 or 255 tokens
@pytest.mark.parametrize("turn", [1, 2, 4, 7, 16, 25, 100, 400])
@pytest.mark.parametrize("n,n_roles", [(1, 3), (259, 3), (1023, 64), (40 * 1024 + 257, 5), (300 * 1024 + 511, 17)])
def test_whitening_statistics_of_turns(n, n_roles, turn):
    rng = np.random.default_rng([n, turn])
    adv = (3 + rng.normal(size=n)).astype(np.float32)
    mask = (rng.random(n) < 0.8).astype(np.uint8)
    role = np.repeat(rng.integers(-1, n_roles + 1, size=n // turn + 1), turn)[:n].astype(np.int32)   # a role outside [0, n_roles) joins no group
    off = np.array([0, n // 3, n])
    out = umas.umas_whiten_advantages(P.to_dev(adv), P.to_dev(mask), P.to_dev(role), off, n_roles, umas.WHITEN_MODEL_ROLE).cpu().numpy()
    known = (role >= 0) & (role < n_roles)
    a64, counted = adv.astype(np.float64), (mask * known).astype(np.uint8)
    want = orc.whiten_advantages(a64, counted, np.where(known, role, 0), off, n_roles, orc.WHITEN_MODEL_ROLE)
    bound = P.whiten_bounds(a64, counted, np.where(known, role, 0), off, n_roles, True)
    assert not out[counted == 0].any()
    assert (np.abs(out - want) <= bound).all()


# a last step of K of 8 to 56 columns, behind none, one and many whole ones of 64: in the narrow tiles (up to 128 rows) and the large
@pytest.mark.parametrize("d", [16, 56, 72, 88, 120, 184, 1000, 1016])
@pytest.mark.parametrize("n_sel", [100, 300])
def test_hidden_sizes_between_multiples_of_64(n_sel, d):
    rng = np.random.default_rng([n_sel, d])
    check_scores(rng, n_sel, d, 1030, True, False)
    check_update(rng, n_sel + 30, d, 1030)
    check_update(rng, n_sel + 30, d, 1030, entropy_coef=0.01)
    check_update(rng, n_sel + 30, d, 1030, entropy_coef=0.01,
                 workspace=torch.empty(umas.ppo_workspace_bytes(int(0.8 * (n_sel + 30)), d, 1030, torch.bfloat16, 0, minimum=True), dtype=torch.uint8, device="cuda"))


# float32: the logits kept in the workspace (all rows, one chunk of them and several) and, in the smallest workspace, computed again
@pytest.mark.parametrize("n,d,V", [(1, 3, 5), (40, 64, 1023), (300, 20, 1025), (1500, 33, 300), (4097, 16, 600)])
@pytest.mark.parametrize("entropy_coef", [0.0, 0.05])
def test_float32_logits_kept_and_computed_twice(n, d, V, entropy_coef):
    gen = torch.Generator(device="cuda").manual_seed(n)
    H, W = torch.randn(n, d, device="cuda", generator=gen), 0.5 * torch.randn(V, d, device="cuda", generator=gen)
    ids = torch.randint(0, V, (n,), device="cuda", generator=gen, dtype=torch.int32)
    adv, old = torch.randn(n, device="cuda", generator=gen), -4 + torch.randn(n, device="cuda", generator=gen)
    sel = torch.randperm(n, device="cuda", generator=gen)[:max(1, n - n // 5)].to(torch.int32)
    sizes = [umas.ppo_workspace_bytes(len(sel), d, V, torch.float32, 0, minimum=m) for m in (False, True)]
    out = []
    for nbytes, kernel in zip(sizes, ("k_dz_kept_f32", "k_dz_f32")):
        umas.profile_enable(True)
        try:
            out.append(umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, old, adv, None, 0, 0.2, entropy_coef=entropy_coef,
                                                  workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(255)))
            assert kernel in umas.profile_read()
        finally:
            umas.profile_enable(False)
    # float64 sums in other orders (the row kernel's, the tiles'), rounded to float32 where log-probs and dz are stored
    for a, b in zip(out[0][1:], out[1][1:]):
        assert float((a - b).norm()) <= 2.0 ** -21 * float(a.norm())


# the log-probs of the KL penalty are read through the caches or past them, by what of the call fits the 256 MiB of the last one
@pytest.mark.parametrize("n", [(256 << 20) // 13, (256 << 20) // 13 + 1, 64 << 20, (64 << 20) + 1])
def test_kl_rewards_on_both_sides_of_the_cache(n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    r, logp = torch.randn(n, device="cuda", generator=gen), -torch.rand(n, device="cuda", generator=gen)
    ref = logp + 0.1 * torch.randn(n, device="cuda", generator=gen)
    mask = (torch.rand(n, device="cuda", generator=gen) < 0.7).to(torch.uint8)
    out, kl = umas.umas_kl_rewards(r, logp, ref, mask, 0.05)
    diff = (logp - ref) * mask
    want = r - 0.05 * diff
    # one rounding of the product (or none) and one of the sum on either side
    assert ((out - want).abs() <= 2.0 ** -23 * (r.abs() + diff.abs())).all() and torch.equal(out[mask == 0], r[mask == 0])
    mean = float(diff.double().sum()) / int(mask.sum())
    assert abs(float(kl) - mean) <= 2.0 ** -23 * abs(mean) + 2.0 ** -40


# ... and the whitened advantages leave the same two ways
@pytest.mark.parametrize("n,scope", [((256 << 20) // 13, umas.WHITEN_MODEL_ROLE), ((256 << 20) // 13 + 1, umas.WHITEN_MODEL_ROLE), ((256 << 20) // 9 + 1, umas.WHITEN_MODEL)])
def test_whitening_on_both_sides_of_the_cache(n, scope):
    rng = np.random.default_rng(n)
    adv, mask, role = (1 + rng.standard_normal(n, dtype=np.float32)), (rng.random(n, dtype=np.float32) < 0.8).astype(np.uint8), rng.integers(0, 2, size=n, dtype=np.int32)
    off = np.array([0, n // 3, n])
    out = umas.umas_whiten_advantages(P.to_dev(adv), P.to_dev(mask), P.to_dev(role), off, 2, scope).cpu().numpy()
    a64 = adv.astype(np.float64)
    want = orc.whiten_advantages(a64, mask, role, off, 2, scope)
    assert not out[mask == 0].any()
    assert (np.abs(out - want) <= P.whiten_bounds(a64, mask, role, off, 2, scope == umas.WHITEN_MODEL_ROLE)).all()
