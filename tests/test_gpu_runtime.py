"""Run-time behaviour of the boundary on the GPU: the calls that take host arrays do not wait for the stream, the
pinned staging ring survives back-to-back calls, and results do not depend on scheduling."""
import time

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import umas_oracle as orc
import paper_2605_26646_amd as umas
from tests import parity as P

pytestmark = pytest.mark.gpu

SMALL_BF16 = [(128, 1000, "bf16")]


def assign_kwargs(w, mask):
    return dict(n_roles=w.n_roles, n_models=w.n_models, role_to_model=w.role_to_model, traj_turn_off=w.traj_turn_off,
                turn_role=w.turn_role, turn_tok_off=w.turn_tok_off, tok_mask_global=mask, turn_pred_off=w.turn_pred_off,
                turn_pred=w.turn_pred, traj_group=w.traj_group, role_reward=w.role_reward, turn_reward=w.turn_reward,
                traj_reward=w.traj_reward, place_mode=w.place_mode, norm_eps=w.norm_eps)


def queue_long_work(n_matmuls=60):
    """About 0.4 s of matrix products on the current stream; returns an event recorded behind them."""
    x = torch.randn(16384, 16384, device="cuda", dtype=torch.bfloat16)
    y = x
    for _ in range(n_matmuls):
        y = x @ x
    ev = torch.cuda.Event()
    ev.record()
    return ev, y


def test_calls_with_host_arrays_return_while_earlier_work_is_still_running():
    w = wl.make_workload(2, n_traj=8, tokens_per_turn=48, models=SMALL_BF16)
    rho, st, r, adv_o, ret_o = P.oracle_front(w)
    mask = P.to_dev(w.tok_mask)
    kw = assign_kwargs(w, mask)
    s = umas.umas_assign_token_rewards(**kw)              # first use: the staging memory is allocated here
    umas.umas_ready_batch(s, w.traj_turn_off, 2)
    queue_long_work(2)
    torch.cuda.synchronize()
    ev, _ = queue_long_work()
    t0 = time.perf_counter()
    s = umas.umas_assign_token_rewards(**kw)
    t1 = time.perf_counter()
    still_running_after_assign = not ev.query()
    rows, off = umas.umas_ready_batch(s, w.traj_turn_off, 2)
    t2 = time.perf_counter()
    still_running_after_batch = not ev.query()
    torch.cuda.synchronize()
    assert still_running_after_assign, f"umas_assign_token_rewards returned after {1e3 * (t1 - t0):.1f} ms, when the earlier work had ended"
    assert still_running_after_batch, f"umas_ready_batch returned after {1e3 * (t2 - t1):.1f} ms, when the earlier work had ended"
    assert t2 - t0 < 0.1, f"the two calls took {1e3 * (t2 - t0):.1f} ms of host time"
    adv, ret = umas.umas_advantages(s, P.to_dev(w.value), w.gamma, w.lam, w.gamma_turn, w.seg_mode)
    P.check_front(w, s, adv, ret, rho, st, r, adv_o, ret_o)
    rows_o, off_o = orc.ready_batch(st, w.traj_turn_off, np.ones(w.n_traj, np.uint8), np.arange(w.n_traj), 2)
    assert np.array_equal(off.cpu().numpy(), off_o) and np.array_equal(rows.cpu().numpy()[:len(rows_o)], rows_o)


def test_staging_ring_keeps_every_queued_call_apart():
    """Ten routing calls on ten different graphs queued behind long-running work, none of them waited for: more calls
    than the ring has blocks, sizes going up and down, so blocks are reused and regrown while copies are pending.  The
    caller's host arrays are scribbled over right after each call returns."""
    cases = []
    for k, (cfg, n_traj, L) in enumerate([(2, 6, 40), (0, 3, 16), (4, 4, 64), (1, 16, 24), (3, 5, 32), (2, 30, 56), (0, 1, 8),
                                          (4, 8, 128), (1, 8, 8), (3, 12, 20)]):
        w = wl.make_workload(cfg, n_traj=n_traj, tokens_per_turn=L, seed_offset=k,
                             models=SMALL_BF16 * (2 if cfg == 3 else 1))
        cases.append((w, P.oracle_front(w)))
    s0 = umas.umas_assign_token_rewards(**assign_kwargs(cases[0][0], P.to_dev(cases[0][0].tok_mask)))   # allocate the first block
    torch.cuda.synchronize()
    ev, _ = queue_long_work(30)
    outs = []
    for w, _o in cases:
        kw = assign_kwargs(w, P.to_dev(w.tok_mask))
        host = {k: (None if v is None else np.array(v, copy=True)) for k, v in kw.items() if isinstance(v, np.ndarray) or v is None}
        kw.update(host)
        s = umas.umas_assign_token_rewards(**kw)
        for v in host.values():                            # the call has read them: the caller may reuse its arrays
            if v is not None:
                v[...] = 0
        value = None if w.value is None else P.to_dev(w.value)
        outs.append((s, *umas.umas_advantages(s, value, w.gamma, w.lam, w.gamma_turn, w.seg_mode)))
    torch.cuda.synchronize()
    for (w, (rho, st, r, adv_o, ret_o)), (s, adv, ret) in zip(cases, outs):
        P.check_front(w, s, adv, ret, rho, st, r, adv_o, ret_o)


# thin arrays of about 11 to 340 KB: on both sides of the 16 KB from which a kernel copies them, one to many workgroups of it
@pytest.mark.parametrize("n_traj", [150, 200, 215, 230, 430, 900, 4500])
def test_thin_arrays_of_all_sizes_reach_the_device(n_traj):
    from tests import arraywise as aw
    w = wl.make_workload(1, n_traj=n_traj, tokens_per_turn=8, models=SMALL_BF16)
    s, adv, ret = P.gpu_front(w)
    sa = aw.streams(w)
    for f in ("perm", "tok_turn", "tok_role", "tok_mask", "turn_seg_off", "tok_flags"):
        assert np.array_equal(getattr(s, f).cpu().numpy(), sa[f]), f
    P.close(s.turn_scalar.cpu().numpy(), aw.composed_rewards(w), 1e-5, "turn_scalar")
    rng = np.random.default_rng(n_traj)
    keep, order = (rng.random(n_traj) < 0.9).astype(np.uint8), rng.permutation(n_traj).astype(np.int32)
    rows, off = umas.umas_ready_batch(s, w.traj_turn_off, 4, keep, order)
    rows_a, off_a = aw.ready_batch(w, sa, keep, order, 4, False)
    assert np.array_equal(off.cpu().numpy(), off_a) and np.array_equal(rows.cpu().numpy()[:len(rows_a)], rows_a)


def test_blocks_that_a_kernel_reads_are_used_again():
    """Three rounds over the staging ring with arrays of one size and other contents, behind long-running work: every call's kernel
    reads the pinned block that an earlier call's kernel has read, with what the host has written there since."""
    from tests import arraywise as aw
    cases = [wl.make_workload(1, n_traj=430, tokens_per_turn=8, models=SMALL_BF16, seed_offset=k) for k in range(12)]
    masks = [P.to_dev(w.tok_mask) for w in cases]
    torch.cuda.synchronize()
    queue_long_work(30)
    outs = [umas.umas_assign_token_rewards(**assign_kwargs(w, mask)) for w, mask in zip(cases, masks)]
    torch.cuda.synchronize()
    for w, s in zip(cases, outs):
        sa = aw.streams(w)
        for f in ("perm", "tok_mask", "tok_flags"):
            assert np.array_equal(getattr(s, f).cpu().numpy(), sa[f]), f
        P.close(s.turn_scalar.cpu().numpy(), aw.composed_rewards(w), 1e-5, "turn_scalar")


def test_results_do_not_depend_on_scheduling():
    """Two runs of the whole path on the same inputs: routing, placement, advantages, log-probs, statistics and dH are
    bit-equal (no atomics on their way); dW adds its one-hot rows with float atomics in whatever order the wavefronts
    arrive (its dense part has one writer per entry and a fixed order), so it is equal up to float32 rounding of those
    sums: 1e-4 relative here against the 1e-2 of the gradient bar."""
    w = wl.make_workload(3, n_traj=12, tokens_per_turn=96, models=[(256, 3000, "bf16"), (320, 2100, "bf16")])
    mask = P.to_dev(w.tok_mask)
    runs = []
    for _ in range(2):
        s = umas.umas_assign_token_rewards(**assign_kwargs(w, mask))
        adv, ret = umas.umas_advantages(s, P.to_dev(w.value), w.gamma, w.lam, w.gamma_turn, w.seg_mode)
        per_model = []
        off = s.model_tok_off.cpu().numpy()
        roff = s.model_rowsel_off.cpu().numpy()
        for m in range(w.n_models):
            t = w.model_tensors(m)
            a, e = int(off[m]), int(off[m + 1])
            H, W, ids = P.to_dev(t["H"], torch.bfloat16), P.to_dev(t["W"], torch.bfloat16), P.to_dev(t["ids"])
            rowsel = s.rowsel[int(roff[m]):int(roff[m + 1])]
            logp, lse, ent = umas.umas_policy_logprobs(H, W, ids, rowsel)
            logp_old = logp + P.to_dev(t["noise"].astype(np.float32))
            stats, logp_new, dH, dW = umas.umas_ppo_loss_fwd_bwd(H, W, ids, rowsel, logp_old, adv[a:e].contiguous(),
                                                                s.tok_role[a:e].contiguous(), w.n_roles, w.clip_eps)
            torch.cuda.synchronize()
            per_model.append((logp, lse, ent, stats, logp_new, dH, dW))
        runs.append((s, adv, ret, per_model))
    (s1, adv1, ret1, pm1), (s2, adv2, ret2, pm2) = runs
    for f in ("model_tok_off", "perm", "tok_turn", "tok_role", "tok_mask", "tok_flags", "tok_reward", "turn_seg_off", "seg_turn",
              "model_turn_off", "traj_seg_off", "model_trajrun_off", "model_rowsel_off", "turn_scalar", "turn_step"):
        assert torch.equal(getattr(s1, f), getattr(s2, f)), f
    n_scored = int(s1.model_rowsel_off[-1].item())
    assert torch.equal(s1.rowsel[:n_scored], s2.rowsel[:n_scored])
    assert torch.equal(adv1, adv2) and torch.equal(ret1, ret2)
    for a, b in zip(pm1, pm2):
        for k, name in enumerate(("logp", "lse", "entropy", "stats", "logp_new", "dH")):
            assert torch.equal(a[k], b[k]), name
        dW1, dW2 = a[6], b[6]
        # a frequent token's row of dW is a float32 sum of hundreds of one-hot terms in arrival order: up to about
        # sqrt(terms) 2^-24 of their magnitudes apart between runs, two orders of magnitude inside the gradient bar
        P.close(dW2.cpu().numpy(), dW1.cpu().numpy().astype(np.float64), 1e-4, "dW of the second run against the first")


def test_binding_refuses_a_row_selection_out_of_range():
    """Row selections are device data the library cannot check; the binding's optional check (on for the tests)
    reads the range back and raises before anything is launched."""
    from paper_2605_26646_amd import binding
    assert binding.CHECK_ROWS
    H = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((300, 64), dtype=torch.bfloat16, device="cuda")
    ids = torch.zeros(8, dtype=torch.int32, device="cuda")
    z = torch.zeros(8, device="cuda")
    for bad in ([0, 3, 8], [-1, 2]):
        sel = torch.tensor(bad, dtype=torch.int32, device="cuda")
        with pytest.raises(umas.UmasError, match="outside"):
            umas.umas_policy_logprobs(H, W, ids, sel)
        with pytest.raises(umas.UmasError, match="outside"):
            umas.umas_ppo_loss_fwd_bwd(H, W, ids, sel, z, z, None, 0, 0.2)
        with pytest.raises(umas.UmasError, match="outside"):
            umas.umas_values(H, torch.ones(64, dtype=torch.bfloat16, device="cuda"), 0.0, sel)
        with pytest.raises(umas.UmasError, match="outside"):
            umas.umas_value_loss_fwd_bwd(H, torch.ones(64, dtype=torch.bfloat16, device="cuda"), 0.0, sel, z, z, None, 0, 0.2)


@pytest.mark.parametrize("form", [
    lambda a: None if a is None else np.asarray(a).tolist(),                                             # lists
    lambda a: None if a is None else np.asarray(a).astype(np.float64 if np.asarray(a).dtype.kind == "f" else np.int64),   # other types
    lambda a: None if a is None else np.repeat(np.asarray(a), 2)[::2],                                   # not contiguous
    lambda a: None if a is None else np.asarray(a).astype(np.asarray(a).dtype.newbyteorder(">")),         # the other byte order
    lambda a: None if a is None else torch.from_numpy(np.array(a)),                                      # tensors on the host
])
def test_host_arrays_in_any_form_give_the_same(form):
    w = wl.make_workload(2, n_traj=9, tokens_per_turn=48, models=SMALL_BF16)
    kw = assign_kwargs(w, P.to_dev(w.tok_mask))
    arrays = [k for k, v in kw.items() if v is not None and k not in ("n_roles", "n_models", "tok_mask_global", "place_mode", "norm_eps")]
    a, b = umas.umas_assign_token_rewards(**kw), umas.umas_assign_token_rewards(**{**kw, **{k: form(kw[k]) for k in arrays}})
    keep, order = np.arange(9) % 3 != 1, np.random.default_rng(1).permutation(9).astype(np.int32)
    for cut in (lambda s, f: umas.umas_ready_batch(s, f(w.traj_turn_off), 3, f(keep.astype(np.uint8)), f(order)),
                lambda s, f: umas.umas_ready_batch_packed(s, f(w.traj_turn_off), 40, f(keep.astype(np.uint8)), f(order))):
        kept = int(cut(a, np.asarray)[1].max())
        for x, y in zip(cut(a, np.asarray), cut(b, form)):
            assert torch.equal(x[:kept] if x.dim() == 1 else x, y[:kept] if y.dim() == 1 else y)
    for name, x in vars(a).items():
        y = getattr(b, name)
        assert torch.equal(x, y) if torch.is_tensor(x) and name != "rowsel" else torch.is_tensor(x) or x == y, name
    n = int(a.model_rowsel_off[-1])
    assert torch.equal(a.rowsel[:n], b.rowsel[:n])


def test_arguments_of_other_types_are_refused():
    w = wl.make_workload(2, n_traj=3, tokens_per_turn=48, models=SMALL_BF16)
    kw = assign_kwargs(w, P.to_dev(w.tok_mask))
    H, x = torch.zeros(4, 64, device="cuda", dtype=torch.float16), torch.zeros(4, device="cuda")
    for call in (lambda: umas.umas_assign_token_rewards(**{**kw, "n_roles": 2.0}), lambda: umas.umas_assign_token_rewards(**{**kw, "norm_eps": None}),
                 lambda: umas.umas_assign_token_rewards(**{**kw, "tok_mask_global": w.tok_mask.tolist()}),
                 lambda: umas.umas_values(H, x), lambda: umas.umas_policy_logprobs(H, H, x), lambda: umas.umas_kl_rewards(x, x, None, x, 0.1)):
        with pytest.raises((TypeError, AttributeError)):
            call()
    with pytest.raises(umas.UmasError):
        umas.umas_assign_token_rewards(**{**kw, "traj_turn_off": None})


def test_two_pipelines_on_two_streams_at_once():
    """Routing, the scan and the ready batch have kernels whose workgroups wait for words that their other workgroups
    publish; their grids are a fraction of what the device holds, so two such pipelines on different streams (disjoint
    outputs and workspaces) run side by side.  Both must give what they give alone."""
    ws = [wl.make_workload(1, n_traj=20000, tokens_per_turn=64), wl.make_workload(4, n_traj=200, tokens_per_turn=8192)]      # trajectory runs of up to 30 720 tokens: cut inside
    masks = [P.to_dev(w.tok_mask) for w in ws]
    values = [None if w.value is None else P.to_dev(w.value) for w in ws]
    rngs = [np.random.default_rng(50 + i) for i in range(2)]
    orders = [r.permutation(w.n_traj).astype(np.int32) for r, w in zip(rngs, ws)]
    keeps = [(r.random(w.n_traj) < 0.9).astype(np.uint8) for r, w in zip(rngs, ws)]

    def pipeline(i):
        w = ws[i]
        s = umas.umas_assign_token_rewards(**assign_kwargs(w, masks[i]))
        adv, ret = umas.umas_advantages(s, values[i], w.gamma, w.lam, 0.97, wl.SEG_TRAJ)
        rows, off = umas.umas_ready_batch(s, w.traj_turn_off, 8, keeps[i], orders[i])
        return s, adv, ret, rows, off

    alone = [pipeline(0), pipeline(1)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]        # default priority
    got = [None, None]
    for rep in range(6):                                         # interleaved issue: the two pipelines overlap on the device
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                got[i] = pipeline(i)
    torch.cuda.synchronize()
    for i in range(2):
        (s0, a0, r0, rows0, off0), (s1, a1, r1, rows1, off1) = alone[i], got[i]
        n_scored = int(s0.model_rowsel_off[-1].item())
        for f in ("perm", "tok_turn", "tok_flags", "tok_reward", "turn_seg_off", "model_rowsel_off"):
            assert torch.equal(getattr(s0, f), getattr(s1, f)), f
        assert torch.equal(s0.rowsel[:n_scored], s1.rowsel[:n_scored])
        assert torch.equal(a0, a1) and torch.equal(r0, r1)
        assert torch.equal(off0, off1)
        n_kept = int(off0[-1, -1].item())
        assert torch.equal(rows0[:n_kept], rows1[:n_kept])


def test_every_output_has_memory_of_its_own():
    """One that is resized, freed or written to a file is that and no more."""
    w = wl.make_workload(2, n_traj=8, tokens_per_turn=48, models=SMALL_BF16)
    s = umas.umas_assign_token_rewards(**assign_kwargs(w, P.to_dev(w.tok_mask)))
    streams = [t for t in vars(s).values() if isinstance(t, torch.Tensor)]
    assert len(streams) == 16
    adv, ret = umas.umas_advantages(s, P.to_dev(w.value), w.gamma, w.lam)
    logp = torch.zeros_like(adv)
    out, kl = umas.umas_kl_rewards(s.tok_reward, logp, logp, s.tok_mask, 0.05)
    rows, off, parts = umas.umas_ready_batch_packed(s, w.traj_turn_off, 100)
    outputs = streams + [adv, ret, out, kl, rows, off, parts]
    for t in outputs:
        assert t.storage_offset() == 0 and t.untyped_storage().nbytes() == t.numel() * t.element_size()
    before = [t.clone() for t in outputs]
    for t in outputs:
        t.resize_(t.numel() + 5000).fill_(1)
    for t, b in zip(outputs, before):
        t.copy_(torch.cat([b.flatten(), torch.ones(5000, dtype=b.dtype, device="cuda")]))
    assert all(torch.equal(t[:b.numel()], b.flatten()) and (t[b.numel():] == 1).all() for t, b in zip(outputs, before))


def test_calls_with_host_arrays_are_not_recorded():
    """A graph would read the staging block again after later calls have overwritten it: refused, and the ring stays as it was."""
    w = wl.make_workload(2, n_traj=8, tokens_per_turn=48, models=SMALL_BF16)
    front = P.oracle_front(w)
    kw = assign_kwargs(w, P.to_dev(w.tok_mask))
    s = umas.umas_assign_token_rewards(**kw)
    rows, off = umas.umas_ready_batch(s, w.traj_turn_off, 2)
    graph, x = torch.cuda.CUDAGraph(), torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        for _ in range(5):                               # more than the ring has blocks
            with pytest.raises(Exception, match="cannot be recorded"):
                umas.umas_assign_token_rewards(**kw)
            with pytest.raises(Exception, match="cannot be recorded"):
                umas.umas_ready_batch(s, w.traj_turn_off, 2)
        x += 1                                           # the capture itself goes on
    for k in range(3):
        graph.replay()
        for _ in range(5):
            s2 = umas.umas_assign_token_rewards(**kw)
            rows2, off2 = umas.umas_ready_batch(s2, w.traj_turn_off, 2)
        torch.cuda.synchronize()
        assert float(x) == k + 1 and torch.equal(off, off2) and torch.equal(rows[:int(off[-1, -1])], rows2[:int(off[-1, -1])])
    adv, ret = umas.umas_advantages(s2, P.to_dev(w.value), w.gamma, w.lam, w.gamma_turn, w.seg_mode)
    P.check_front(w, s2, adv, ret, *front)
