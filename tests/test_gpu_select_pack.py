"""GPU parity of dppo_select and dppo_pack against the CPU oracle: masks, counts and every
packing offset bit-exact; float outputs to float32 rounding."""
import numpy as np
import pytest
import torch

import workloads as WL
from oracle import dppo_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def lib():
    import paper_2603_04135_amd as P
    P.load()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return P


def _cmp_select(P, rewards, hist, up, uc, r_q, r_o, ddof=1, eps=1e-6, bottom=0.5, fixed=False, realised=True):
    ref = O.select(rewards, hist, up, uc, r_q, r_o, ddof=ddof, eps=eps, bottom_frac=bottom, fixed_count=fixed,
                   realised_rate=realised)
    got = P.dppo_select(rewards, hist, up, uc, r_q, r_o, adv_eps=eps, std_ddof=ddof, bottom_frac=bottom,
                        fixed_count=fixed, realised_rate=realised, device=DEV)
    g = {k: v.cpu().numpy() for k, v in got.items()}
    assert np.array_equal(g["keep_prompt"], ref["keep_prompt"])
    assert np.array_equal(g["keep_comp"], ref["keep_comp"])
    assert np.array_equal(g["counts"], ref["counts"])
    for k in ("adv", "mean_abs_adv", "gamma_q", "gamma_o", "coef"):
        assert np.allclose(g[k], ref[k], rtol=2e-6, atol=1e-9), k
    assert np.allclose(g["prune_q"], ref["P_q"], rtol=2e-7, atol=0) and np.allclose(g["prune_o"], ref["P_o"], rtol=2e-7, atol=0)
    return ref, g


@pytest.mark.parametrize("name", list(WL.WORKLOADS))
def test_select_matches_oracle_on_workloads(lib, name):
    rb = WL.make_rollout(name)
    wl = rb.wl
    ref, _ = _cmp_select(lib, rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, wl.r_q, wl.r_o)
    assert 0 < ref["keep_comp"].sum() < wl.Q * wl.G
    # first epoch: no history, prompt pruning skipped
    _cmp_select(lib, rb.rewards, None, None, rb.u_comp, wl.r_q, wl.r_o)
    # no pruning at all recovers plain GRPO weights
    ref, g = _cmp_select(lib, rb.rewards, None, None, None, wl.r_q, wl.r_o)
    assert np.allclose(g["coef"], 1.0 / (wl.Q * wl.G), rtol=1e-6)


def test_select_edge_cases(lib):
    rng = np.random.default_rng(5)
    # balanced and constant binary groups (ties decide the whole candidate set), odd Q, tied history
    for G in (2, 4, 8, 16):
        r = np.zeros((7, G), dtype=np.float32)
        r[0, : G // 2] = 1; r[1, :] = 1; r[3, :1] = 1; r[4, : G - 1] = 1; r[5, ::2] = 1; r[6, : G // 2 + 1] = 1
        hist = np.array([0.2, 0.0, 0.2, 0.0, 0.7, 0.0, 0.2], dtype=np.float32)
        for seed in range(3):
            rr = np.random.default_rng(seed)
            _cmp_select(lib, r, hist, rr.random(7, dtype=np.float32), rr.random((7, G), dtype=np.float32), 0.5, 0.5)
    # G = 1 needs the population std; real-valued rewards; ddof 0; other bottom fractions
    _cmp_select(lib, rng.random((5, 1)).astype(np.float32), None, None, rng.random((5, 1), dtype=np.float32), 0.3, 0.9, ddof=0)
    r = rng.normal(size=(33, 6)).astype(np.float32)
    _cmp_select(lib, r, rng.random(33).astype(np.float32), rng.random(33, dtype=np.float32),
                rng.random((33, 6), dtype=np.float32), 0.7, 0.25, ddof=0, bottom=0.3)
    # uniforms that prune everything that can be pruned (whole groups disappear)
    r = (rng.random((6, 4)) < 0.5).astype(np.float32)
    ref, _ = _cmp_select(lib, r, np.zeros(6, np.float32), np.zeros(6, np.float32), np.zeros((6, 4), np.float32), 0.9, 0.9)
    assert ref["keep_prompt"].sum() == 3


@pytest.mark.parametrize("name", list(WL.WORKLOADS))
def test_fixed_count_select_matches_oracle(lib, name):
    rb = WL.make_rollout(name)
    wl = rb.wl
    for realised in (True, False):
        ref, _ = _cmp_select(lib, rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, wl.r_q, wl.r_o, fixed=True,
                             realised=realised)
    n_b = wl.Q // 2
    assert wl.Q - ref["keep_prompt"].sum() == O.fixed_prune_count(wl.r_q, n_b)
    _cmp_select(lib, rb.rewards, None, None, rb.u_comp, wl.r_q, wl.r_o, fixed=True)
    _cmp_select(lib, rb.rewards, rb.hist, rb.u_prompt, None, wl.r_q, wl.r_o, fixed=True)
    # rates that are not float32-exact, tied uniforms
    u_tied = np.round(rb.u_comp, 1).astype(np.float32)
    for r in (0.9, 0.7, 0.3, 0.0):
        _cmp_select(lib, rb.rewards, rb.hist, np.round(rb.u_prompt, 1).astype(np.float32), u_tied, r, r, fixed=True)


# both sides of the sizes up to which one launch does the selection (512 prompts), groups that do not fill
# a workgroup, a last workgroup with one group
@pytest.mark.parametrize("Q,G", [(1, 1024), (3, 341), (2, 342), (5, 100), (513, 3), (512, 3), (257, 2), (129, 85), (5, 1024), (3, 513)])
@pytest.mark.parametrize("fixed", [False, True])
def test_select_on_both_sides_of_its_sizes(lib, Q, G, fixed):
    rng = np.random.default_rng(Q * 1000 + G)
    r = (rng.random((Q, G)) < rng.random((Q, 1))).astype(np.float32)
    hist = np.round(rng.random(Q), 2).astype(np.float32)
    up, uc = np.round(rng.random(Q), 2).astype(np.float32), np.round(rng.random((Q, G)), 3).astype(np.float32)
    _cmp_select(lib, r, hist, up, uc, 0.5, 0.4, fixed=fixed)
    _cmp_select(lib, rng.normal(size=(Q, G)).astype(np.float32), None, None, uc, 0.5, 0.4, ddof=0, fixed=fixed)


# Results share memory, but each is a tensor of its own: it takes in-place use with gradients, and writing one leaves what
# autograd saved of another as it is.
def test_results_are_tensors_of_their_own(lib):
    rng = np.random.default_rng(4)
    Q, G = 3, 5
    u = lambda *shape: rng.random(shape, dtype=np.float32)
    sel = lib.dppo_select(u(Q, G), u(Q), u(Q), u(Q, G), 0.5, 0.5, device=DEV)
    pk = lib.dppo_pack(rng.integers(1, 9, Q * G), rng.integers(1, 9, Q * G), None, 20, 4, device=DEV)
    for out in (sel, pk):
        names = [k for k, t in out.items() if torch.is_tensor(t)]
        spans = sorted((out[k].data_ptr(), out[k].data_ptr() + out[k].numel() * out[k].element_size()) for k in names)
        assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
        assert all(a % 16 == 0 for a, _ in spans)
        for k in names:
            versions = {j: out[j]._version for j in names if j != k}
            out[k].mul_(1)
            assert versions == {j: out[j]._version for j in names if j != k}, k
    for k in ("adv", "coef", "gamma_o", "prune_o"):
        w = torch.ones(Q, G, device=DEV, requires_grad=True)
        kept = sel[k].clone()
        sel[k].mul_(w)
        sel[k].sum().backward()
        assert torch.equal(w.grad, kept)


def test_history_update_matches_oracle(lib):
    rng = np.random.default_rng(3)
    table = rng.random(1000).astype(np.float32)
    idx = rng.permutation(1000)[:256].astype(np.int32)
    keep = (rng.random(256) < 0.6).astype(np.uint8)
    score = rng.random(256).astype(np.float32)
    ref = O.history_update(table, idx, keep, score)
    t = torch.as_tensor(table.copy(), device=DEV)
    got = lib.dppo_history_update(t, idx, keep, score).cpu().numpy()
    assert np.array_equal(got, ref)
    assert (got != table).sum() == int(keep.sum())
    # a select -> update round trip: the emitted mean |A| becomes the next epoch's score
    rb = WL.make_rollout("small")
    sel = lib.dppo_select(rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, 0.4, 0.5, fixed_count=True, device=DEV)
    t = torch.as_tensor(rb.hist.copy(), device=DEV)
    lib.dppo_history_update(t, np.arange(rb.wl.Q, dtype=np.int32), sel["keep_prompt"], sel["mean_abs_adv"])
    o = O.select(rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, 0.4, 0.5, fixed_count=True)
    want = O.history_update(rb.hist, np.arange(rb.wl.Q), o["keep_prompt"], o["mean_abs_adv"].astype(np.float32))
    assert np.allclose(t.cpu().numpy(), want, rtol=2e-6, atol=1e-9)
    assert np.array_equal(t.cpu().numpy()[o["keep_prompt"] == 0], rb.hist[o["keep_prompt"] == 0])


@pytest.mark.parametrize("name", ["small", "qwen3_4b", "stress"])
def test_variance_terms_match_oracle(lib, name):
    # App. D: g = a stand-in gradient component that is small where |A| is small (the paper's premise)
    rb = WL.make_rollout(name)
    wl = rb.wl
    sel = lib.dppo_select(rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, wl.r_q, wl.r_o, device=DEV)
    adv = sel["adv"].cpu().numpy()
    rng = np.random.default_rng(3)
    for g in ((adv * rng.normal(1.0, 0.3, size=adv.shape)).astype(np.float32),
              rng.normal(size=adv.shape).astype(np.float32)):
        got = lib.dppo_variance_terms(g, sel["prune_q"], sel["prune_o"], device=DEV)
        ref = O.variance_terms(g, sel["prune_q"].cpu().numpy(), sel["prune_o"].cpu().numpy())
        grp, tot = got["group"].cpu().numpy(), got["total"].cpu().numpy()
        scale = float((g.astype(np.float64) ** 2).mean())
        for col, key in enumerate(("G_q", "var_O", "var_o")):
            assert np.allclose(grp[:, col], ref[key], rtol=1e-9, atol=1e-12 * scale), key
        # the 0/1 condition flags may differ only where the two sides of the inequality tie to rounding
        assert (grp[:, 3] != ref["cond_o"]).mean() <= 0.01
        for idx, key in ((0, "G_bar"), (1, "var_Q"), (2, "term1"), (4, "egamma2"), (5, "mean_var_O"), (6, "term2"),
                         (7, "total"), (8, "bound")):
            assert abs(tot[idx] - ref[key]) <= 1e-9 * abs(ref[key]) + 1e-12 * scale, key
        assert tot[3] == float(ref["cond_q"])
    # the closed-form prompt factor of Theorem D.1 with half the prompts candidates
    closed = (1 - 0.5 * wl.r_q) * (1 - 0.5 * wl.r_q) / (1 - wl.r_q)
    assert abs(tot[4] - closed) <= 1e-6 * closed + (0 if wl.Q % 2 == 0 else 0.05)


def test_batch_estimator_is_unbiased_over_sampled_masks(lib):
    # Monte-Carlo over masks with the selection kernel itself: E[sum_i coef_i g_i] = mean g (Eq. 13)
    rb = WL.make_rollout("small")
    wl = rb.wl
    rng = np.random.default_rng(5)
    g = torch.as_tensor(rng.normal(1.0, 1.0, size=rb.rewards.shape).astype(np.float32), device=DEV)
    vals = []
    for _ in range(400):
        up = rng.random(wl.Q, dtype=np.float32)
        uc = rng.random((wl.Q, wl.G), dtype=np.float32)
        sel = lib.dppo_select(rb.rewards, rb.hist, up, uc, wl.r_q, wl.r_o, device=DEV)
        vals.append((sel["coef"].double() * g.double()).sum())
    vals = torch.stack(vals).cpu().numpy()
    se = vals.std() / np.sqrt(len(vals))
    assert abs(vals.mean() - float(g.double().mean())) < 5 * se


def test_maximum_sizes(lib):
    # the largest supported batch of prompts, and a long item stream through the packer
    rng = np.random.default_rng(1)
    Q, G = 16384, 16
    r = (rng.random((Q, G)) < 0.5).astype(np.float32)
    hist = np.round(rng.random(Q), 3).astype(np.float32)
    up, uc = rng.random(Q, dtype=np.float32), rng.random((Q, G), dtype=np.float32)
    for fixed in (False, True):
        ref, _ = _cmp_select(lib, r, hist, up, uc, 0.5, 0.5, fixed=fixed)
    n = 65536
    pl = rng.integers(16, 512, size=n).astype(np.int32)
    cl = rng.integers(16, 2048, size=n).astype(np.int32)
    _cmp_pack(lib, pl, cl, ref["keep_comp"].reshape(-1)[:n], 8192, 32)
    with pytest.raises(lib.DppoError):
        lib.dppo_select(np.zeros((16385, 2), np.float32), None, None, None, 0.5, 0.5, device=DEV)


def test_select_rejects_bad_arguments(lib):
    r = np.zeros((2, 2), dtype=np.float32)
    with pytest.raises(lib.DppoError):
        lib.dppo_select(r, None, None, None, 1.0, 0.5, device=DEV)
    with pytest.raises(lib.DppoError):
        lib.dppo_select(np.zeros((2, 1), np.float32), None, None, None, 0.5, 0.5, std_ddof=1, device=DEV)


def _cmp_pack(P, pl, cl, keep, cap, n_win, policy="first_fit"):
    ref = O.pack(pl, cl, keep, cap, n_win, policy=policy)
    got = P.dppo_pack(pl, cl, keep, cap, n_win, device=DEV, policy=policy)
    assert got["device_status"] == 0
    assert (got["n_rows"], got["T"], got["N"], got["S"]) == (ref["n_rows"], ref["T"], ref["N"], ref["S"])
    assert got["capacity"] == ref["capacity"] and got["density"] == pytest.approx(ref["density"], rel=1e-12)
    for k in ("order", "row_ptr", "cu_seqlens", "loss_cu", "loss_pos"):
        assert np.array_equal(got[k].cpu().numpy(), ref[k]), k
    return ref


@pytest.mark.parametrize("name", list(WL.WORKLOADS))
def test_pack_matches_oracle_on_workloads(lib, name):
    rb = WL.make_rollout(name)
    wl = rb.wl
    keep = O.select(rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, wl.r_q, wl.r_o)["keep_comp"].reshape(-1)
    n = int(keep.sum())
    for n_win in sorted({1, 2, wl.n_win, 64, 65, n, n + 3}):
        ref = _cmp_pack(lib, rb.item_prompt_len, rb.item_comp_len, keep, wl.capacity, n_win)
        if n_win <= 1000:      # the oracle's best-fit scan is quadratic in the pool
            bf = _cmp_pack(lib, rb.item_prompt_len, rb.item_comp_len, keep, wl.capacity, n_win, policy="best_fit")
            assert bf["T"] == ref["T"]
    assert ref["T"] > 0
    _cmp_pack(lib, rb.item_prompt_len, rb.item_comp_len, None, wl.capacity, wl.n_win)


def test_pack_edge_cases(lib):
    rng = np.random.default_rng(17)
    for trial in range(40):
        n = int(rng.integers(1, 300))
        cap = int(rng.integers(4, 200))
        pl = rng.integers(1, cap // 2 + 1, size=n).astype(np.int32)
        cl = rng.integers(1, cap - pl + 1).astype(np.int32)
        if trial % 4 == 0:
            pl[0], cl[0] = 1, cap - 1                       # an item that fills a row exactly
        keep = (rng.random(n) < 0.7).astype(np.uint8) if trial % 2 else None
        if keep is not None and keep.sum() == 0:
            keep[0] = 1
        for n_win in (1, 2, 7, 64, 130, n + 1):
            _cmp_pack(lib, pl, cl, keep, cap, n_win)
            _cmp_pack(lib, pl, cl, keep, cap, n_win, policy="best_fit")
            if trial % 5 == 0:
                _cmp_pack(lib, pl + cl, None, keep, (0, cap)[trial % 2], n_win, policy=("first_fit", "best_fit")[n_win % 2])
    # one-token prompts and completions
    _cmp_pack(lib, np.ones(100, np.int32), np.ones(100, np.int32), None, 7, 5)
    # everything pruned: empty result, no error
    got = lib.dppo_pack(np.array([3, 4], np.int32), np.array([2, 2], np.int32), np.zeros(2, np.uint8), 16, 4, device=DEV)
    assert (got["n_rows"], got["T"], got["N"], got["S"], got["device_status"]) == (0, 0, 0, 0, 0)


@pytest.mark.parametrize("name", list(WL.PROMPT_DATASETS))
def test_pack_whole_prompt_dataset(lib, name):
    # Sec. 4.3 as the paper uses it: prompts alone, the whole dataset as the stream, L_max = longest prompt
    pl = WL.make_prompt_dataset(name)
    dens = {}
    for policy in ("first_fit", "best_fit"):
        for n_win in (1, 64, 256, 1000) + ((len(pl),) if policy == "first_fit" else ()):
            ref = _cmp_pack(lib, pl, None, None, 0, n_win, policy=policy)
            assert ref["capacity"] == int(pl.max()) and ref["N"] == 0
            dens[policy, n_win] = ref["density"]
    # a wider pool never hurts much and the dense packing beats one prompt per slot by far
    assert dens["first_fit", 256] > dens["first_fit", 1] > float(pl.mean()) / float(pl.max())
    assert dens["best_fit", 1000] > 0.95
    # with an explicit capacity and a keep mask
    keep = (np.arange(len(pl)) % 3 != 0).astype(np.uint8)
    _cmp_pack(lib, pl, None, keep, 4096, 128, policy="best_fit")


@pytest.mark.parametrize("n_win", [31, 32, 33, 95, 96, 97])
@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1024, 1025, 15360, 15361])
def test_pack_pool_and_stream_edges(lib, n, n_win):
    """Pools around what one and two registers per lane hold (32, 96) and what falls back to scanning, item counts
    around a wavefront, the workgroup and the stream lengths that fit in LDS (15 360); rows of very many and of few
    items, so that the pool is closed up inside a row and between rows; loss positions written by the packing
    workgroup (capacity up to 16 384) and by the grid-wide kernel. Bit-exact."""
    rng = np.random.default_rng(n * 100 + n_win)
    pl, cl = rng.integers(1, 5, size=n).astype(np.int32), rng.integers(1, 20, size=n).astype(np.int32)
    for cap, policy in ((24, "first_fit"), (900, "first_fit"), (24, "best_fit"), (900, "best_fit")):
        if policy == "first_fit" or n <= 1025:      # the oracle's best-fit scan is quadratic in the pool
            _cmp_pack(lib, pl, cl, None, cap, n_win, policy=policy)


def test_pack_reports_device_detected_errors(lib):
    # item longer than the window
    got = lib.dppo_pack(np.array([3, 9], np.int32), np.array([2, 8], np.int32), None, 16, 4, device=DEV)
    assert got["device_status"] == 1 and got["S"] == 0 and got["T"] == 0
    # empty completion
    got = lib.dppo_pack(np.array([3, 3], np.int32), np.array([2, 0], np.int32), None, 16, 4, device=DEV)
    assert got["device_status"] == 1
    # ... but not if that item is pruned
    got = lib.dppo_pack(np.array([3, 9], np.int32), np.array([2, 8], np.int32), np.array([1, 0], np.uint8), 16, 4, device=DEV)
    assert got["device_status"] == 0 and got["S"] == 1
    # loss_pos buffer too small
    got = lib.dppo_pack(np.array([3, 3], np.int32), np.array([5, 5], np.int32), None, 16, 4, loss_pos_capacity=9, device=DEV)
    assert got["device_status"] == 2
    with pytest.raises(lib.DppoError):
        lib.dppo_pack(np.array([3], np.int32), np.array([2], np.int32), None, 16, 0, device=DEV)
    # prompts alone: a prompt longer than an explicit capacity, an empty prompt
    got = lib.dppo_pack(np.array([3, 9], np.int32), None, None, 8, 4, device=DEV)
    assert got["device_status"] == 1
    got = lib.dppo_pack(np.array([3, 0], np.int32), None, None, 0, 4, device=DEV)
    assert got["device_status"] == 1


def test_gather_puts_weights_in_packed_order(lib):
    rb = WL.make_rollout("small")
    wl = rb.wl
    sel = O.select(rb.rewards, rb.hist, rb.u_prompt, rb.u_comp, wl.r_q, wl.r_o)
    pk = O.pack(rb.item_prompt_len, rb.item_comp_len, sel["keep_comp"].reshape(-1), wl.capacity, wl.n_win)
    coef = torch.as_tensor(sel["coef"].astype(np.float32), device=DEV)
    got = lib.dppo_gather_f32(torch.as_tensor(pk["order"], device=DEV), coef).cpu().numpy()
    assert np.array_equal(got, sel["coef"].astype(np.float32).reshape(-1)[pk["order"]])
