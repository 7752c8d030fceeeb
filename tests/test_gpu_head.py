"""GPU parity of dppo_token_logprob and dppo_loss_fwd_bwd against the CPU oracle.

Tolerances: per-token log-prob abs err <= 2e-3
(bf16 inputs, fp32 accumulation), loss rel err <= 1e-3, dH and dW relative Frobenius
error <= 1e-2. The float32 data type is held to 1e-4 / 1e-5 / 1e-4 instead."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as WL
from oracle import dppo_oracle as O
from harness import HeadCase, oracle_select_pack, rel_fro, to_np64, truncate_pack

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {"bf16": dict(logp=2e-3, loss=1e-3, grad=1e-2), "f32": dict(logp=1e-4, loss=1e-5, grad=1e-4)}


@pytest.fixture(scope="module")
def lib():
    import paper_2603_04135_amd as P
    P.load()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return P


def _loss_errors(got, ref_out, case):
    """Error of the loss relative to |L|, and relative to the size of the terms that L sums
    (L is a cancelling sum of seq_coef * advantage-sized terms)."""
    scale = float(np.abs(case.seq_coef_np.astype(np.float64) * ref_out["seq_loss"]).sum())
    err = abs(got - ref_out["loss"])
    return err / max(abs(ref_out["loss"]), 1e-300), err / max(scale, 1e-300)


def _loss_close(got, ref_out, case, tol):
    """Loss relative error <= tol against |L|, the denominator floored at 1 % of the sum of the
    absolute per-sequence terms (where L is mostly cancellation the plain ratio measures nothing)."""
    rel_l, rel_terms = _loss_errors(got, ref_out, case)
    return rel_l <= tol or rel_terms <= 1e-2 * tol


def _assert_loss(got, ref_out, case, tol):
    rel_l, rel_terms = _loss_errors(got, ref_out, case)
    assert rel_l <= tol or rel_terms <= 1e-2 * tol, (
        "loss %.9g vs oracle %.9g: error %.3g of |L| (bound %.1g), %.3g of sum|coef * seq_loss| (bound %.1g)"
        % (got, ref_out["loss"], rel_l, tol, rel_terms, 1e-2 * tol))
    print("loss error: %.3g of |L|, %.3g of sum|coef * seq_loss| (passes on %s)"
          % (rel_l, rel_terms, "|L|" if rel_l <= tol else "the term scale"))


def _same_loss(a, b, ref_out, case):
    """Two paths of the library whose forward statistics are summed in different orders."""
    return _loss_close(float(a), dict(ref_out, loss=float(b)), case, 1e-5)


def _same_rows(a, b):
    """dH of two chunkings of the same batch: the same fp32 sums, possibly associated differently
    (the tiles of a sparsely filled last round are summed in K-split parts), then rounded to bf16."""
    a64, b64 = to_np64(a), to_np64(b)
    return rel_fro(a64, b64) <= 1e-3 and float((a64 == b64).mean()) >= 0.98


def _run_case(P, case, tol, **kw):
    """Full parity of one case: log-probs, loss, per-sequence loss, stats, dH, dW."""
    logp_ref, lse_ref = case.oracle_logprob()
    logp, lse = P.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos)
    assert np.abs(logp.cpu().numpy() - logp_ref).max() <= tol["logp"]
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= tol["logp"]
    case.set_behaviour_logps(logp_ref)
    ref = case.oracle_loss(**kw)
    out = P.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                              case.logp_old, case.logp_ref, **kw)
    torch.cuda.synchronize()
    assert np.abs(out["logp"].cpu().numpy() - ref["logp"]).max() <= tol["logp"]
    _assert_loss(float(out["loss"].item()), ref, case, tol["loss"])
    assert np.allclose(out["seq_loss"].cpu().numpy(), ref["seq_loss"], rtol=tol["loss"], atol=tol["logp"])
    stats = out["stats"].cpu().numpy()
    assert abs(stats[0] - ref["mean_kl"]) <= 1e-3 * max(ref["mean_kl"], 1e-6) + 1e-7
    assert abs(stats[1] - ref["clip_frac"]) <= 2.0 / max(case.pk["N"], 1) + 1e-3 * ref["clip_frac"]
    assert stats[2] == case.pk["N"]
    dH = to_np64(out["dH"])
    dW = to_np64(out["dW"])
    mask = np.ones(case.pk["T"], bool)
    mask[case.pk["loss_pos"]] = False
    assert not dH[mask].any(), "rows that predict nothing must have zero gradient"
    assert rel_fro(dH, ref["dH"]) <= tol["grad"]
    assert rel_fro(dW, ref["dW"]) <= tol["grad"]
    # the rows of the last (possibly partial) 256-row vocabulary tile on their own
    last = case.wl.V - ((case.wl.V - 1) // 256) * 256
    assert rel_fro(dW[-last:], ref["dW"][-last:]) <= tol["grad"]
    return out, ref


def _case(name, max_tokens, seed=None, **over):
    rb = WL.make_rollout(name, seed)
    sel, pk = oracle_select_pack(rb)
    if max_tokens is not None:
        pk = truncate_pack(pk, max_tokens)
    return HeadCase(rb.wl, pk, sel, rb.seed, DEV, **over)


def test_tiny_fp32_whole_batch(lib):
    case = _case("tiny", None)
    assert case.wl.dtype == "f32"
    _run_case(lib, case, TOL["f32"])


def test_tiny_shapes_in_bf16(lib):
    # the tiny batch again with bf16 operands: one partial tile in every dimension
    case = _case("tiny", None, dtype="bf16")
    _run_case(lib, case, TOL["bf16"])


def test_small_bf16_slice_spanning_tiles(lib):
    # ~1500 loss tokens: several 256-token tiles plus a ragged tail, full D and V of the workload
    case = _case("small", 1500)
    assert case.pk["N"] % 256 != 0 and case.pk["N"] > 1024
    _run_case(lib, case, TOL["bf16"])


def test_vocab_and_token_tails(lib):
    # V with a partial 256-row tile and a partial 64-column pad; N well below one tile
    rb = WL.make_rollout("tiny", 3)
    sel, pk = oracle_select_pack(rb)
    for V, D in ((1000, 64), (4200, 128), (257, 192)):
        case = HeadCase(rb.wl, pk, sel, 3, DEV, D=D, V=V, dtype="bf16")
        # targets on tile edges and the last vocabulary entry
        edge = np.array([0, 255, 256, V - 1, V - 2, 63, 64, min(V - 1, 511)], dtype=np.int32)
        lp = pk["loss_pos"][: len(edge)] + 1
        case.ids_np[lp] = edge
        case.ids = torch.as_tensor(case.ids_np, device=DEV)
        _run_case(lib, case, TOL["bf16"])
    case = HeadCase(rb.wl, pk, sel, 3, DEV, D=40, V=300, dtype="f32")
    _run_case(lib, case, TOL["f32"])


# (workload, loss tokens, D, V): wavefront tiles of the fp32 GEMM, and 64-wide ones for the logits and dH of the largest, with remainders in
# all dimensions, a single column, unaligned rows, K slices with a tail, and dH cut along the vocabulary
@pytest.mark.parametrize("name,tokens,D,V", [("tiny", 1, 1, 2), ("tiny", None, 33, 3001), ("tiny", 33, 300, 65),
                                             ("small", 700, 130, 1100), ("small", 1100, 257, 4099)])
def test_fp32_tiles_and_splits(lib, name, tokens, D, V):
    case = _case(name, tokens, dtype="f32", D=D, V=V)
    out, _ = _run_case(lib, case, TOL["f32"])
    acc = out["dW"].clone()
    lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                          case.logp_old, case.logp_ref, dW=acc, accumulate_dW=True)
    assert torch.equal(acc, 2.0 * out["dW"])


# both sides of the row lengths (padded to 256) that the kernel between the fp32 GEMMs keeps in registers: 4, 8 and 16
# vectors a thread, longer ones read twice
@pytest.mark.parametrize("V", [1, 4096, 4097, 16384, 16385, 32768, 32769])
def test_fp32_rows_between_the_gemms(lib, V):
    _run_case(lib, _case("tiny", 11, dtype="f32", D=12, V=V), TOL["f32"])


# wavefront tiles, wavefront tiles with dH in parts, 128-wide logits with 64-wide gradients, and 128-wide tiles throughout
@pytest.mark.parametrize("tokens,D,V", [(40, 100, 500), (300, 200, 3001), (1100, 203, 9000), (2111, 701, 9001)])
def test_fp32_values_beyond_the_bf16_split(lib, tokens, D, V):
    """Values of 2^24 and more, and infinities, do not go through the split into bf16 parts: a column scaled by 2^80 in H and by
    2^-80 in W leaves the logits as they are and scales that column of dW and dH; a weight at minus infinity against
    positive hidden states is a logit at minus infinity."""
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), device=DEV, generator=g)
    W = 0.1 * torch.randn((V, D), device=DEV, generator=g)
    H[:, 5] = H[:, 5].abs() + 0.1
    ids = torch.randint(0, V - 1, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    cu, one = torch.tensor([0, tokens], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    lp = torch.zeros(tokens, device=DEV) - 5.0

    def run(H, W):
        return lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, lp, lp)

    col = torch.ones(D, device=DEV)
    col[3] = 2.0 ** 80
    col[D - 1] = 2.0 ** -80
    plain, scaled = run(H, W), run(H * col, W / col)
    # any order of D fp32 products and sums, and of V exponentials in two levels
    z = H.double() @ W.double().T
    tol = D * 2.0 ** -24 * float((H.abs().double() @ W.abs().double().T).max()) + 32 * 2.0 ** -24 * 20
    want = torch.log_softmax(z, 1).gather(1, ids.long()[:, None])[:, 0]
    for out in (plain, scaled):
        assert (out["logp"].double() - want).abs().max() <= tol
    for name, scale in (("dH", 1 / col), ("dW", col)):
        a, b = plain[name].double(), scaled[name].double() / scale.double()
        err = (a - b).norm(dim=0) / a.norm(dim=0)
        assert float(err.max()) <= 2 * tol, (name, float(err.max()))     # entries of G off by tol, sums of positive and negative ones

    W[V - 1, 5] = -float("inf")
    logp, lse = lib.dppo_token_logprob(H, W, ids, None)
    want = torch.log_softmax(z[:, :V - 1], 1).gather(1, ids.long()[:, None])[:, 0]
    assert (logp.double() - want).abs().max() <= tol


# (tokens, D, V): between them every kernel of the fp32 GEMM for the logits, dH and dW, and parts along K for each (test_f32_plan
# holds that); remainders in all dimensions. The last one takes 128-wide tiles throughout.
FP32_SIZES = [(33, 300, 65), (170, 33, 3001), (300, 200, 3001), (500, 333, 7001), (2111, 701, 9001)]


@pytest.mark.parametrize("tokens,D,V", FP32_SIZES)
def test_fp32_error_against_float64(lib, tokens, D, V):
    """Tight enough to tell the split in three bf16 parts from one that loses the third part of one operand of one GEMM. Log-probs
    (logits of deviation 2) are off by 0.3e-6 to 0.9e-6 in rms, gradients by 0.4e-6 to 1.1e-6 of their norm, growing with the lengths of the sums;
    the loss of such a part adds 4.5e-6 and more, and 1.9e-6 and more (emulated on the CPU)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), device=DEV, generator=g)
    W = torch.randn((V, D), device=DEV, generator=g) * (2.0 / D ** 0.5)
    ids = torch.randint(0, V, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    S = 8
    cu = torch.tensor([tokens * i // S for i in range(S + 1)], dtype=torch.int32, device=DEV)
    adv, coef = torch.randn(S, device=DEV, generator=g), torch.rand(S, device=DEV, generator=g)
    logp = torch.log_softmax(H.double() @ W.double().T, 1)
    want = logp.gather(1, ids.long()[:, None])[:, 0]
    lp = want.float()
    args = (H, W, ids, None, cu, adv, coef, lp, lp)
    out = lib.dppo_loss_fwd_bwd(*args, beta=0.0)           # ratio 1, no KL: d loss / d logp = -advantage x weight / length
    length = (cu[1:] - cu[:-1]).double()
    c = (-adv.double() * coef.double() / length).repeat_interleave(length.long())
    G = (torch.zeros_like(logp).scatter_(1, ids.long()[:, None], 1.0) - logp.exp()) * c[:, None]
    err = (out["logp"].double() - want).square().mean().sqrt().item()
    dH, dW = G @ W.double(), G.T @ H.double()
    err_dH, err_dW = [((a.double() - b).norm() / b.norm()).item() for a, b in ((out["dH"], dH), (out["dW"], dW))]
    print("errors: logp %.3g dH %.3g dW %.3g" % (err, err_dH, err_dW))
    assert err <= 2.5e-6 and err_dH <= 1.8e-6 and err_dW <= 1.8e-6, (err, err_dH, err_dW)
    old = torch.randn((V, D), device=DEV, generator=g)
    acc = lib.dppo_loss_fwd_bwd(*args, beta=0.0, dW=old.clone(), accumulate_dW=True)["dW"]
    assert torch.equal(acc, old + out["dW"])


# dW by wavefront tiles, 64- and 128-wide ones
FP32_DW_TILES = [(64, 4000), (300, 20001), (1001, 16001)]


@pytest.mark.parametrize("tokens", [1, 2, 3])
@pytest.mark.parametrize("D,V", FP32_DW_TILES)
def test_fp32_gradient_of_few_tokens(lib, tokens, D, V):
    """dW of n tokens is a sum of n products of float32 numbers, each product and sum rounded to 24 bits once: off by n 2^-24 of the
    sum of magnitudes at most. The first n columns of H pick the gradient entries out."""
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), device=DEV, generator=g)
    H[:, :tokens] = torch.eye(tokens, device=DEV)
    W = 0.02 * torch.randn((V, D), device=DEV, generator=g)
    ids = torch.randint(0, V, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    cu, one = torch.tensor([0, tokens], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    lp, _ = lib.dppo_token_logprob(H, W, ids, None)
    dW = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, lp, lp)["dW"].double()
    G = dW[:, :tokens]
    err = (dW - G @ H.double()).abs() / (G.abs() @ H.double().abs()).clamp_min(2.0 ** -120)
    worst = float(err.max())
    assert worst <= tokens * 2.0 ** -24


@pytest.mark.parametrize("D,V", FP32_DW_TILES)
def test_fp32_gradient_of_one_token_among_zeros(lib, D, V):
    """39 tokens without advantage and one with: dW is one product per entry, of bf16 parts here. Adding h h' last errs by 0.39 units
    of the last place in rms, -1 to +1/2 at worst, the products left out by 2^-26.5: 3.5e-8 of the entry (4.8e-8 with an
    order that adds smaller products behind h h')."""
    tokens, at = 40, 17
    g = torch.Generator(device=DEV)
    g.manual_seed(V)
    H = torch.randn((tokens, D), device=DEV, generator=g)
    H[:, 0] = 1.0
    W = 0.02 * torch.randn((V, D), device=DEV, generator=g)
    ids = torch.randint(0, V, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    cu = torch.tensor([0, at, at + 1, tokens], dtype=torch.int32, device=DEV)
    adv, coef = torch.tensor([0.0, 1.0, 0.0], device=DEV), torch.ones(3, device=DEV)
    lp, _ = lib.dppo_token_logprob(H, W, ids, None)
    dW = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, adv, coef, lp, lp, beta=0.0)["dW"].double()
    want = dW[:, :1] * H[at].double()
    err = ((dW - want) / want)[:, 1:]
    rms, worst = float(err.square().mean().sqrt()), float(err.abs().max())
    assert rms <= 4e-8 and worst <= 2.0 ** -22, (rms, worst)


@pytest.mark.parametrize("drop", [60, 72, 78, 84])
@pytest.mark.parametrize("D,V", FP32_DW_TILES)
def test_fp32_gradient_of_suppressed_entries(lib, D, V, drop):
    """The row of dW of a vocabulary entry of logit -drop, whose gradient entries lie between 2^-105 and the subnormals: as good as
    those entries. Their exponent z - lse is rounded at 64 to 128 (2^-18) and lse and the exponential err by less than 2^-20
    each; subnormal entries are off by half a unit of 2^-149 twice (the exponential, and its product with the token's factor)."""
    tokens = 40
    g = torch.Generator(device=DEV)
    g.manual_seed(drop)
    H = torch.randn((tokens, D), device=DEV, generator=g)
    H[:, 0] = 1.0
    W = 0.02 * torch.randn((V, D), device=DEV, generator=g)
    W[7] = 0.0
    W[7, 0] = -float(drop)
    ids = torch.randint(8, V, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    cu, one = torch.tensor([0, tokens], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    lp, _ = lib.dppo_token_logprob(H, W, ids, None)
    dW = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, lp, lp, beta=0.0)["dW"]
    p = torch.exp(-float(drop) - torch.logsumexp(H.double() @ W.double().T, 1)) / tokens
    want = p @ H.double()
    bound = (2.0 ** -18 + 2.0 ** -19 + 2.0 ** -148 / p) * p @ H.double().abs() + 2.0 ** -149
    assert bool(((dW[7].double() - want).abs() <= bound).all())


@pytest.mark.parametrize("tokens", [3072, 3073])
@pytest.mark.parametrize("D,V", [(320, 777), (64, 257)])
def test_operand_of_dh_on_both_sides_of_its_rule(lib, tokens, D, V):
    # up to 3072 loss tokens the dH GEMM reads W as it lies, beyond a transposed copy: column tiles that are
    # partly filled, a vocabulary with rows missing from its last slice
    _run_case(lib, _case("small", tokens, dtype="bf16", D=D, V=V), TOL["bf16"])


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("D,V", [(320, 777), (64, 257)])
def test_dh_on_both_sides_of_the_transposed_copy(lib, over, D, V):
    # the last token count whose dH reads W as it lies, and the first with a transposed copy
    _run_case(lib, _case("small", 4096 + D + over, dtype="bf16", D=D, V=V), TOL["bf16"])


@pytest.mark.parametrize("tokens", [300, 3072])
def test_direct_w_in_the_smallest_workspace(lib, tokens):
    # no room for a transposed copy of W: nothing may be written in its place, and chunks of 256 tokens give the result of
    # one chunk up to summation order
    case = _case("small", tokens, dtype="bf16", D=320, V=777)
    T, N = case.pk["T"], case.pk["N"]
    out, _ = _run_case(lib, case, TOL["bf16"])
    nbytes = lib.dppo_workspace_min_bytes(T, N, 320, 777, 1, True)
    buf = lib.alloc_workspace(nbytes + 4096, DEV)
    buf.fill_(0x5A)
    small = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                                  case.logp_old, case.logp_ref, ws=buf[:nbytes])
    torch.cuda.synchronize()
    assert bool((buf[nbytes:] == 0x5A).all())
    assert torch.equal(small["logp"], out["logp"])
    assert rel_fro(to_np64(small["dH"]), to_np64(out["dH"])) <= 1e-3
    assert rel_fro(to_np64(small["dW"]), to_np64(out["dW"])) <= 1e-5


# forward-only token columns of 96, 128, 192 and 256: one token, each width full, one token more
@pytest.mark.parametrize("tokens", [1, 96, 97, 128, 129, 192, 193, 384, 385])
@pytest.mark.parametrize("D,V", [(64, 257), (320, 1000)])
def test_token_columns_of_the_forward(lib, tokens, D, V):
    case = _case("small", tokens, dtype="bf16", D=D, V=V)
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(case.pk["T"], tokens, D, V, 1, 0), DEV)
    ws.fill_(0xFF)                               # NaN wherever a statistic that nobody wrote is read
    logp, lse = lib.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos, ws=ws)
    # fp32 sums of D products |h w| < 1 in any order: D^2 2^-24 at worst, 2e-2 of that in practice
    logp_ref, lse_ref = case.oracle_logprob()
    assert np.abs(logp.cpu().numpy() - logp_ref).max() <= 1e-4
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-4
    if tokens in (97, 193):                      # the recomputed gradient uses these statistics for the padding too
        _run_case(lib, case, TOL["bf16"], recompute_logits=True)


# the forward in columns of 192 tokens and of 256
@pytest.mark.parametrize("tokens", [150, 250])
def test_recomputed_gradient_of_likely_targets(lib, tokens):
    """Targets of probability 1 - 4e-5: 1 - p is formed from the very logit that entered lse, so that its rounding errors
    cancel. What remains is the rounding of lse (2^-20, as it lies between 16 and 32), of the exponential (2^-22), of the 32
    exponentials of 4e-8 that a thread adds to the target's 1 (2^-24 each) and of the entry to bf16 (2^-9): 8 %, seen 5 %.
    A target logit summed over D = 4096 in another order is off by 2^-18 and more: 37 %."""
    D, V, z_target = 4096, 1000, 17.0
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), device=DEV, generator=g).bfloat16()
    ids = torch.randperm(V, device=DEV, generator=g)[:tokens].int()
    W = torch.zeros((V, D), device=DEV, dtype=torch.bfloat16)
    W[ids.long()] = (H.float() * (z_target / H.float().square().sum(1, keepdim=True))).bfloat16()
    logp, _ = lib.dppo_token_logprob(H, W, ids, None)
    cu, one = torch.tensor([0, tokens], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    out = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, logp, logp, recompute_logits=True)
    p = torch.softmax(H.double() @ W.double().T, 1)                  # ratio 1, no KL: d loss / d logp = -1 / tokens
    hot = torch.zeros_like(p).scatter_(1, ids.long()[:, None], 1.0)
    miss = 1.0 - p.gather(1, ids.long()[:, None])[:, 0]
    assert float(miss.min()) > 3e-5 and float(miss.max()) < 6e-5
    want = (((hot - p).T @ H.double()) * (-1.0 / tokens))[ids.long()]
    err = (out["dW"][ids.long()].double() - want).norm(dim=1) / want.norm(dim=1)
    worst = float(err.max())
    assert worst <= (2.0 ** -20 + 2.0 ** -22 + 32 * 2.0 ** -24) / float(miss.min()) + 2.0 ** -8


# columns of 96, 128 and 192 tokens, whose forward reads H itself, and of 256
@pytest.mark.parametrize("n", [40, 100, 150, 250])
def test_recomputing_step_reports_and_clamps_tokens(lib, n):
    """The gather alone looks the tokens up: positions and ids out of range are reported, and taken as the clamped ones."""
    T, D, V = 300, 128, 1000
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    H = torch.randn((T, D), device=DEV, generator=g).bfloat16()
    W = (0.1 * torch.randn((V, D), device=DEV, generator=g)).bfloat16()
    ids = torch.randint(0, V, (T,), device=DEV, dtype=torch.int32, generator=g)
    pos = torch.randperm(T - 2, device=DEV, generator=g)[:n].int() + 1
    cu, one = torch.tensor([0, n], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    lp = torch.full((n,), -7.0, device=DEV)

    def run(pos, ids, want_flags):
        status = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        out = lib.dppo_loss_fwd_bwd(H, W, ids, pos, cu, one, one, lp, lp, recompute_logits=True, status=status)
        assert int(status) == want_flags
        return out

    bad_pos, bad_ids, at = pos.clone(), ids.clone(), int(pos[3]) + 1
    bad_pos[0], pos[0] = -5, 0
    bad_ids[at], ids[at] = V + 3, V - 1
    good = run(pos, ids, 0)
    bad = run(pos, bad_ids, lib.HEAD_BAD_TARGET)
    for name in ("logp", "dH", "dW", "loss"):
        assert torch.equal(good[name], bad[name]), name
    bad = run(bad_pos, ids, lib.HEAD_BAD_POSITION)
    assert torch.equal(good["logp"][1:], bad["logp"][1:]) and torch.isfinite(bad["logp"]).all()


@pytest.mark.parametrize("tokens,D", [(40, 64), (256, 320), (257, 64)])
def test_dh_of_few_tiles_in_many_parts(lib, tokens, D):
    # 313 slices of the vocabulary against one or two tiles of dH: cut into 19 parts of 16 and 17 slices
    _run_case(lib, _case("small", tokens, dtype="bf16", D=D, V=20001), TOL["bf16"])


@pytest.mark.parametrize("V", [3, 16384, 16385, 33001])
def test_fp32_row_statistics(lib, V):
    # one sweep of the row, one logit more, three sweeps with a ragged end; the padding of the logits holds NaN
    case = _case("tiny", 40, dtype="f32", D=16, V=V)
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(case.pk["T"], case.pk["N"], 16, V, 0, 0), DEV)
    ws.fill_(0xFF)
    logp, lse = lib.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos, ws=ws)
    # fp32 sums of V positive terms, 64 partial sums and more: a few times 2^-24 of a log-sum of at most 12
    logp_ref, lse_ref = case.oracle_logprob()
    assert np.abs(logp.cpu().numpy() - logp_ref).max() <= 1e-5
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-5


@pytest.mark.parametrize("tokens,V", [(7936, 1000), (7937, 1000), (8190, 33000)])
def test_statistics_of_many_tokens(lib, tokens, V):
    # both sides of 8192 padded tokens, from where 32 tokens are combined per workgroup; 4 and 129 tiles for 16 lane groups
    # of eight loads each
    case = _case("small", tokens, dtype="bf16", D=64, V=V)
    logp_ref, lse_ref = case.oracle_logprob()
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(case.pk["T"], tokens, 64, V, 1, 1), DEV)
    ws.fill_(0xFF)                               # NaN wherever a statistic that nobody wrote is read
    logp, lse = lib.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos, ws=ws)
    case.set_behaviour_logps(logp_ref)
    out = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                                case.logp_old, case.logp_ref, ws=ws)
    # fp32 sums of 64 products |h w| < 1 and of V exponentials in two levels: a few 2^-24 of a log-sum of at most 11
    assert np.abs(logp.cpu().numpy() - logp_ref).max() <= 1e-4
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-4
    assert np.abs(out["logp"].cpu().numpy() - logp_ref).max() <= 1e-4


def _logits_as_given(dtype, z, tokens):
    """H, W and ids of `tokens` positions that all have exactly the logits z (bfloat16: rounded): W holds them in its
    first column, H picks that column. Targets walk down the vocabulary from its last entry."""
    V, D = len(z), 64 if dtype == torch.bfloat16 else 1
    W = torch.zeros((V, D), dtype=dtype, device=DEV)
    W[:, 0] = torch.as_tensor(z, device=DEV).to(dtype)
    H = torch.zeros((tokens, D), dtype=dtype, device=DEV)
    H[:, 0] = 1.0
    ids = ((V - 1 - torch.arange(tokens, device=DEV, dtype=torch.int64) * 997) % V).to(torch.int32)
    return H, W, ids, to_np64(W[:, 0])


# one workgroup column of 96, 192 and 256 tokens; V: 71 and 142 softmax tiles against 64 lane groups of the combination,
# for float32 three sweeps of a row
@pytest.mark.parametrize("dtype,tokens,V", [(torch.bfloat16, 5, 18001), (torch.bfloat16, 130, 18001), (torch.bfloat16, 250, 18001),
                                            (torch.float32, 5, 33001)])
@pytest.mark.parametrize("kind", ["tile", "most", "lowest", "all", "nan", "inf"])
def test_logits_that_are_not_finite(lib, dtype, tokens, V, kind):
    """Vocabulary entries at minus infinity or at the type's lowest value carry no weight, also where they fill a softmax
    tile, all tiles but one, or a whole sweep; a NaN entry and an entry at plus infinity make lse and log-prob NaN."""
    z = np.random.default_rng(V).normal(size=V)
    if kind == "tile":
        z[256:512] = -np.inf                     # one tile of the 256-row and two of the 128-row GEMM
    elif kind == "most":
        z[:17920] = -np.inf                      # float32: the whole first sweep of 16384
    elif kind == "lowest":
        z[: V // 2] = float(torch.finfo(dtype).min)
    elif kind == "all":
        z[:] = -np.inf
    elif kind == "nan":
        z[300] = np.nan
    elif kind == "inf":
        z[V - 2] = np.inf
    H, W, ids, z64 = _logits_as_given(dtype, z, tokens)
    logp, lse = lib.dppo_token_logprob(H, W, ids, None)
    one, cu = torch.ones(1, device=DEV), torch.tensor([0, tokens], dtype=torch.int32, device=DEV)
    zeros = torch.zeros(tokens, device=DEV)
    out = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, zeros, zeros)
    torch.cuda.synchronize()
    got = [logp.cpu().numpy().astype(np.float64), out["logp"].cpu().numpy().astype(np.float64)]
    lse = lse.cpu().numpy().astype(np.float64)
    if kind in ("all", "nan", "inf"):
        assert np.isnan(got[0]).all() and np.isnan(got[1]).all()
        assert np.isnan(lse).all() or (kind == "all" and (lse == -np.inf).all())
        return
    m = z64.max()
    want = m + np.log(np.exp(z64 - m).sum())
    # fp32 sums of at most 33001 positive terms in two levels and fp32 exponentials: below 32 2^-24 of a log-sum of 11
    assert np.abs(lse - want).max() <= 32 * 2.0 ** -24 * 11
    want = z64[ids.cpu().numpy()] - want
    far = want < -1e30
    for g in got:
        assert np.abs(g[~far] - want[~far]).max() <= 32 * 2.0 ** -24 * 20
        assert (g[far] < -1e30).all()


# columns of 96, 128 and 192 tokens read the rows of H where they lie (bfloat16), columns of 256 a gathered copy
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n", [1, 96, 97, 128, 129, 192, 193, 257, 384, 385, 576, 577])
def test_scoring_tokens_where_they_lie(lib, dtype, n):
    """Positions in any order, repeated, out of range (clamped and reported), and without a list of positions."""
    T, D, V = 700, 192, 3001
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    H = torch.randn((T, D), device=DEV, generator=g).to(dtype)
    W = (0.1 * torch.randn((V, D), device=DEV, generator=g)).to(dtype)
    ids = torch.randint(0, V, (T,), device=DEV, dtype=torch.int32, generator=g)
    all_logp = torch.log_softmax(H.double() @ W.double().T, 1)
    tol = D * 2.0 ** -24 * float((H.abs().double() @ W.abs().double().T).max()) + 32 * 2.0 ** -24 * 20   # any order of the fp32 sums

    def check(pos, ids, want_flags):
        status = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        h = H if pos is not None else H[:n]
        logp, lse = lib.dppo_token_logprob(h, W, ids[:len(h)], pos, status=status)
        row = pos.long() if pos is not None else torch.arange(n, device=DEV)
        target = ids.long()[(row + (pos is not None)).clamp(0, len(h) - 1)].clamp(0, V - 1)
        want = all_logp[row.clamp(0, len(h) - 1), target]
        assert (logp.double() - want).abs().max() <= tol
        assert int(status) == want_flags

    pos = torch.randint(0, T - 1, (n,), device=DEV, dtype=torch.int32, generator=g)
    check(pos, ids, 0)
    check(None, ids, 0)
    pos[0] = -5 if n % 2 else T + 7
    check(pos, ids, lib.HEAD_BAD_POSITION)
    ids = ids.clone()
    ids[:n] = V + 3
    check(None, ids, lib.HEAD_BAD_TARGET)


# more sequences than workgroups of the reduction (4096), and one alone
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("S", [1, 2, 300, 4096, 4097, 9000])
def test_totals_of_many_sequences(lib, dtype, S):
    """The loss is the fp64 sum over the sequences rounded once (2^-24, and 2^-40 of the terms for the order of the fp64 sums),
    in every call into the same workspace: more sequences than workgroups, and one alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(S)
    D, V = 64, 257
    H = torch.randn((S, D), device=DEV, generator=g).to(dtype)
    W = (0.1 * torch.randn((V, D), device=DEV, generator=g)).to(dtype)
    ids = torch.randint(0, V, (S,), device=DEV, dtype=torch.int32, generator=g)
    cu = torch.arange(S + 1, device=DEV, dtype=torch.int32)
    adv, coef = torch.randn(S, device=DEV, generator=g), torch.rand(S, device=DEV, generator=g)
    lp = torch.full((S,), -5.5, device=DEV)
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(S, S, D, V, 1 if dtype == torch.bfloat16 else 0, True), H.device)
    for _ in range(3):
        out = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, adv, coef, lp, lp, ws=ws)
        terms = coef.double() * out["seq_loss"].double()
        assert abs(float(out["loss"]) - float(terms.sum())) <= 2.0 ** -24 * abs(float(terms.sum())) + 2.0 ** -40 * float(terms.abs().sum())
        assert float(out["stats"][2]) == S


# 143 and 300 tiles of dH (a last round of 143 and of 44), both operand layouts, against 1188 slices of the vocabulary
@pytest.mark.parametrize("tokens,D", [(2810, 3328), (7500, 2560)])
def test_dh_parts_in_the_memory_of_dw(lib, tokens, D):
    """A call that overwrites dW keeps partial tiles of dH there first, one that adds to it may not: the same dW, and dH the
    same but for the rounding of another order of the fp32 sums to bf16. Rows of every block of 256 tokens against float64."""
    V = 76000
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), device=DEV, generator=g).bfloat16()
    W = (0.02 * torch.randn((V, D), device=DEV, generator=g)).bfloat16()
    ids = torch.randint(0, V, (tokens,), device=DEV, dtype=torch.int32, generator=g)
    cu, one = torch.tensor([0, tokens], dtype=torch.int32, device=DEV), torch.ones(1, device=DEV)
    lp = torch.full((tokens,), -11.0, device=DEV)
    args = (H, W, ids, None, cu, one, one, lp, lp)
    over = lib.dppo_loss_fwd_bwd(*args)
    added = lib.dppo_loss_fwd_bwd(*args, dW=torch.zeros((V, D), device=DEV), accumulate_dW=True)
    assert torch.equal(over["dW"], added["dW"])
    a, b = over["dH"].float(), added["dH"].float()
    assert float((a - b).norm() / b.norm()) <= 2.0 ** -9       # each value within a rounding (2^-9) of the same sum, few differ
    assert torch.isfinite(a).all()
    rows = torch.arange(37, tokens, 251, device=DEV)
    W64 = W.double()
    logp64 = torch.log_softmax(H[rows].double() @ W64.T, 1)
    t = ids.long()[rows]
    l = logp64.gather(1, t[:, None])[:, 0]
    rho = torch.exp(l + 11.0)                                  # advantage 1: clipped away above 1.2
    c = (torch.where(rho > 1.2, 0.0, -rho) + 0.04 * (1.0 - 1.0 / rho)) / tokens
    want = (W64[t] - logp64.exp() @ W64) * c[:, None]
    for got in (a, b):
        err = (got[rows].double() - want).norm(dim=1) / want.norm(dim=1)
        worst = float(err.max())
        assert worst <= TOL["bf16"]["grad"]


@pytest.mark.parametrize("tokens", [40, 300, 700])
@pytest.mark.parametrize("D,V", [(1088, 33000), (512, 70000)])
def test_dw_tiles_walked_by_resident_workgroups(lib, tokens, D, V):
    # 645 and 548 tiles of dW for 256 workgroups, the last column or row of them partly filled, K of 4, 8 and 12 slices
    case = _case("small", tokens, dtype="bf16", D=D, V=V)
    out, _ = _run_case(lib, case, TOL["bf16"])
    old = torch.randn(V, D, device=DEV)
    acc = old.clone()
    lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                          case.logp_old, case.logp_ref, dW=acc, accumulate_dW=True)
    assert torch.equal(acc, old + out["dW"])


@pytest.mark.parametrize("tokens", [64, 128, 129, 16384, 16385])
def test_dw_walks_agree(lib, tokens):
    # resident workgroups add to what is there up to 16384 tokens and overwrite with up to 128; all other launches
    # have a workgroup per tile (270 tiles here). The sums are the same numbers in the same order
    D, V = 64, 69000
    g = torch.Generator(device=DEV)
    g.manual_seed(tokens)
    H = torch.randn((tokens, D), generator=g, device=DEV).to(torch.bfloat16)
    W = (torch.randn((V, D), generator=g, device=DEV) * 0.1).to(torch.bfloat16)
    ids = torch.randint(0, V, (tokens,), generator=g, device=DEV, dtype=torch.int32)
    one, cu = torch.ones(1, device=DEV), torch.tensor([0, tokens], dtype=torch.int32, device=DEV)
    logp, _ = lib.dppo_token_logprob(H, W, ids, None)
    old = torch.randn((V, D), generator=g, device=DEV)
    acc = old.clone()
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(tokens, tokens, D, V, 1, 1), DEV)
    out = lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, logp, logp, ws=ws)
    lib.dppo_loss_fwd_bwd(H, W, ids, None, cu, one, one, logp, logp, dW=acc, accumulate_dW=True, ws=ws)
    assert torch.equal(acc, old + out["dW"])
    # ratio 1, no KL: d loss / d logp = -1 / tokens for every token; one vocabulary slice in float64
    lo, hi = V - 300, V
    p = torch.exp(H.double() @ W.double()[lo:hi].T - torch.logsumexp(H.float() @ W.float().T, dim=1, keepdim=True).double())
    hot = (ids.long()[:, None] == torch.arange(lo, hi, device=DEV)[None]).double()
    want = ((hot - p).T @ H.double()) * (-1.0 / tokens)
    assert rel_fro(to_np64(out["dW"][lo:hi]), to_np64(want)) <= TOL["bf16"]["grad"]


@pytest.mark.parametrize("tokens", [1, 64, 65, 128, 192, 193, 321])
def test_dw_sums_over_whole_slices_of_tokens(lib, tokens):
    # one to six slices of 64 tokens, whatever the chunk is padded to; 270 tiles for 256 resident workgroups
    case = _case("small", tokens, dtype="bf16", D=320, V=34500)
    _run_case(lib, case, TOL["bf16"])
    _run_case(lib, case, TOL["bf16"], recompute_logits=True)


def test_long_chunk_with_few_output_tiles(lib):
    # 8400 loss tokens against a dW of 8 x 1 tiles: the dW GEMM's last (only) round of tiles is
    # nearly empty, so its tiles are cut along the token axis and summed by the second kernel
    case = _case("small", 8400, dtype="bf16", D=256, V=2000)
    assert case.pk["N"] >= 8300
    out, _ = _run_case(lib, case, TOL["bf16"])
    # the summing kernel also honours accumulation into an existing dW
    acc = out["dW"].clone()
    lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                          case.logp_old, case.logp_ref, dW=acc, accumulate_dW=True)
    assert torch.equal(acc, 2.0 * out["dW"])
    # a chunk of exactly 2048 tokens: the transposed hidden-state chunk gets a padded row pitch
    case = _case("small", 2048, dtype="bf16", D=256, V=2000)
    assert case.pk["N"] == 2048
    _run_case(lib, case, TOL["bf16"])


def test_clipping_zero_advantage_and_single_token_sequences(lib):
    rng = np.random.default_rng(8)
    # hand-built batch: constant groups (A = 0), one-token completions, both advantage signs
    rewards = np.array([[1, 1, 1, 1], [0, 1, 0, 1], [1, 0, 0, 0], [0, 0, 0, 0]], dtype=np.float32)
    sel = O.select(rewards, None, None, rng.random((4, 4), dtype=np.float32), 0.0, 0.5)
    pl = np.repeat(rng.integers(1, 9, size=4), 4).astype(np.int32)
    cl = rng.integers(1, 40, size=16).astype(np.int32)
    cl[[1, 6, 11]] = 1
    pk = O.pack(pl, cl, sel["keep_comp"].reshape(-1), 64, 3)
    wl = dataclasses.replace(WL.WORKLOADS["tiny"], D=128, V=777, dtype="bf16")
    # old-policy noise large enough that |log rho| > log 1.2 often: both clip branches active
    case = HeadCase(wl, pk, sel, 8, DEV, logp_noise=0.3)
    out, ref = _run_case(lib, case, TOL["bf16"], clip_lo=0.2, clip_hi=0.28, beta=0.1)
    assert 0.05 < ref["clip_frac"] < 0.9
    case32 = HeadCase(dataclasses.replace(wl, dtype="f32"), pk, sel, 8, DEV, logp_noise=0.3)
    _run_case(lib, case32, TOL["f32"], clip_lo=0.2, clip_hi=0.28, beta=0.1)


VARIANTS = [("token", "token_sum"), ("sequence", "seq_mean"), ("sequence", "token_sum")]


@pytest.mark.parametrize("ratio_level,aggregation", VARIANTS)
def test_objective_variants(lib, ratio_level, aggregation):
    """Sequence-level ratio and token-sum aggregation (the objectives the method is plugged into), with a
    decoupled clip tight enough that whole sequences are clipped away at the sequence level."""
    rb = WL.make_rollout("small")
    wl = rb.wl
    sel, pk = oracle_select_pack(rb)
    # token-normalised weights for the token sum: coef * G / (completion tokens of the group)
    if aggregation == "token_sum":
        want = O.token_norm_coef(sel["coef"], rb.comp_len)
        got = lib.dppo_token_norm_coef(torch.as_tensor(sel["coef"].astype(np.float32), device=DEV), rb.comp_len)
        assert np.allclose(got.cpu().numpy(), want, rtol=2e-6, atol=0)
        sel = dict(sel, coef=want)
    # advantages of both signs on every sequence (the workload's own are mostly zero on a short prefix)
    sel = dict(sel, adv=np.random.default_rng(12).normal(size=sel["adv"].shape).astype(np.float32))
    pk = truncate_pack(pk, 6000)
    case = HeadCase(wl, pk, sel, rb.seed, DEV, logp_noise=0.3)
    clip = dict(clip_lo=0.2, clip_hi=0.28)
    if ratio_level == "sequence":
        # sequence ratios sit much closer to 1 than token ratios: clip at their median distance from 1
        base, _ = case.oracle_logprob()
        case.set_behaviour_logps(base)
        cu = case.pk["loss_cu"]
        dist = [abs(np.expm1(np.mean(base[cu[i]:cu[i + 1]] - case.logp_old_np[cu[i]:cu[i + 1]]))) for i in range(len(cu) - 1)]
        clip = dict(clip_lo=float(np.median(dist)), clip_hi=float(np.median(dist)) * 1.5)
    out, ref = _run_case(lib, case, TOL["bf16"], beta=0.04, ratio_level=ratio_level, aggregation=aggregation, **clip)
    assert 0.0 < ref["clip_frac"] < 1.0
    # the workspace-limited (several chunks) and recompute paths agree with the default one
    T, N, D, V = case.pk["T"], case.pk["N"], wl.D, wl.V
    ws_min, ws_full = lib.dppo_workspace_min_bytes(T, N, D, V, 1, True), lib.dppo_workspace_bytes(T, N, D, V, 1, True)
    args = (case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
            case.logp_ref)
    kw = dict(beta=0.04, ratio_level=ratio_level, aggregation=aggregation, **clip)
    small = lib.dppo_loss_fwd_bwd(*args, ws=lib.alloc_workspace((ws_min + ws_full) // 2, DEV), **kw)
    # (the sequence ratios of the chunked call come from the forward-only pass, whose log-probs may differ
    # in the last bit from those of the pass that also keeps the exponentials)
    same_seq = torch.equal if ratio_level == "token" else (lambda a, b: torch.allclose(a, b, rtol=1e-5, atol=1e-6))
    assert _same_rows(small["dH"], out["dH"]) and same_seq(small["seq_loss"], out["seq_loss"])
    rec = lib.dppo_loss_fwd_bwd(*args, recompute_logits=True, **kw)
    assert rel_fro(to_np64(rec["dW"]), ref["dW"]) <= 1e-2 and _same_loss(rec["loss"], out["loss"], ref, case)


def test_sequence_ratio_with_forward_running_ahead(lib):
    """Sequence-level ratio with max_seq_tokens given: the forward of chunk c + 1 runs ahead of the backward of
    chunk c (one vocabulary GEMM per chunk, not two), the results are those of the single-chunk call, a broken
    promise is flagged, and without the promise the extra forward pass is taken."""
    rb = WL.make_rollout("small")
    sel, pk = oracle_select_pack(rb)
    sel = dict(sel, adv=np.random.default_rng(12).normal(size=sel["adv"].shape).astype(np.float32))
    pk = truncate_pack(pk, 6000)
    case = HeadCase(rb.wl, pk, sel, rb.seed, DEV, logp_noise=0.3)
    base, _ = case.oracle_logprob()
    case.set_behaviour_logps(base)
    cu = case.pk["loss_cu"]
    longest = int(np.diff(cu).max())
    assert 512 < longest <= 1024
    dist = [abs(np.expm1(np.mean(base[cu[i]:cu[i + 1]] - case.logp_old_np[cu[i]:cu[i + 1]]))) for i in range(len(cu) - 1)]
    kw = dict(beta=0.04, ratio_level="sequence", clip_lo=float(np.median(dist)), clip_hi=float(np.median(dist)) * 1.5)
    out, ref = _run_case(lib, case, TOL["bf16"], **kw)            # one chunk
    assert 0.0 < ref["clip_frac"] < 1.0
    T, N, D, V = case.pk["T"], case.pk["N"], case.wl.D, case.wl.V
    args = (case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
            case.logp_ref)
    lo2, hi2 = lib.dppo_workspace_min_bytes(T, N, D, V, 1, 2), lib.dppo_workspace_bytes(T, N, D, V, 1, 2)
    assert hi2 > lib.dppo_workspace_bytes(T, N, D, V, 1, 1) and lo2 > lib.dppo_workspace_min_bytes(T, N, D, V, 1, 1)
    # a workspace for two sets of chunks of about 1300 tokens (256 at lo2, 6144 at hi2, linear in between)
    ws = lib.alloc_workspace(lo2 + (hi2 - lo2) * (1300 - 256) // (6144 - 256), DEV)
    status = torch.full((1,), -1, dtype=torch.int32, device=DEV)

    def launches(**more):
        lib.dppo_timing_enable(True)
        lib.dppo_timing_read(reset=True)
        res = lib.dppo_loss_fwd_bwd(*args, ws=ws, status=status, **kw, **more)
        torch.cuda.synchronize()
        t = lib.dppo_timing_read(reset=True)
        lib.dppo_timing_enable(False)
        return res, t["logits_gemm"][1], t["dh_gemm"][1]

    for recompute in (False, True):
        got, n_logits, n_dh = launches(max_seq_tokens=longest, recompute_logits=recompute)
        assert n_dh >= 4 and n_logits == (2 if recompute else 1) * n_dh, (n_logits, n_dh)
        assert int(status.item()) == 0
        if not recompute:
            assert _same_rows(got["dH"], out["dH"]) and torch.equal(got["seq_loss"], out["seq_loss"])
        assert rel_fro(to_np64(got["dW"]), ref["dW"]) <= 1e-2 and rel_fro(to_np64(got["dH"]), ref["dH"]) <= 1e-2
        assert _same_loss(got["loss"], out["loss"], ref, case)
        assert np.abs(got["logp"].cpu().numpy() - ref["logp"]).max() <= TOL["bf16"]["logp"]
    # no promise: one forward-only pass first
    got, n_logits, n_dh = launches()
    assert n_logits == 2 * n_dh and int(status.item()) == 0
    assert _same_rows(got["dH"], out["dH"]) and torch.allclose(got["seq_loss"], out["seq_loss"], rtol=1e-5, atol=1e-6)
    # a promise the chunks cannot hold falls back to that pass as well
    got, n_logits, n_dh = launches(max_seq_tokens=4 * longest)
    assert n_logits == 2 * n_dh and int(status.item()) == 0
    # a broken promise (sequences of up to 1012 tokens against chunks of 256): flagged, every kernel runs to the end
    ws = lib.alloc_workspace(lo2, DEV)
    got, n_logits, n_dh = launches(max_seq_tokens=256)
    assert n_logits == n_dh == -(-N // 256)
    assert int(status.item()) & lib.HEAD_SEQ_TOO_LONG
    assert np.abs(got["logp"].cpu().numpy() - ref["logp"]).max() <= TOL["bf16"]["logp"]


@pytest.mark.parametrize("case_seed", [11, 12, 13, 14, 15, 16, 17, 18])
def test_random_shapes_with_tails(lib, case_seed):
    """Seeded random shapes (D any multiple of 64, so the 256-row blocks of the backward GEMMs' B operands are
    partly filled; V and N with tails), a workspace of random size between the minimum and the recommended one
    (several chunks), both gradient modes, and the sequence-level ratio with the forward running ahead."""
    rng = np.random.default_rng(case_seed)
    D = int(rng.choice([64, 128, 192, 320, 448, 576, 1024, 1088]))
    V = int(rng.integers(100, 6000))
    case = _case("small", int(rng.integers(150, 2600)), seed=int(rng.integers(1, 10**6)), dtype="bf16", D=D, V=V)
    T, N = case.pk["T"], case.pk["N"]
    out, ref = _run_case(lib, case, TOL["bf16"])
    args = (case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
            case.logp_ref)
    lo, hi = lib.dppo_workspace_min_bytes(T, N, D, V, 1, True), lib.dppo_workspace_bytes(T, N, D, V, 1, True)
    ws = lib.alloc_workspace(int(lo + (hi - lo) * float(rng.uniform(0.0, 0.9))), DEV)
    for recompute in (False, True):
        got = lib.dppo_loss_fwd_bwd(*args, ws=ws, recompute_logits=recompute)
        assert rel_fro(to_np64(got["dW"]), ref["dW"]) <= 1e-2 and rel_fro(to_np64(got["dH"]), ref["dH"]) <= 1e-2
        assert np.abs(got["logp"].cpu().numpy() - ref["logp"]).max() <= TOL["bf16"]["logp"]
        _assert_loss(float(got["loss"].item()), ref, case, TOL["bf16"]["loss"])
    ref_s = case.oracle_loss(ratio_level="sequence")
    lo2, hi2 = lib.dppo_workspace_min_bytes(T, N, D, V, 1, 2), lib.dppo_workspace_bytes(T, N, D, V, 1, 2)
    ws2 = lib.alloc_workspace(int(lo2 + (hi2 - lo2) * float(rng.uniform(0.3, 1.0))), DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    got = lib.dppo_loss_fwd_bwd(*args, ws=ws2, ratio_level="sequence", status=status,
                                max_seq_tokens=int(np.diff(case.pk["loss_cu"]).max()))
    assert int(status.item()) == 0
    assert rel_fro(to_np64(got["dW"]), ref_s["dW"]) <= 1e-2 and rel_fro(to_np64(got["dH"]), ref_s["dH"]) <= 1e-2
    _assert_loss(float(got["loss"].item()), ref_s, case, TOL["bf16"]["loss"])


def test_objective_variants_fp32(lib):
    case = _case("tiny", None)
    for ratio_level, aggregation in VARIANTS:
        _run_case(lib, case, TOL["f32"], clip_lo=0.002, clip_hi=0.003, ratio_level=ratio_level, aggregation=aggregation)


def test_targets_of_vanishing_probability(lib):
    # The bf16 backward pass keeps exp(z - z_target) per stored entry; rows whose target has a
    # log-prob below about -34.5 leave the range that scheme is used in and must come out right through
    # the exact row path (some of them overflow the stored exponentials outright), next to rows just
    # above the limit, with stored exponentials up to e^34, and ordinary rows on the fast path.
    # Second shape: D beyond one 2048-column slab of the exact path.
    for D, V, factor, mid in ((128, 777, 64.0, 16.0), (2304, 300, 16.0, 4.0)):
        case = _case("tiny", None, dtype="bf16", D=D, V=V)
        lp = torch.as_tensor(case.pk["loss_pos"], device=DEV).long()
        case.H[lp[::3]] *= factor       # exact in bf16
        case.H[lp[1::3]] *= mid
        logp_ref, _ = case.oracle_logprob()
        assert (logp_ref < -100).sum() >= 5 and (logp_ref > -15).sum() >= 5
        assert ((logp_ref > -34) & (logp_ref < -20)).sum() >= 5 and ((logp_ref > -69) & (logp_ref < -35)).sum() >= 5
        _run_case(lib, case, TOL["bf16"])
    # several chunks (smallest workspace), each with its own list of rows to redo
    case = _case("small", 1500)
    lp = torch.as_tensor(case.pk["loss_pos"], device=DEV).long()
    case.H[lp[::5]] *= 64.0
    logp_ref, _ = case.oracle_logprob()
    assert (logp_ref < -100).sum() >= 100
    case.set_behaviour_logps(logp_ref)
    ref = case.oracle_loss()
    T, N, D, V = case.pk["T"], case.pk["N"], case.wl.D, case.wl.V
    ws = lib.alloc_workspace(lib.dppo_workspace_min_bytes(T, N, D, V, 1, True), DEV)
    out = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                                case.logp_old, case.logp_ref, ws=ws)
    assert np.abs(out["logp"].cpu().numpy() - ref["logp"]).max() <= TOL["bf16"]["logp"]
    assert rel_fro(to_np64(out["dH"]), ref["dH"]) <= 1e-2 and rel_fro(to_np64(out["dW"]), ref["dW"]) <= 1e-2


def test_coincident_policies(lib):
    case = _case("tiny", None, dtype="bf16")
    logp, _ = lib.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos)
    out = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef,
                                logp, logp)
    # ratio 1 and KL 0: each sequence's loss is minus its advantage
    assert np.allclose(out["seq_loss"].cpu().numpy(), -case.seq_adv_np, rtol=1e-5, atol=1e-6)
    assert abs(float(out["stats"][0])) < 1e-9 and float(out["stats"][1]) == 0.0


def test_identity_rows_chunking_accumulation_and_recompute(lib):
    case = _case("small", 1200)
    logp_ref, _ = case.oracle_logprob()
    case.set_behaviour_logps(logp_ref)
    ref = case.oracle_loss()
    P = lib
    args = (case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
            case.logp_ref)
    base = P.dppo_loss_fwd_bwd(*args)
    # (a) a workspace that only fits small chunks gives the same result up to summation order
    T, N, D, V = case.pk["T"], case.pk["N"], case.wl.D, case.wl.V
    ws_min, ws_full = P.dppo_workspace_min_bytes(T, N, D, V, 1, True), P.dppo_workspace_bytes(T, N, D, V, 1, True)
    small_ws = P.alloc_workspace((ws_min + ws_full) // 2, DEV)
    assert ws_min < small_ws.numel() < ws_full
    chunked = P.dppo_loss_fwd_bwd(*args, ws=small_ws)
    assert rel_fro(to_np64(chunked["dW"]), ref["dW"]) <= 1e-2
    assert rel_fro(to_np64(chunked["dW"]), to_np64(base["dW"])) <= 1e-4
    assert _same_rows(chunked["dH"], base["dH"])
    assert abs(float(chunked["loss"]) - float(base["loss"])) <= 1e-6 * abs(float(base["loss"])) + 1e-9
    # (b) accumulate_dW adds to the buffer
    acc = base["dW"].clone()
    P.dppo_loss_fwd_bwd(*args, dW=acc, accumulate_dW=True)
    assert rel_fro(to_np64(acc), 2.0 * to_np64(base["dW"])) <= 1e-6
    # (c) recomputing the logits in the backward instead of keeping a chunk of exponentials
    rec = P.dppo_loss_fwd_bwd(*args, recompute_logits=True)
    assert rel_fro(to_np64(rec["dH"]), ref["dH"]) <= 1e-2
    assert rel_fro(to_np64(rec["dW"]), ref["dW"]) <= 1e-2
    assert _same_loss(rec["loss"], base["loss"], ref, case)
    # (d) identity loss rows: compact H rows and targets handed over directly
    lp = case.pk["loss_pos"]
    Hc = case.H[torch.as_tensor(lp, device=DEV).long()].contiguous()
    yc = case.ids[torch.as_tensor(lp + 1, device=DEV).long()].contiguous()
    ident = P.dppo_loss_fwd_bwd(Hc, case.W, yc, None, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
                                case.logp_ref)
    assert torch.equal(ident["dH"], base["dH"][torch.as_tensor(lp, device=DEV).long()])
    assert rel_fro(to_np64(ident["dW"]), to_np64(base["dW"])) <= 1e-6
    lpi, _ = P.dppo_token_logprob(Hc, case.W, yc, None)
    assert np.abs(lpi.cpu().numpy() - logp_ref).max() <= 2e-3


def test_empty_batch(lib):
    # every completion pruned: packed tokens may exist, loss tokens do not
    for dtype in (torch.bfloat16, torch.float32):
        T, D, V = 37, 128, 300
        H = torch.randn(T, D, device=DEV).to(dtype)
        W = torch.randn(V, D, device=DEV).to(dtype)
        ids = torch.zeros(T, dtype=torch.int32, device=DEV)
        none_i = torch.zeros(0, dtype=torch.int32, device=DEV)
        none_f = torch.zeros(0, dtype=torch.float32, device=DEV)
        cu = torch.zeros(1, dtype=torch.int32, device=DEV)
        logp, lse = lib.dppo_token_logprob(H, W, ids, none_i)
        assert logp.numel() == 0 and lse.numel() == 0
        out = lib.dppo_loss_fwd_bwd(H, W, ids, none_i, cu, none_f, none_f, none_f, none_f)
        torch.cuda.synchronize()
        assert float(out["loss"]) == 0.0 and out["seq_loss"].numel() == 0 and float(out["stats"][2]) == 0.0
        assert not bool(out["dH"].any()) and not bool(out["dW"].any())
        keep = torch.full((V, D), 3.0, device=DEV)
        lib.dppo_loss_fwd_bwd(H, W, ids, none_i, cu, none_f, none_f, none_f, none_f, dW=keep, accumulate_dW=True)
        assert bool((keep == 3.0).all())


def test_hip_graph_replays_match_eager(lib):
    # The entry points only enqueue kernels on the caller's stream (no allocation, no
    # synchronisation, no memset nodes), so a whole loss step can be captured once and replayed.
    # Every replay is checked against the eager result, with eager work, changed inputs and
    # synchronisations between the replays.
    case = _case("small", 1500)
    logp_ref, _ = case.oracle_logprob()
    case.set_behaviour_logps(logp_ref)
    args = (case.H, case.W, case.ids, case.loss_pos, case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old,
            case.logp_ref)
    eager = lib.dppo_loss_fwd_bwd(*args)            # also runs the one-time kernel attribute setup
    T, N, D, V = case.pk["T"], case.pk["N"], case.wl.D, case.wl.V
    ws = lib.alloc_workspace(lib.dppo_workspace_bytes(T, N, D, V, 1, True), DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        out = lib.dppo_loss_fwd_bwd(*args, ws=ws)
    keys = ("loss", "logp", "seq_loss", "stats", "dH", "dW")
    for rep in range(3):
        for k in keys:
            out[k].fill_(float("nan"))               # eager work between the replays
        if rep == 2:                                 # changed inputs: the graph reads the same buffers
            case.logp_old.add_(0.05)
            eager = lib.dppo_loss_fwd_bwd(*args)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in keys:
            assert torch.equal(out[k], eager[k]), (rep, k)


def test_argument_validation(lib):
    case = _case("tiny", None, dtype="bf16")
    P = lib
    with pytest.raises(P.DppoError):      # workspace too small
        P.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos, ws=P.alloc_workspace(256, DEV))
    H_bad = torch.zeros((case.pk["T"], 72), dtype=torch.bfloat16, device=DEV)   # D % 64 != 0
    W_bad = torch.zeros((64, 72), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(P.DppoError):
        P.dppo_token_logprob(H_bad, W_bad, case.ids, case.loss_pos)


@pytest.mark.parametrize("name,recompute", [("qwen3_4b", False), ("qwen3_8b", False), ("stress", False),
                                            ("stress", True), ("qwen3_4b", True)])
def test_full_width_slices(lib, name, recompute):
    # full hidden and vocabulary size of the Qwen3-shaped workloads on the first packed sequences up to
    # 2100 loss tokens: eight full 256-token tiles and a ragged ninth, V = 151936 (593 full vocabulary
    # tiles and one half tile). With recompute the backward runs the vocabulary GEMM a second time
    # (the mode the stress configuration is stated in), whose epilogue masks the half tile by itself.
    case = _case(name, 2100)
    assert case.pk["N"] == 2100 and case.wl.V % 256 != 0
    _run_case(lib, case, TOL["bf16"], recompute_logits=recompute)


def test_status_word_and_empty_segment(lib):
    """Conditions only the device can see: a target id outside [0, V) and a loss_pos entry outside
    [0, T - 1) are clamped and reported in the status word; every kernel still finishes and the
    tokens that were fine come out as without the fault. An empty segment of loss_cu contributes 0."""
    case = _case("tiny", None, dtype="bf16", D=128, V=1000)
    logp_ref, _ = case.oracle_logprob()
    case.set_behaviour_logps(logp_ref)
    ref = case.oracle_loss()
    args = (case.loss_cu, case.seq_adv, case.seq_coef, case.logp_old, case.logp_ref)
    status = torch.full((1,), 77, dtype=torch.int32, device=DEV)
    good = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, *args, status=status)
    assert int(status.item()) == 0
    lib.dppo_token_logprob(case.H, case.W, case.ids, case.loss_pos, status=status.fill_(77))
    assert int(status.item()) == 0
    N, T, V = case.pk["N"], case.pk["T"], case.wl.V
    # (a) a target id beyond the vocabulary (token 5) and a negative one (token 9)
    ids_bad = case.ids.clone()
    lp = case.pk["loss_pos"]
    ids_bad[int(lp[5]) + 1] = V + 7
    ids_bad[int(lp[9]) + 1] = -3
    logp, _ = lib.dppo_token_logprob(case.H, case.W, ids_bad, case.loss_pos, status=status.fill_(77))
    assert int(status.item()) == lib.HEAD_BAD_TARGET
    okay = np.ones(N, bool)
    okay[[5, 9]] = False
    assert np.abs(logp.cpu().numpy() - logp_ref)[okay].max() <= 2e-3 and torch.isfinite(logp).all()
    out = lib.dppo_loss_fwd_bwd(case.H, case.W, ids_bad, case.loss_pos, *args, status=status.fill_(77))
    assert int(status.item()) == lib.HEAD_BAD_TARGET
    assert torch.isfinite(out["dH"].float()).all() and torch.isfinite(out["dW"]).all()
    # (b) loss positions outside the packed tokens
    pos_bad = case.loss_pos.clone()
    pos_bad[3] = T + 1000
    pos_bad[4] = -5
    pos_bad[N - 1] = T - 1                     # its target would be token T
    logp, _ = lib.dppo_token_logprob(case.H, case.W, case.ids, pos_bad, status=status.fill_(77))
    assert int(status.item()) == lib.HEAD_BAD_POSITION
    okay = np.ones(N, bool)
    okay[[3, 4, N - 1]] = False
    assert np.abs(logp.cpu().numpy() - logp_ref)[okay].max() <= 2e-3
    out = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, pos_bad, *args, status=status.fill_(77))
    torch.cuda.synchronize()
    assert int(status.item()) == lib.HEAD_BAD_POSITION
    assert torch.isfinite(out["dH"].float()).all() and torch.isfinite(out["dW"]).all()
    # both at once
    lib.dppo_loss_fwd_bwd(case.H, case.W, ids_bad, pos_bad, *args, status=status.fill_(77))
    assert int(status.item()) == lib.HEAD_BAD_TARGET | lib.HEAD_BAD_POSITION
    # (c) an empty segment in the middle and one at the end: same loss and gradients as without them
    cu = case.pk["loss_cu"]
    S = len(cu) - 1
    cu2 = np.concatenate([cu[:3], [cu[2]], cu[3:], [cu[-1]]]).astype(np.int32)
    ins = lambda a, v: np.concatenate([a[:2], [v], a[2:], [v]]).astype(np.float32)
    for ratio_level in ("token", "sequence"):
        base = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, *args, ratio_level=ratio_level)
        out = lib.dppo_loss_fwd_bwd(case.H, case.W, case.ids, case.loss_pos, torch.as_tensor(cu2, device=DEV),
                                    torch.as_tensor(ins(case.seq_adv_np, 1.5), device=DEV),
                                    torch.as_tensor(ins(case.seq_coef_np, 0.25), device=DEV), case.logp_old,
                                    case.logp_ref, ratio_level=ratio_level)
        # (the final sum over sequences associates differently once the indices shift)
        assert torch.allclose(out["loss"], base["loss"], rtol=1e-6, atol=0) and torch.equal(out["dH"], base["dH"])
        assert torch.equal(out["dW"], base["dW"])
        sl = out["seq_loss"].cpu().numpy()
        assert sl[2] == 0.0 and sl[-1] == 0.0 and np.array_equal(np.delete(sl, [2, S + 1]), base["seq_loss"].cpu().numpy())
    assert abs(float(good["loss"]) - ref["loss"]) <= 1e-3 * max(abs(ref["loss"]), 1e-3)
