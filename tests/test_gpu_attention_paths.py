"""The attention kernels where a path of theirs begins or ends: tile edges of both sequences, every number of 16-column steps of the head, and
inputs whose softmax reference has to move late, against the oracle's operations."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import ops

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2      # operands, probabilities and results in bf16 (2^-9 each), fp32 sums: max error over the largest element


def _late_moves(logits):
    """Replays the forward's rule on the oracle's logits: a wave (32 queries) moves its references at a tile of 64 keys when the probabilities that
    one of its lanes adds up (32 keys: accumulator rows 8 i + 4 g .. + 3 of both halves for lane half g) exceed 2^8 relative to the old reference; the new
    one is 2^8 above the largest score.  (steps after the first tile, moves among them)"""
    s = np.asarray(logits) * 1.4426950408889634
    s = s.reshape((-1,) + s.shape[-2:])
    half = (np.arange(64) // 4) % 2
    steps = moves = 0
    for one in s:
        for q0 in range(0, one.shape[0], 32):
            blk = one[q0:q0 + 32]
            ref = np.full(blk.shape[0], -np.inf)
            for k0 in range(0, blk.shape[1], 64):
                t = blk[:, k0:k0 + 64]
                if k0 > 0:
                    with np.errstate(over="ignore"):
                        e = np.exp2(t - ref[:, None])
                    h = half[:t.shape[1]]
                    bump = bool(np.any(e[:, h == 0].sum(1) > 256) or np.any(e[:, h == 1].sum(1) > 256))
                    steps += 1
                    moves += bump
                if k0 == 0 or bump:
                    ref = np.maximum(ref, t.max(axis=1) + 8)
    return steps, moves


def _run(B_, H, Nq, Nk, dh, gain, shift, seed=5, backward=True):
    import torch
    from paper_2405_01248_amd import binding as B
    from paper_2405_01248_amd.harness import _dev_to_np, _np_to_dev, rel_err
    d = H * dh
    q, k, v, do = si.make_attention_inputs(B_, H, Nq, Nk, dh, seed=seed, gain=gain, row_shift=shift)
    dq_, dk_, dv_, ddo = (_np_to_dev(t, "bf16") for t in (q, k, v, do))
    o = torch.zeros((B_, Nq, d), dtype=torch.bfloat16, device="cuda:0")
    lse = torch.zeros((B_, H, Nq), dtype=torch.float32, device="cuda:0")
    scale = 1.0 / np.sqrt(dh)
    B.op_attention_fwd(B.DP_BF16, B_, H, Nq, Nk, dh, False, scale, dq_, d, dk_, d, dv_, d, o, d, lse)
    torch.cuda.synchronize()
    errs = {"o": rel_err(_dev_to_np(o), ops.attention_fwd(q, k, v, H, False))}
    if backward:
        gq, gk, gv = (torch.zeros_like(t) for t in (dq_, dk_, dv_))
        delta = torch.zeros((B_, H, Nq), dtype=torch.float32, device="cuda:0")
        B.op_attention_bwd(B.DP_BF16, B_, H, Nq, Nk, dh, scale, dq_, d, dk_, d, dv_, d, o, d, lse, ddo, d, delta, gq, d, gk, d, gv, d)
        torch.cuda.synchronize()
        for n, g, r in zip(("dq", "dk", "dv"), (gq, gk, gv), ops.attention_bwd(do, q, k, v, H, False)):
            errs[n] = rel_err(_dev_to_np(g), r)
    return q, k, errs


@pytest.mark.parametrize("dh", [8, 40, 48, 56, 64, 72, 80, 88, 96])
@pytest.mark.parametrize("Nq,Nk", [(1, 1), (33, 65), (129, 64), (64, 129), (191, 257)])
def test_edges_of_tiles_and_heads(Nq, Nk, dh):
    _, _, errs = _run(1, 2, Nq, Nk, dh, 1.0, 0.0)
    print(f"\n[attention q{Nq} k{Nk} dh{dh}] {errs}", flush=True)
    if Nk == 1:      # one key: the probabilities are 1 and dS = dP - delta is 0 but for the rounding of O, which a relative error of dq, dk would show
        errs.pop("dq"), errs.pop("dk")
    assert max(errs.values()) <= TOL_BF16, errs


@pytest.mark.parametrize("dh", [40, 64, 72, 96])
@pytest.mark.parametrize("Nk", [1, 31, 32, 77, 96, 127, 128, 129, 160, 225, 255, 256, 257])
def test_backward_with_all_keys_in_a_workgroup(Nk, dh):
    """Up to 256 keys: one kernel, four or eight waves of 32 keys, of which the last may be partly filled or empty."""
    for Nq in (1, 64, 65, 200):
        _, _, errs = _run(1, 2, Nq, Nk, dh, 1.0, 0.0, seed=Nk + Nq)
        print(f"\n[attention q{Nq} k{Nk} dh{dh}] {errs}", flush=True)
        if Nk == 1:
            errs.pop("dq"), errs.pop("dk")
        assert max(errs.values()) <= TOL_BF16, errs


@pytest.mark.parametrize("Nk,dh", [(77, 64), (200, 72), (300, 64), (300, 72), (300, 96)])
def test_rows_of_very_low_logits_meet_keys_that_are_not_there(Nk, dh):
    """Rows shifted by up to +-200: where all logits of a row lie below -88 the probability of a padded key (score 0) overflows."""
    q, k, errs = _run(1, 2, 150, Nk, dh, 1.001, 200.0)
    from softmax_schedule import head_logits
    assert head_logits(q, k, 2).max(axis=-1).min() < -90
    print(f"\n[attention low logits k{Nk} dh{dh}] {errs}", flush=True)
    assert all(np.isfinite(e) for e in errs.values()) and max(errs.values()) <= TOL_BF16, errs


@pytest.mark.parametrize("case", [(1, 3, 200, 449, 64, 16.0, 80.0), (1, 2, 160, 384, 72, 8.0, 40.0), (1, 2, 96, 320, 40, 16.0, 0.0)])
def test_late_moves_of_the_softmax_reference(case):
    from softmax_schedule import head_logits
    q, k, errs = _run(*case)
    steps, moves = _late_moves(head_logits(q, k, case[1]))
    print(f"\n[attention late moves {case}] {moves} of {steps} steps, {errs}", flush=True)
    assert moves > 0, "the inputs do not reach the path"
    assert max(errs.values()) <= TOL_BF16, errs


def _heads_of_one_batch(heads, tokens, causal, dh=64, keys=None):
    """The first head's rows of a launch with all heads and of one with that head alone, on the same operands."""
    import torch
    from paper_2405_01248_amd import binding as B
    d, keys = heads * dh, keys or tokens
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((n, d), generator=gen, device="cuda").to(torch.bfloat16) for n in (tokens, keys, keys))
    outs = []
    for h in (heads, 1):
        o = torch.zeros((tokens, d), dtype=torch.bfloat16, device="cuda")
        lse = torch.zeros((h, tokens), dtype=torch.float32, device="cuda")
        B.op_attention_fwd(B.DP_BF16, 1, h, tokens, keys, dh, causal, dh ** -0.5, q, d, k, d, v, d, o, d, lse)
        torch.cuda.synchronize()
        outs.append((o[:, :dh].clone(), lse[0].clone()))
    return outs


@pytest.mark.parametrize("heads,tokens", [(72, 512), (132, 192)])
def test_waves_that_take_turns_give_the_same_bits(heads, tokens):
    """More workgroups than CUs (288 of eight tiles of keys, 264 of three), all resident: wave priorities rotate.  They change the order in time and nothing else: the first head alone (few workgroups, no
    turns) has the same bits."""
    import torch
    (o, _), (alone, _) = _heads_of_one_batch(heads, tokens, False)
    assert torch.equal(o, alone)


@pytest.mark.parametrize("dh", [40, 56, 64, 72])
@pytest.mark.parametrize("heads", [384, 385, 512, 513])
def test_causal_workgroups_that_a_cu_holds_three_and_four_of(heads, dh):
    """768 workgroups of 128 queries are three a CU, 1024 four, which another instance of the kernel takes at widths above 48: the first head alone has the
    same bits."""
    import torch
    (o, lse), (alone, lse_alone) = _heads_of_one_batch(heads, 256, True, dh)
    assert torch.equal(o, alone) and torch.equal(lse, lse_alone)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dh", [40, 64, 72, 96])
@pytest.mark.parametrize("heads,tokens,keys", [(511, 128, 128), (512, 128, 128), (512, 97, 121), (512, 113, 120), (256, 129, 125)])
def test_forward_of_many_heads_in_the_loop_and_with_all_keys_at_once(heads, tokens, keys, dh, causal):
    """From 512 workgroups of one tile of queries on the loop takes 121 to 128 keys, below that and for one head alone they lie in LDS at once: the same bits."""
    import torch
    (o, lse), (alone, lse_alone) = _heads_of_one_batch(heads, tokens, causal, dh, keys)
    assert torch.equal(o, alone) and torch.equal(lse, lse_alone)


@pytest.mark.parametrize("B,H,Nq,Nk,dh", [(1, 1, 1, 1, 1), (2, 4, 64, 64, 16), (1, 3, 65, 63, 7), (1, 2, 256, 256, 24), (1, 2, 257, 256, 24), (1, 1, 5, 512, 33), (1, 1, 5, 513, 33), (2, 1, 130, 9, 200)])
def test_f32_backward_in_one_launch_and_in_two(B, H, Nq, Nk, dh):
    # one launch up to 512 keys over batch and heads and 256 queries, two beyond; widths that are no multiple of four, rows wider than the heads
    import torch
    from paper_2405_01248_amd import binding as bd
    g = torch.Generator().manual_seed(Nq * 1000 + Nk)
    d, ld = H * dh, H * dh + 3
    q, k, v, do = (torch.randn(B, n, ld, generator=g) for n in (Nq, Nk, Nk, Nq))
    scale = dh ** -0.5
    Q, K, V, DO = (x[..., :d].double().reshape(B, -1, H, dh).transpose(1, 2).contiguous() for x in (q, k, v, do))
    S = (Q @ K.transpose(2, 3).contiguous() * scale).softmax(-1)
    O = S @ V
    dS = S * (DO @ V.transpose(2, 3).contiguous() - (DO * O).sum(-1, keepdim=True))
    want = {"o": O, "dq": dS @ K * scale, "dk": dS.transpose(2, 3).contiguous() @ Q * scale, "dv": S.transpose(2, 3).contiguous() @ DO}
    q, k, v, do = (x.cuda() for x in (q, k, v, do))
    o, dq, dk, dv = torch.full_like(q, 7.0), torch.full_like(q, 7.0), torch.full_like(k, 7.0), torch.full_like(v, 7.0)
    lse, delta = torch.empty(B, H, Nq, device="cuda"), torch.empty(B, H, Nq, device="cuda")
    bd.op_attention_fwd(bd.DP_F32, B, H, Nq, Nk, dh, False, scale, q, ld, k, ld, v, ld, o, ld, lse)
    bd.op_attention_bwd(bd.DP_F32, B, H, Nq, Nk, dh, scale, q, ld, k, ld, v, ld, o, ld, lse, do, ld, delta, dq, ld, dk, ld, dv, ld)
    torch.cuda.synchronize()
    for name, x in (("o", o), ("dq", dq), ("dk", dk), ("dv", dv)):
        x = x.cpu()
        assert (x[..., d:] == 7.0).all(), name
        got, ref = x[..., :d].double().reshape(B, -1, H, dh).transpose(1, 2), want[name]
        # sums of at most 513 terms in fp32, logits of a few units: 513 eps / 2 would be 3e-5 if every rounding had the same sign; a gradient that
        # cancels (one key: dS = 0) is held against the size of its terms instead
        size = max(float(ref.norm()), 1e-2 * float(DO.norm()))
        assert float((got - ref).norm()) <= 3e-5 * size, name


@pytest.mark.parametrize("dh", [40, 64, 72, 80, 96])
@pytest.mark.parametrize("tokens,ctx,shares", [(250, 77, 2), (293, 129, 2), (421, 77, 3), (421, 256, 3), (2100, 77, 11), (2100, 200, 11)])
def test_shares_of_the_queries_with_all_keys_in_a_workgroup(dh, tokens, ctx, shares):
    """Cross-attention of a stage, which has scratch for the shares' sums.  4 query tiles in shares of 2 and 2, 5 in 3 and 2, 7 in 3, 3 and 1, 33 in eleven of 3,
    the last tile partly filled; three to six 16-wide steps over the head; four and eight waves."""
    import torch
    from paper_2405_01248_amd import binding as B
    from paper_2405_01248_amd.harness import DeviceStage
    from test_gpu_parity import _compare, _oracle_stage
    cfg = si.StageConfig(f"shares_q{tokens}_k{ctx}_dh{dh}", si.UNET, "bf16", 1, 1, tokens, 2 * dh, 2, dh, ctx, 64, 128)
    inp = si.make_stage_inputs(cfg, seed=tokens + dh)
    ds = DeviceStage(cfg, inp)
    B.ktime_begin(256)
    ds.step()
    torch.cuda.synchronize()
    rows = B.ktime_end(256)
    assert [r["k"] for r in rows if r["kind"] == "reduce" and (r["m"], r["n"]) == (ctx, 2 * dh)] == [shares], rows
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))


@pytest.mark.parametrize("B,H,Nq,Nk,dh", [(2, 4, 64, 64, 16), (1, 2, 200, 256, 24)])
def test_f32_backward_in_the_place_of_its_inputs(B, H, Nq, Nk, dh):
    # dQ over O, dK over K, dV over V, one at a time and all together, at sizes where separate results are formed in one launch
    import torch
    from paper_2405_01248_amd import binding as bd
    g = torch.Generator(device="cuda").manual_seed(Nk)
    d, scale = H * dh, dh ** -0.5
    q, k, v, do = (torch.randn(B, n, d, generator=g, device="cuda") for n in (Nq, Nk, Nk, Nq))
    o, lse, delta = torch.empty_like(q), torch.empty(B, H, Nq, device="cuda"), torch.empty(B, H, Nq, device="cuda")
    bd.op_attention_fwd(bd.DP_F32, B, H, Nq, Nk, dh, False, scale, q, d, k, d, v, d, o, d, lse)

    def backward(over):
        K, V, O = k.clone(), v.clone(), o.clone()
        dq = O if "q" in over else torch.empty_like(q)
        dk = K if "k" in over else torch.empty_like(k)
        dv = V if "v" in over else torch.empty_like(v)
        bd.op_attention_bwd(bd.DP_F32, B, H, Nq, Nk, dh, scale, q, d, K, d, V, d, O, d, lse, do, d, delta, dq, d, dk, d, dv, d)
        torch.cuda.synchronize()
        return dq, dk, dv

    want = backward("")
    for over in ("q", "k", "v", "qkv"):
        for x, y in zip(backward(over), want):
            # delta is formed in another order in one launch: a few roundings of a sum of dh terms
            assert float((x - y).norm()) <= 1e-6 * float(y.norm()), over
