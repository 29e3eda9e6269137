"""Attention (non-expert) layer on the GPU against the CPU oracle, through the C ABI.

Tolerance: the layer output and the appended cache rows are bf16 results of contractions over
bf16 operands (the normalised activations are rounded to bf16 for the matrix cores): 2e-2
relative / 1e-2 absolute, the bar of the bf16 MoE outputs.  Cache rows the step does not
write must come back bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import attn_ref as R
from paper_2502_06888_amd import attn_binding as A
from paper_2502_06888_amd import inputs as I

from test_attn_ranges import CUT, ranges  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def oracle_group(w, ws, hs, caches):
    raw = {k: I.as_raw(v) for k, v in ws.items()}
    out = []
    for b in range(w.n_batches):
        y, k2, v2 = R.attn_decode(I.as_f32(hs[b]), raw["norm"], raw["wq"], raw["wk"], raw["wv"], raw["wo"],
                                  I.as_raw(caches[b][0]), I.as_raw(caches[b][1]), w.batch_pos[b],
                                  w.n_q_heads, w.n_kv_heads, w.head_dim, w.rope_theta, w.rms_eps)
        out.append((y, k2, v2))
    return out


def widen(bits):
    return torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).to(torch.float64).numpy()


def check_group(w, batches, want):
    for b, (bt, (y, k2, v2)) in enumerate(zip(batches, want)):
        got = bt.h_out.cpu().to(torch.float64).numpy()
        err = np.abs(got - y) - (1e-2 + 2e-2 * np.abs(y))
        assert err.max() <= 0, f"batch {b}: output off by {err.max()} beyond tolerance"
        for name, g, o in (("K", bt.k_cache, k2), ("V", bt.v_cache, v2)):
            gb = I.as_raw(g.cpu())
            pos = w.batch_pos[b]
            keep_mask = np.ones(gb.shape[2], bool)
            keep_mask[pos] = False
            assert np.array_equal(gb[:, :, keep_mask, :], o[:, :, keep_mask, :]), \
                f"batch {b}: {name} rows other than pos changed"
            # the appended row: same bar as the layer output, and much closer than that on average
            gr, orow = widen(gb[:, :, pos, :]), widen(o[:, :, pos, :])
            err = np.abs(gr - orow) - (1e-2 + 2e-2 * np.abs(orow))
            assert err.max() <= 0, f"batch {b}: new {name} row off by {err.max()} beyond tolerance"
            rms = np.sqrt((orow ** 2).mean())
            assert np.abs(gr - orow).mean() <= 4e-3 * rms, \
                f"batch {b}: new {name} row mean error {np.abs(gr - orow).mean() / rms:.2e} of rms"


def run_group(w, on_host, layer=0, ctx=None, set_weights=True, prefetch=None):
    ws = I.gen_attn_weights(w, layer)
    hs = [I.gen_attn_hidden(w, layer, b) for b in range(w.n_batches)]
    caches = [I.gen_kv_cache(w, layer, b) for b in range(w.n_batches)]
    own = ctx is None
    if own:
        ctx = A.AttnContext(A.config_for(w), DEV)
    if set_weights:
        ctx.set_weights(*[ws[n].to(DEV) for n in ("norm", "wq", "wk", "wv", "wo")], layer=layer)
    batches = []
    for b in range(w.n_batches):
        host_b = on_host[b % len(on_host)] if isinstance(on_host, (tuple, list)) else on_host
        if host_b:
            k, v = caches[b][0].clone().pin_memory(), caches[b][1].clone().pin_memory()
            h_in = hs[b].clone().pin_memory()
            h_out = torch.zeros_like(h_in).pin_memory()
        else:
            k, v = caches[b][0].to(DEV), caches[b][1].to(DEV)
            h_in = hs[b].to(DEV)
            h_out = torch.zeros_like(h_in)
        batches.append(A.AttnBatch(k, v, h_in, h_out, w.batch_pos[b]))
    torch.cuda.synchronize()
    if prefetch is not None:
        ctx.prefetch(batches[prefetch])
    ctx.forward_group(batches, layer=layer)
    ctx.synchronize()
    torch.cuda.synchronize()
    check_group(w, batches, oracle_group(w, ws, hs, caches))
    if own:
        ctx.close()


@pytest.mark.parametrize("on_host", [False, True])
def test_tiny_group_matches_oracle(on_host):
    run_group(I.ATTN_WORKLOADS["attn_tiny"], on_host)


def test_device_group_batch_by_batch():
    """A context not sized for the whole group (max_group_seqs = 0) runs a device-resident group
    batch by batch; sized for it, in one pass.  Both against the oracle."""
    w = I.ATTN_WORKLOADS["attn_tiny"]
    for grouped in (False, True):
        ctx = A.AttnContext(A.config_for(w, grouped=grouped), DEV)
        run_group(w, on_host=False, ctx=ctx)
        ctx.close()


@pytest.mark.parametrize("hd,hq,hkv", [(32, 8, 8), (64, 4, 2), (128, 8, 1), (128, 2, 1), (128, 6, 1), (64, 6, 2),
                                       (32, 20, 4), (128, 7, 1)])
def test_head_shapes(hd, hq, hkv):
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv,
                 d_model=256, batch_seqs=(33, 2), batch_pos=(70, 3), max_len=80, seed=3)
    run_group(w, on_host=True)


@pytest.mark.parametrize("hd,hq,hkv,seqs,pos,on_host", [
    (128, 6, 1, (1,), (4000,), False),           # one sequence: as many ranges as pay off
    (128, 8, 1, (2, 1), (1023, 30), False),      # a short cache next to a long one: its last ranges are empty
    (64, 20, 4, (3,), (2047,), True),            # whole loop passes, caches streamed
    (32, 4, 4, (1, 2, 1), (1500, 0, 255), False),
    (128, 5, 1, (1,), (64, ), False),            # just too short to be cut
    (128, 14, 2, (7,), (321,), False)])
def test_long_caches_of_few_sequences_are_cut_into_ranges(hd, hq, hkv, seqs, pos, on_host):
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv,
                 d_model=256, batch_seqs=seqs, batch_pos=pos, max_len=max(pos) + 2, seed=17)
    run_group(w, on_host=on_host)


def quiet(w):
    """Weights, hidden states and caches of a group whose output is the attention's alone: the residual is
    2^-13 of its usual size (normalised all the same, rms_eps is smaller still) and the value rows of the
    new positions are eight times theirs, so that a position lost shows."""
    ws = I.gen_attn_weights(w, 0)
    ws["wv"] = ws["wv"] * 8
    hs = [I.gen_attn_hidden(w, 0, b) * 2.0 ** -13 for b in range(w.n_batches)]
    caches = [I.gen_kv_cache(w, 0, b) for b in range(w.n_batches)]
    return ws, hs, caches


def run_quiet(w, ws, hs, caches, on_host=False):
    ctx = A.AttnContext(A.config_for(w), DEV)
    ctx.set_weights(*[ws[n].to(DEV) for n in ("norm", "wq", "wk", "wv", "wo")])
    put = (lambda t: t.clone().pin_memory()) if on_host else (lambda t: t.to(DEV))
    batches = [A.AttnBatch(put(k), put(v), put(h), put(torch.zeros_like(h)), p)
               for (k, v), h, p in zip(caches, hs, w.batch_pos)]
    torch.cuda.synchronize()
    ctx.forward_group(batches)
    ctx.synchronize()
    torch.cuda.synchronize()
    ctx.close()
    return [b.h_out.cpu() for b in batches]


@pytest.mark.parametrize("hd,hq,hkv,seqs,pos,on_host,n", CUT)
def test_every_range_of_a_cut_cache_counts(hd, hq, hkv, seqs, pos, on_host, n):
    """Relative error of the output of each batch without the residual.  Operands rounded to bf16 (relative
    2^-9 at most, 2^-9 / sqrt(3) on average) enter four times: normalised row, new cache row, attention
    output, result; 2^-9 * 2 = 4e-3 bounds their sum in the 2-norm.  In the oracle the loss of any one
    range is planted: it must move the output by at least three times that."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_model=256,
                 batch_seqs=seqs, batch_pos=pos, max_len=max(pos) + 2, seed=59, rms_eps=1e-14)
    ws, hs, caches = quiet(w)
    want = oracle_group(w, ws, hs, caches)
    got = run_quiet(w, ws, hs, caches, on_host)
    limit = 2.0 ** -8
    for b, (y, (ref, _, _)) in enumerate(zip(got, want)):
        err = np.linalg.norm(y.double().numpy() - ref) / np.linalg.norm(ref)
        assert err <= limit, f"batch {b}: {err:.2e} of the result"
        if n[b] == 1:
            continue
        per = -(-(pos[b] + 1) // n[b])
        for r in sorted({0, 1, n[b] // 2, n[b] - 1}):
            lost, ws2 = [list(c) for c in caches], dict(ws)
            lost[b][1] = lost[b][1].clone()
            lost[b][1][:, :, r * per:(r + 1) * per] = 0
            if r == n[b] - 1:
                ws2["wv"] = torch.zeros_like(ws["wv"])      # the new position is in the last range
            planted = oracle_group(w, ws2, hs, lost)[b][0]
            moved = np.linalg.norm(planted - ref) / np.linalg.norm(ref)
            assert moved >= 3 * limit, f"range {r} of batch {b} moves the result by {moved:.2e} only"


@pytest.mark.parametrize("rising", [True, False])
@pytest.mark.parametrize("hd,hq,hkv,seqs,pos", [(128, 6, 1, 3, 1500), (128, 4, 2, 2, 31), (64, 8, 1, 2, 257),
                                                (32, 8, 4, 5, 700), (128, 8, 1, 1, 16)])
def test_scores_that_rise_or_fall_along_the_cache(hd, hq, hkv, seqs, pos, rising):
    """Scores of standard deviation 0 to 5 (base 2) along the positions: a rising cache moves the running reference
    again and again, a falling one not after the first rows (where a wavefront has several passes: 257 and
    700 positions; the lag itself is tested below, pass by pass).  The 2-norm bound of
    the ranges' test, plus what an error of 2^-9 of a score does to its weight: scores reach 5 standard
    deviations of 5, 25 * ln 2 * 2^-9 = 3.4e-2 of a single weight, less on average."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_model=256,
                 batch_seqs=(seqs,), batch_pos=(pos,), max_len=pos + 2, seed=71, rms_eps=1e-14)
    ws, hs, caches = quiet(w)
    h = hs[0].double()
    q = (h / h.pow(2).mean(1, keepdim=True).sqrt() * ws["norm"].double()) @ ws["wq"].double().T
    size = q.reshape(seqs, hq, hd).norm(dim=2).mean() * 1.4427 / hd ** 0.5  # of a score with unit normal keys
    ramp = torch.linspace(0, 5, pos, dtype=torch.float64) if rising else torch.linspace(5, 0, pos, dtype=torch.float64)
    k, v = caches[0]
    gen = torch.Generator().manual_seed(73)
    k = k.clone()
    k[:, :, :pos] = (torch.randn(seqs, hkv, pos, hd, generator=gen).double() * (ramp / size)[:, None]).to(k.dtype)
    want = oracle_group(w, ws, hs, [(k, v)])[0][0]
    got = run_quiet(w, ws, hs, [(k, v)])[0].double().numpy()
    assert np.linalg.norm(got - want) <= (2.0 ** -8 + 25 * np.log(2) * 2.0 ** -9) * np.linalg.norm(want)


def group_queries(w, ws, h):
    """The first batch's rotated queries in 64 bits: [sequences, kv heads, queries of the group, head_dim]."""
    norm, wq = (I.as_f32(ws[n]).astype(np.float64) for n in ("norm", "wq"))
    q = np.stack([R.rmsnorm(r, norm, w.rms_eps) for r in I.as_f32(h)]) @ wq.T
    q = np.stack([R.rope(v, w.batch_pos[0], w.rope_theta) for v in q.reshape(-1, w.head_dim)])
    return q.reshape(h.shape[0], w.n_kv_heads, -1, w.head_dim)


# Score (base 2) of every position of a loop pass over the cache, pass by pass
LEVELS = {"late": lambda p: np.array([0, 6, 9.5])[np.minimum(p, 2)],        # 6 below the lag of 8, then past it
          "far": lambda p: np.where(p == 0, 0, 140.0),                      # a reference left behind overflows
          "falling": lambda p: np.array([0, -5, -9])[np.minimum(p, 2)],
          "saw": lambda p: 9.5 * (p % 3),
          "limit": lambda p: np.where(p == 0, 0, 7.0)}                      # values near the limit of fp32, see below


@pytest.mark.parametrize("mode", list(LEVELS))
@pytest.mark.parametrize("hd,hq,hkv,seqs,pos,cut", [
    (128, 6, 1, 3, 200, False), (128, 8, 2, 2, 150, False), (128, 5, 1, 1, 97, False), (64, 8, 1, 2, 257, False),
    (32, 4, 4, 2, 600, False), (128, 12, 2, 20, 2500, True), (128, 4, 1, 70, 2500, True)])
def test_scores_that_step_from_pass_to_pass(ranges, hd, hq, hkv, seqs, pos, cut, mode):  # noqa: F811
    """Keys along the queries' pseudo-inverse give all positions of a loop pass one score, which rises below the
    lag of the running reference, past it, far past it, falls, or both.  Every wavefront has three passes or
    more, whole caches and cut ones.  With values of 2^119 to 2^120 the sums of weights of 2^7 leave fp32 in a
    slot of a wavefront (four rows or more: 2^(7 + 119 + 2)), with the 2^115 of longer caches where slots and
    wavefronts meet (124 rows or more); those of weights up to 1 do neither.  Bound: the ranges' test's, plus
    the weights' error: 2^-9 of the largest score that is weighed against another one."""
    step = 4 * (512 // hd) * 2
    n = ranges(pos + 1, seqs * hkv, hq // hkv, hd)
    assert (n > 1) == cut and (pos + 1) // n >= 3 * step
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_model=256,
                 batch_seqs=(seqs,), batch_pos=(pos,), max_len=pos + 2, seed=71, rms_eps=1e-14)
    ws, hs, caches = quiet(w)
    unit = np.linalg.pinv(group_queries(w, ws, hs[0])).sum(-1) * hd ** 0.5 * np.log(2)                  # scores 1 with every query of the group
    level = LEVELS[mode](np.arange(pos) // step)
    k, v = (t.clone() for t in caches[0])
    k[:, :, :pos] = torch.from_numpy(unit[:, :, None] * level[:, None]).to(k.dtype)
    if mode == "limit":
        gen = torch.Generator().manual_seed(79)
        v[:, :, :pos] = ((1 + torch.rand(v[:, :, :pos].shape, generator=gen)) * 2.0 ** (119 if pos <= 200 else 115)).to(v.dtype)
    want = oracle_group(w, ws, hs, [(k, v)])[0][0]
    got = run_quiet(w, ws, hs, [(k, v)])[0].double().numpy()
    finite = bool(np.isfinite(got).all())
    assert finite
    weighed = {"far": 0, "limit": 0, "saw": 19}.get(mode, 9.5)
    err = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    assert err <= 2.0 ** -8 + weighed * np.log(2) * 2.0 ** -9


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("hd,hq,hkv,seqs,pos", [(128, 4, 1, 3, 200), (128, 6, 1, 2, 200), (32, 4, 4, 2, 600)])
def test_an_infinite_score_behind_the_first_pass(hd, hq, hkv, seqs, pos, sign):
    """-inf is a position without weight; +inf makes its sequence NaN and no other.  Bound: the ranges' test's,
    plus 2^-9 of the largest score's distance (5 standard deviations of about 2 around the mean)."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=hd, n_q_heads=hq, n_kv_heads=hkv, d_model=256,
                 batch_seqs=(seqs,), batch_pos=(pos,), max_len=pos + 2, seed=71, rms_eps=1e-14)
    ws, hs, caches = quiet(w)
    q = group_queries(w, ws, hs[0])[0, 0]                   # of sequence 0's first key-value head: [queries, hd]
    j = int(np.argmax(np.abs(np.sign(q).sum(0))))           # the element most of them agree on the sign of
    if abs(np.sign(q[:, j]).sum()) < len(q):
        pytest.skip("no element with one sign")
    k, v = (t.clone() for t in caches[0])
    k[0, 0, pos * 2 // 3, j] = float("inf") * float(np.sign(q[0, j])) * sign
    got = run_quiet(w, ws, hs, [(k, v)])[0].double().numpy()
    if sign > 0:
        assert bool(np.isnan(got[0]).all())
        k = caches[0][0]
    want = oracle_group(w, ws, hs, [(k, v)])[0][0]
    first = 1 if sign > 0 else 0
    err = float(np.linalg.norm(got[first:] - want[first:]) / np.linalg.norm(want[first:]))
    assert err <= 2.0 ** -8 + 10 * np.log(2) * 2.0 ** -9


def test_a_sequence_does_not_depend_on_the_lengths_of_the_others():
    """The same first batch beside short and beside long caches, same number of rows: same bits."""
    outs = []
    for other in (3, 700, 3000):
        w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=128, n_q_heads=8, n_kv_heads=1, d_model=256,
                     batch_seqs=(24, 2), batch_pos=(900, other), max_len=3008, seed=61, rms_eps=1e-14)
        ws, hs, caches = quiet(w)
        outs.append(run_quiet(w, ws, hs, caches)[0])
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("pos", [321, 30])
def test_infinite_values_in_a_cache_row_stay_infinite(pos):
    """One infinite element of a value row (first and last rows of the ranges of 30 positions that the
    longer cache is cut into): the heads that read it are infinite there, not NaN, whatever rows the kernel
    reads beside it with weight zero.  Output weights all alike: such a sequence's outputs are infinite,
    the others' are untouched."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], head_dim=128, n_q_heads=4, n_kv_heads=2, d_model=256,
                 batch_seqs=(7,), batch_pos=(pos,), max_len=324, seed=67, rms_eps=1e-14)
    ws, hs, caches = quiet(w)
    ws["wo"] = torch.full_like(ws["wo"], 0.0625)
    clean = run_quiet(w, ws, hs, caches)[0]
    for row in (0, 29, 30, 59, 300, pos - 1):
        if row >= pos:
            continue
        k, v = caches[0][0], caches[0][1].clone()
        v[3, 1, row, 5] = float("inf")
        y = run_quiet(w, ws, hs, [(k, v)])[0]
        assert (y[3] == float("inf")).all(), f"row {row}: {y[3, :4]}"
        y[3] = clean[3]
        assert torch.equal(y, clean)


def test_ragged_rows_and_several_row_tiles():
    # 130 sequences: five row blocks -> two row tiles of four blocks, the last one ragged
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64,
                 batch_seqs=(130, 1, 64), batch_pos=(9, 255, 128), max_len=256, seed=5)
    run_group(w, on_host=False)
    run_group(w, on_host=True)


@pytest.mark.parametrize("rows,hq,hkv,hd", [(512, 8, 8, 64), (513, 8, 8, 64),    # 4 workgroups per row: 2048, and 2052
                                            (682, 8, 1, 128), (683, 8, 1, 128)])  # 3: 2046, and 2049; nine heads in pairs
def test_rotation_of_one_or_two_heads_per_thread(rows, hq, hkv, hd):
    """Around the line between one and two heads per thread; an odd number of heads leaves one alone."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd,
                 batch_seqs=(rows - 2, 2), batch_pos=(5, 11), max_len=16, seed=71)
    run_group(w, on_host=False)


def test_group_mixing_host_and_device_batches():
    """Batches whose caches live on the host next to batches that live on the device, in both
    alternations and with a run of device batches between two host batches."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], batch_seqs=(4, 7, 2, 9, 3, 5), batch_pos=(11, 30, 0, 47, 8, 21), seed=11)
    ctx = A.AttnContext(A.config_for(w), DEV)
    run_group(w, on_host=(True, False), ctx=ctx)
    run_group(w, on_host=(False, True), ctx=ctx)
    run_group(w, on_host=(True, False, False, False, True, False), ctx=ctx)
    ctx.close()


@pytest.mark.parametrize("n_batches", [64, 66])
def test_many_small_batches(n_batches):
    """64 batches is the most one pass over a device-resident group takes; 66 fall back to the
    batch-by-batch loop.  One or two sequences per batch, positions all different."""
    seqs = tuple(1 + (b % 2) for b in range(n_batches))
    pos = tuple((7 * b) % 47 for b in range(n_batches))
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], batch_seqs=seqs, batch_pos=pos, seed=13)
    run_group(w, on_host=False)


def test_empty_group_and_full_cache():
    w = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], batch_seqs=(8,), batch_pos=(47,), seed=17)   # last free position
    ctx = A.AttnContext(A.config_for(w), DEV)
    run_group(w, on_host=True, ctx=ctx)
    run_group(w, on_host=False, ctx=ctx)
    ctx.forward_group([])            # nothing to do, no error
    ctx.synchronize()
    ctx.close()


def test_context_reuse_with_shrinking_batches():
    big = I.scaled(I.ATTN_WORKLOADS["attn_tiny"], batch_seqs=(8, 8, 8, 8, 8), batch_pos=(40, 41, 42, 43, 44), seed=7)
    small = I.scaled(big, batch_seqs=(3, 2), batch_pos=(5, 0), seed=8)
    ctx = A.AttnContext(A.config_for(big), DEV)
    run_group(big, True, ctx=ctx)
    run_group(small, True, ctx=ctx)
    run_group(big, False, ctx=ctx)
    ctx.close()


def test_several_layers_in_one_context():
    """Three layers' weights in one context, used out of order; inputs differ per layer."""
    w = I.ATTN_WORKLOADS["attn_tiny"]
    ctx = A.AttnContext(A.config_for(w, n_layers=3), DEV)
    for layer in (2, 0, 1):
        ws = I.gen_attn_weights(w, layer)
        ctx.set_weights(*[ws[n].to(DEV) for n in ("norm", "wq", "wk", "wv", "wo")], layer=layer)
    for layer in (1, 2, 0, 2):
        run_group(w, on_host=(layer != 1), layer=layer, ctx=ctx, set_weights=False)
    from paper_2502_06888_amd import binding as B
    with pytest.raises(B.MoeError) as ei:
        run_group(w, on_host=False, layer=3, ctx=ctx, set_weights=False)
    assert ei.value.status == B.MOE_ERR_INVALID_ARG
    ctx.close()


def test_prefetch_of_the_first_batch():
    """The first batch's caches brought in ahead of the call (and a prefetch of some other batch,
    which the call must ignore): same results; the call then loads fewer bytes."""
    w = I.ATTN_WORKLOADS["attn_tiny"]
    ctx = A.AttnContext(A.config_for(w), DEV)
    ctx.set_profiling(1)
    run_group(w, on_host=True, ctx=ctx)
    plain = ctx.profile().bytes_loaded
    run_group(w, on_host=True, ctx=ctx, prefetch=0)
    ahead = ctx.profile().bytes_loaded
    run_group(w, on_host=True, ctx=ctx, prefetch=2)
    other = ctx.profile().bytes_loaded
    assert plain - ahead == w.kv_bytes(0) and other == plain
    run_group(w, on_host=False, ctx=ctx, prefetch=0)   # device-resident caches: nothing to move
    ctx.close()


def test_argument_errors():
    from paper_2502_06888_amd import binding as B
    w = I.ATTN_WORKLOADS["attn_tiny"]
    ctx = A.AttnContext(A.config_for(w), DEV)
    k, v = [t.to(DEV) for t in I.gen_kv_cache(w, 0, 0)]
    h = I.gen_attn_hidden(w, 0, 0).to(DEV)
    with pytest.raises(B.MoeError) as ei:
        ctx.forward_group([A.AttnBatch(k, v, h, h, 1)])
    assert ei.value.status == B.MOE_ERR_STATE
    ws = I.gen_attn_weights(w, 0)
    ctx.set_weights(*[ws[n] for n in ("norm", "wq", "wk", "wv", "wo")])   # plain host tensors
    with pytest.raises(B.MoeError) as ei:
        ctx.forward_group([A.AttnBatch(k, v, h, h, w.max_len)])
    assert ei.value.status == B.MOE_ERR_INVALID_ARG
    with pytest.raises(B.MoeError) as ei:   # pageable host memory where pinned is required
        ctx.forward_group([A.AttnBatch(k.cpu(), v.cpu(), h, h, 1)])
    assert ei.value.status == B.MOE_ERR_NOT_PINNED
    ctx.forward_group([A.AttnBatch(k, v, h, h, w.batch_pos[0])])          # in place, still usable
    ctx.synchronize()
    ctx.close()
    with pytest.raises(B.MoeError) as ei:
        A.workspace_bytes(A.MoeAttnConfig(200, 8, 2, 32, 4, 16, 1, 0, 1e4, 1e-5))
    assert ei.value.status == B.MOE_ERR_SHAPE


def test_full_size_sampled_sequences():
    """Mixtral-8x7B attention shape in the launch configuration the benchmark times (64 sequences
    per batch, 512 cached positions, caches streamed from pinned host memory); the oracle checks a
    sample of sequences one by one (rows of a batch are independent of each other)."""
    w = I.scaled(I.ATTN_WORKLOADS["attn_mixtral8x7b_decode"], batch_seqs=(64, 64, 37), batch_pos=(512, 512, 575))
    ws = I.gen_attn_weights(w, 0)
    hs = [I.gen_attn_hidden(w, 0, b) for b in range(w.n_batches)]
    caches = [I.gen_kv_cache(w, 0, b) for b in range(w.n_batches)]
    ctx = A.AttnContext(A.config_for(w), DEV)
    ctx.set_weights(*[ws[n].to(DEV) for n in ("norm", "wq", "wk", "wv", "wo")])
    batches = []
    for b in range(w.n_batches):
        h_in = hs[b].clone().pin_memory()
        batches.append(A.AttnBatch(caches[b][0].clone().pin_memory(), caches[b][1].clone().pin_memory(),
                                   h_in, torch.zeros_like(h_in).pin_memory(), w.batch_pos[b]))
    ctx.forward_group(batches)
    ctx.synchronize()
    raw = {k: I.as_raw(v) for k, v in ws.items()}
    for b, rows in ((0, [0, 31, 63]), (1, [32]), (2, [0, 36])):
        pos = w.batch_pos[b]
        y, k2, v2 = R.attn_decode(I.as_f32(hs[b])[rows], raw["norm"], raw["wq"], raw["wk"], raw["wv"], raw["wo"],
                                  I.as_raw(caches[b][0])[rows], I.as_raw(caches[b][1])[rows], pos,
                                  w.n_q_heads, w.n_kv_heads, w.head_dim, w.rope_theta, w.rms_eps)
        got = batches[b].h_out.to(torch.float64).numpy()[rows]
        err = np.abs(got - y) - (1e-2 + 2e-2 * np.abs(y))
        assert err.max() <= 0, f"batch {b}: output off by {err.max()} beyond tolerance"
        for name, g, o in (("K", batches[b].k_cache, k2), ("V", batches[b].v_cache, v2)):
            gr, orow = widen(I.as_raw(g)[rows][:, :, pos, :]), widen(o[:, :, pos, :])
            err = np.abs(gr - orow) - (1e-2 + 2e-2 * np.abs(orow))
            assert err.max() <= 0, f"batch {b}: new {name} row off by {err.max()} beyond tolerance"
    # properties that hold for every sequence: cache rows before pos untouched, outputs finite
    for b in range(w.n_batches):
        pos = w.batch_pos[b]
        assert torch.equal(batches[b].k_cache[:, :, :pos], caches[b][0][:, :, :pos])
        assert torch.equal(batches[b].v_cache[:, :, :pos], caches[b][1][:, :, :pos])
        assert torch.isfinite(batches[b].h_out.float()).all()
    ctx.close()


def test_full_size_one_pass_group():
    """The benchmark's device-resident configuration (8 batches x 64 sequences, 512 cached
    positions, caches in HBM, the whole group in one pass); sampled sequences against the oracle,
    properties on all."""
    w = I.ATTN_WORKLOADS["attn_mixtral8x7b_decode_hbm"]
    ws = I.gen_attn_weights(w, 0)
    hs = [I.gen_attn_hidden(w, 0, b) for b in range(w.n_batches)]
    caches = [I.gen_kv_cache(w, 0, b) for b in range(w.n_batches)]
    ctx = A.AttnContext(A.config_for(w), DEV)
    ctx.set_weights(*[ws[n].to(DEV) for n in ("norm", "wq", "wk", "wv", "wo")])
    group_in = torch.cat(hs).to(DEV)                 # hidden states of the group as one tensor
    group_out = torch.zeros_like(group_in)
    batches, r0 = [], 0
    for b in range(w.n_batches):
        n = w.batch_seqs[b]
        batches.append(A.AttnBatch(caches[b][0].to(DEV), caches[b][1].to(DEV), group_in[r0:r0 + n],
                                   group_out[r0:r0 + n], w.batch_pos[b]))
        r0 += n
    ctx.forward_group(batches)
    ctx.synchronize()
    raw = {k: I.as_raw(v) for k, v in ws.items()}
    for b, rows in ((0, [0, 63]), (3, [17]), (7, [62])):
        pos = w.batch_pos[b]
        y, k2, v2 = R.attn_decode(I.as_f32(hs[b])[rows], raw["norm"], raw["wq"], raw["wk"], raw["wv"], raw["wo"],
                                  I.as_raw(caches[b][0])[rows], I.as_raw(caches[b][1])[rows], pos,
                                  w.n_q_heads, w.n_kv_heads, w.head_dim, w.rope_theta, w.rms_eps)
        got = batches[b].h_out.cpu().to(torch.float64).numpy()[rows]
        err = np.abs(got - y) - (1e-2 + 2e-2 * np.abs(y))
        assert err.max() <= 0, f"batch {b}: output off by {err.max()} beyond tolerance"
        for name, g, o in (("K", batches[b].k_cache, k2), ("V", batches[b].v_cache, v2)):
            gr, orow = widen(I.as_raw(g[rows].cpu())[:, :, pos, :]), widen(o[:, :, pos, :])
            err = np.abs(gr - orow) - (1e-2 + 2e-2 * np.abs(orow))
            assert err.max() <= 0, f"batch {b}: new {name} row off by {err.max()} beyond tolerance"
    for b in range(w.n_batches):
        pos = w.batch_pos[b]
        assert torch.equal(batches[b].k_cache[:, :, :pos].cpu(), caches[b][0][:, :, :pos])
        assert torch.equal(batches[b].v_cache[:, :, :pos].cpu(), caches[b][1][:, :, :pos])
    assert torch.isfinite(group_out.float()).all() and (group_out != 0).any(dim=1).all()
    ctx.close()


@pytest.mark.parametrize("seed", list(range(12)))
def test_seeded_sweep_of_attention_shapes(seed):
    """Head shapes, group sizes, widths, batch structures and positions drawn from a seeded
    generator; caches on the host, on the device, or mixed."""
    g = np.random.Generator(np.random.PCG64(2000 + seed))
    hd = int(g.choice([32, 64, 128]))
    per128 = 128 // hd                       # query heads come in multiples that make Hq*hd % 128 == 0
    group = int(g.integers(1, 9))
    hkv_unit = per128 // np.gcd(per128, group) if per128 > 1 else 1
    hkv = int(hkv_unit * g.integers(1, 3))
    hq = hkv * group
    if (hq * hd) % 128 != 0 or (hkv * hd) % 32 != 0:
        pytest.skip("draw outside the supported head shapes")
    d = int(g.integers(1, 5)) * 128
    nb = int(g.integers(1, 6))
    max_len = int(g.integers(8, 200))
    seqs = tuple(int(v) for v in g.integers(1, 40, size=nb))
    pos = tuple(int(v) for v in g.integers(0, max_len, size=nb))
    w = I.AttnWorkload(f"asweep{seed}", d, hq, hkv, hd, seqs, pos, max_len, rope_theta=float(g.choice([1e4, 1e6])),
                       seed=seed)
    where = [True, False, (True, False), (False, True)][seed % 4]
    run_group(w, on_host=where)
