"""The attention backward's chunk lists: group ids in any order, repeated,
padded in the middle, in the causal future or inside an always-visible chunk;
lists long enough to be cut (sinks); 8-, 16- and 32-token groups; a few query
chunks after a long history, where the lists no longer fit the dq buffer; and
gradients added to what dk and dv hold."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import hga_oracle as O
from paper_2606_30709_amd import workloads as W

from parity_util import BWD_TOL, f64

pytestmark = pytest.mark.gpu


def _check(w, q0, gi, seed):
    """Backward of the last chunks from q0 on for group ids gi, against the oracle."""
    from paper_2606_30709_amd import hga
    rng = np.random.default_rng(seed)
    C, d, G = w.chunk, w.head_dim, w.group
    n = w.n_chunks - q0
    bf = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(torch.bfloat16)  # noqa: E731
    q, dout = bf(w.batch, w.n_q_heads, n * C, d), bf(w.batch, w.n_q_heads, n * C, d)
    k, v = bf(w.batch, w.n_kv_heads, w.seq_len, d), bf(w.batch, w.n_kv_heads, w.seq_len, d)
    dev = [t.cuda() for t in (q, k, v, dout)]
    plan = hga.Plan.for_workload(w)
    out = torch.empty_like(dev[0])
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    ids = torch.from_numpy(gi.astype(np.int32)).cuda()
    hga.hga_gather_attend(plan, dev[0], q0, dev[1], dev[2], ids, None, None, out, lse)
    base = torch.from_numpy(rng.standard_normal(k.shape).astype(np.float32)).cuda()
    dq = torch.full(q.shape, float("nan"), device="cuda")
    dk, dv = base.clone(), -base
    hga.hga_attend_backward(plan, dev[0], q0, dev[1], dev[2], ids, out, lse, dev[3], dq, dk, dv)
    torch.cuda.synchronize()
    valid = gi.copy()
    for i in range(n):  # absent: outside the causal past
        row = valid[:, :, i]
        row[(row < 0) | (row >= (q0 + i) * (C // G))] = -1
    # the writing form: the same sums over zeros, whatever the buffers held; the
    # rows of a resident buffer past the last chunk are written too
    pad = [torch.cat([t, torch.full_like(t[:, :, :70], float("nan"))], 2) for t in dev[1:3]]
    wq = torch.full_like(dq, float("nan"))
    wk = torch.full(pad[0].shape, float("nan"), device="cuda")
    wv = wk.clone()
    hga.hga_attend_backward_write(plan, dev[0], q0, pad[0], pad[1], ids, out, lse, dev[3], wq, wk, wv)
    torch.cuda.synchronize()
    assert torch.equal(wq, dq)
    for got, added in ((wk, dk - base), (wv, dv + base)):
        tail = got[:, :, w.seq_len:]
        assert bool((tail == 0).all())
        top = added.abs().max()
        assert (got[:, :, :w.seq_len] - added).abs().max() <= 1e-5 * (top + base.abs().max())
    x = [f64(t.view(torch.int16).numpy().view(np.uint16), "bf16") for t in (q, k, v, dout)]
    ref = O.attend_backward(x[0], x[1], x[2], x[3], valid, list(range(q0, w.n_chunks)), C, G,
                            w.keep_first, w.keep_last, w.force_prev)
    b = base.cpu().double().numpy()
    for name, got, want in zip(("dq", "dk", "dv"), (dq, dk, dv), (ref[0], ref[1] + b, ref[2] - b)):
        err = np.abs(got.double().cpu().numpy() - want)
        grad = want - (0 if name == "dq" else (b if name == "dk" else -b))
        assert np.isfinite(err).all(), name
        assert err.max() <= BWD_TOL * np.abs(grad).max(), name
        assert np.linalg.norm(err) <= BWD_TOL / 4 * np.linalg.norm(grad), name


def _ids(w, q0, rng):
    """Random valid ids with repeats, then the odd ones the calls accept."""
    n, gpc = w.n_chunks - q0, w.chunk // w.group
    gi = np.full((w.batch, w.n_kv_heads, n, w.topk_groups), -1, dtype=np.int64)
    for i in range(n):
        c = q0 + i
        if c > 1:
            # ids of a few chunks, so that runs and repeats occur, any order
            lo = int(rng.integers(0, max(1, c - 4)))
            gi[:, :, i] = rng.integers(lo * gpc, min(c, lo + 4) * gpc, size=gi[:, :, i].shape)
            if i % 3 == 0:
                gi[:, :, i] = np.sort(gi[:, :, i], axis=-1)
            if i % 4 == 1:
                gi[:, :, i, w.topk_groups // 2] = -1
            if i % 5 == 2:
                gi[:, :, i, 0] = c * gpc       # the causal future
    return gi


@pytest.mark.parametrize("d,group,kv,ratio,kg,first,last", [
    (64, 16, 3, 1, 12, 1, 0),
    (64, 8, 1, 2, 21, 2, 3),
    (64, 32, 2, 3, 5, 1, 1),
    (64, 16, 1, 8, 7, 0, 2),
    (128, 16, 2, 1, 9, 1, 2),
    (128, 8, 1, 4, 13, 1, 0),
    (128, 32, 1, 7, 4, 2, 1),
    (128, 16, 1, 8, 6, 1, 1),     # unit by unit
])
def test_backward_group_id_forms(d, group, kv, ratio, kg, first, last):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    w = W.preset("smalllm").with_(batch=1, n_q_heads=kv * ratio, n_kv_heads=kv, head_dim=d,
                                  seq_len=64 * 21, group=group, topk_groups=kg, topk_chunks=4,
                                  keep_first=first, keep_last=last, needle_mode="none")
    rng = np.random.default_rng(d + group + kg)
    for q0 in (0, 17):
        _check(w, q0, _ids(w, q0, rng), seed=kg + q0)


@pytest.mark.parametrize("d,group,ratio,kg,first,last", [
    (64, 16, 2, 12, 1, 0),
    (64, 8, 3, 21, 2, 3),
    (64, 32, 7, 5, 1, 1),
    (128, 16, 2, 9, 1, 2),
    (128, 8, 4, 13, 1, 0),
    (128, 32, 5, 4, 2, 1),
])
def test_backward_lists_of_several_heads(d, group, ratio, kg, first, last):
    """Several query heads per KV head in launches large enough for the lists
    (smaller ones go unit by unit)."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    tiles = 1 + first + max(last, 1) + -(-kg * group // 64)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    batch = -(-8 * n_cu // (21 * tiles))
    w = W.preset("smalllm").with_(batch=batch, n_q_heads=ratio, n_kv_heads=1, head_dim=d,
                                  seq_len=64 * 21, group=group, topk_groups=kg, topk_chunks=4,
                                  keep_first=first, keep_last=last, needle_mode="none")
    _check(w, 0, _ids(w, 0, np.random.default_rng(d + kg)), seed=kg)


@pytest.mark.parametrize("d,chunks,q0", [
    (64, 2050, 2049),    # the lists do not fit one query chunk's dq
    (64, 2050, 2042),    # they fit eight's, unit by unit is the faster
    (64, 2050, 2026),    # chunk by chunk
    (64, 16410, 16370),
    (64, 16400, 16240),  # key chunks in two ranges
    (128, 70, 69),
    (128, 70, 66),
])
def test_backward_few_query_chunks_after_a_long_history(d, chunks, q0):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    w = W.preset("smalllm").with_(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d,
                                  seq_len=64 * chunks, topk_groups=12, topk_chunks=8,
                                  needle_mode="none")
    rng = np.random.default_rng(chunks + q0)
    gi = np.sort(rng.integers(0, q0 * 4, size=(1, 1, chunks - q0, 12)), axis=-1)
    _check(w, q0, gi, seed=q0)


@pytest.mark.parametrize("d,kv,ratio,q_ranges", [
    (64, 4, 1, False),      # micro-batches: the same queries' chunks, other gradients
    (64, 4, 1, True),       # query ranges of one sequence
    (128, 2, 2, True),
])
def test_overlapping_backwards_add_into_the_same_gradients(d, kv, ratio, q_ranges):
    """Calls on several streams that add into one dk and dv lose no sum."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2606_30709_amd import hga
    nc, n_calls = 96, 4
    w = W.preset("smalllm").with_(batch=2, n_q_heads=kv * ratio, n_kv_heads=kv, head_dim=d,
                                  seq_len=64 * nc, topk_groups=12, topk_chunks=8,
                                  needle_mode="none")
    plan = hga.Plan.for_workload(w)
    g = torch.Generator(device="cuda").manual_seed(d + ratio)
    bf = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    k, v = bf(2, kv, 64 * nc, d), bf(2, kv, 64 * nc, d)
    calls = []
    for i in range(n_calls):
        q0, n = (i * nc // n_calls, nc // n_calls) if q_ranges else (0, nc)
        q, dout = bf(2, kv * ratio, n * 64, d), bf(2, kv * ratio, n * 64, d)
        top = torch.arange(q0, q0 + n, device="cuda").view(1, 1, n, 1) * 4
        ids = (torch.rand(2, kv, n, 12, generator=g, device="cuda") * top).int().sort(-1).values
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
        hga.hga_gather_attend(plan, q, q0, k, v, ids, None, None, out, lse)
        calls.append((q, q0, ids, out, lse, dout, torch.empty(q.shape, device="cuda")))

    def add(call, dk, dv, stream=None):
        q, q0, ids, out, lse, dout, dq = call
        hga.hga_attend_backward(plan, q, q0, k, v, ids, out, lse, dout, dq, dk, dv, stream=stream)

    want = [torch.zeros(k.shape, dtype=torch.float64, device="cuda") for _ in range(2)]
    for call in calls:
        one = [torch.zeros(k.shape, device="cuda") for _ in range(2)]
        add(call, *one)
        for s, x in zip(want, one):
            s += x
    for _ in range(3):
        got = [torch.zeros(k.shape, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in calls]
        for call, s in zip(calls, streams):
            add(call, *got, stream=s)
        torch.cuda.synchronize()
        for x, ref in zip(got, want):
            assert (x.double() - ref).abs().max() <= 1e-5 * ref.abs().max()


@pytest.mark.parametrize("d,group,kg", [(64, 8, 5), (64, 16, 3), (64, 32, 2), (128, 8, 4), (128, 16, 5)])
def test_rows_that_no_query_attends(d, group, kg):
    """A chunk of which only some groups were opened: the other groups' rows
    are not added to (minus zeros stay) and are zeros in the writing form,
    whatever their keys hold."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2606_30709_amd import hga
    nc, n, kv, gpc = 40, 12, 2, 64 // group
    w = W.preset("smalllm").with_(batch=1, n_q_heads=kv, n_kv_heads=kv, head_dim=d, seq_len=64 * nc,
                                  group=group, topk_groups=kg, topk_chunks=kg, needle_mode="none")
    plan, q0 = hga.Plan.for_workload(w), nc - n
    g = torch.Generator(device="cuda").manual_seed(d + group)
    bf = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    q, dout = bf(1, kv, n * 64, d), bf(1, kv, n * 64, d)
    k, v = bf(1, kv, 64 * nc, d), bf(1, kv, 64 * nc, d)
    # groups 0, 2, .. of a chunk (0 and 1 of two): never its last
    ids = torch.randint(2, q0 - 2, (1, kv, n, kg), generator=g, device="cuda") * gpc
    ids = (ids + torch.randint(0, max(1, gpc // 2), ids.shape, generator=g, device="cuda") * 2).int()
    ids = ids.sort(-1).values
    seen = torch.zeros(kv, 64 * nc, dtype=torch.bool, device="cuda")
    for i in range(n):
        for c in [q0 + i, *hga.hga_visible_chunks(plan.params, q0 + i)]:
            seen[:, c * 64:(c + 1) * 64] = True
    for h in range(kv):
        for x in ids[0, h].unique().tolist():
            seen[h, x * group:(x + 1) * group] = True
    partly = seen.view(kv, nc, 64)
    assert bool((partly.any(-1) & ~partly.all(-1)).any())
    k[0][~seen], v[0][~seen] = float("nan"), float("inf")
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
    hga.hga_gather_attend(plan, q, q0, k, v, ids, None, None, out, lse)
    dq = torch.empty(q.shape, device="cuda")
    for fn, before, after in ((hga.hga_attend_backward, -0.0, -2 ** 31), (hga.hga_attend_backward_write, float("nan"), 0)):
        dk, dv = (torch.full(k.shape, before, device="cuda") for _ in range(2))
        fn(plan, q, q0, k, v, ids, out, lse, dout, dq, dk, dv)
        torch.cuda.synchronize()
        for x in (dk[0], dv[0]):
            assert bool((x[~seen].view(torch.int32) == after).all())
            assert bool(x[seen].isfinite().all()) and bool((x[seen] != 0).any())
