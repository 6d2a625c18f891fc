"""The split attention's two kernels: workgroups that each leave a partial
result for a merge kernel, and (launches of a few query tiles) one workgroup
for all splits of a query tile.  They form the same sums in the same order, so
no call's bits depend on which of them it takes."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import hga_oracle as O
from paper_2606_30709_amd import workloads as W

from parity_util import LSE_TOL, OUT_TOL, tensor_to_f64

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def _same(a, b):
    return torch.equal(_bits(a), _bits(b))


class _Case:
    """Random inputs of `n` query chunks after `q0`, with ids of the causal
    past, some padded, repeated or in the future."""

    def __init__(self, d, kv, ratio, group, kg, first, last, q0, n, batch=1, seed=0, distinct=False):
        if not torch.cuda.is_available():
            pytest.skip("needs a GPU")
        from paper_2606_30709_amd import hga
        self.hga = hga
        self.w = w = W.preset("qwen32k").with_(
            batch=batch, n_q_heads=kv * ratio, n_kv_heads=kv, head_dim=d, seq_len=64 * (q0 + n),
            group=group, topk_groups=kg, topk_chunks=min(kg, 8), keep_first=first, keep_last=last,
            needle_mode="none")
        self.plan, self.q0, self.n = hga.Plan.for_workload(w), q0, n
        g = torch.Generator().manual_seed(seed)
        bf = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16).cuda()  # noqa: E731
        self.q = bf(batch, kv * ratio, n * 64, d) * 3
        self.k, self.v = bf(batch, kv, 64 * (q0 + n), d), bf(batch, kv, 64 * (q0 + n), d)
        rng = np.random.default_rng(seed)
        gpc = 64 // group
        gi = np.full((batch, kv, n, kg), -1, dtype=np.int32)
        for i in range(n):
            c = q0 + i
            if c:
                draw = ((lambda: rng.choice(c * gpc, kg, replace=False)) if distinct else
                        (lambda: rng.integers(0, c * gpc, size=kg)))
                gi[:, :, i] = [[np.sort(draw()) for _ in range(kv)] for _ in range(batch)]
                if i % 3 == 1:
                    gi[:, :, i, kg // 2:] = -1
                if i % 4 == 2:
                    gi[:, :, i, 0] = c * gpc
        self.gi = torch.from_numpy(gi).cuda()
        self.kr = torch.full((batch, kv, n, kg * group, d), float("nan"), dtype=torch.bfloat16,
                             device="cuda")
        self.vr = self.kr.clone()
        hga.hga_gather_kv(self.plan, self.gi, q0, self.k, self.v, self.kr, self.vr)

    def split_bytes(self, n):
        """Bytes of one split of n query chunks."""
        return self.hga.hga_attend_split_workspace(self.plan, n) // 16

    def attend_split(self, i, n, workspace_bytes):
        s = slice(i * 64, (i + n) * 64)
        q = self.q[:, :, s].contiguous()
        out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
        ws = torch.full((workspace_bytes // 4,), float("nan"), device="cuda")
        self.hga.hga_attend_split(self.plan, q, self.q0 + i, self.k, self.v,
                                  self.kr[:, :, i:i + n].contiguous(),
                                  self.vr[:, :, i:i + n].contiguous(),
                                  self.gi[:, :, i:i + n].contiguous(), out, ws, lse)
        torch.cuda.synchronize()
        return out, lse


@pytest.mark.parametrize("d,kv,ratio,group,kg,first,last,q0,n", [
    (128, 1, 2, 16, 9, 1, 0, 9, 70),       # 3 splits of a 5-tile unit
    (128, 1, 16, 8, 37, 2, 3, 6, 9),       # 6 splits; routed rows end in a half tile
    (128, 2, 8, 32, 23, 1, 2, 5, 9),       # 8 splits
    (64, 1, 2, 16, 7, 1, 2, 4, 66),        # 3 splits
    (64, 1, 3, 8, 22, 1, 1, 3, 45),        # 3 splits, heads beyond one workgroup
    (64, 1, 16, 32, 6, 1, 0, 3, 9),        # 3 splits, eight workgroups a unit
])
def test_few_units_form_has_the_split_forms_bits(d, kv, ratio, group, kg, first, last, q0, n):
    """A call with more query tiles than compute units takes the workgroup
    form with the merge kernel; its chunks one by one take the other.  The
    split counts agree (two tiles a split bound both)."""
    t = _Case(d, kv, ratio, group, kg, first, last, q0, n)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert 2 * kv * ratio * n > n_cu >= 2 * kv * ratio
    tiles = 1 + len(t.hga.hga_visible_chunks(t.plan.params, q0 + n - 1)) + -(-kg * group // 64)
    assert tiles == 1 + len(t.hga.hga_visible_chunks(t.plan.params, q0)) + -(-kg * group // 64)
    most = -(-n_cu // (kv * n * -(-2 * ratio // (8 if d == 128 else 4))))
    assert 1 < (tiles + 1) // 2 <= most
    out, lse = t.attend_split(0, n, t.hga.hga_attend_split_workspace(t.plan, n))
    assert not out.isnan().any() and not lse.isnan().any()
    for i in range(n):
        o1, l1 = t.attend_split(i, 1, t.hga.hga_attend_split_workspace(t.plan, 1))
        s = slice(i * 64, (i + 1) * 64)
        assert _same(o1, out[:, :, s]) and _same(l1, lse[:, :, s]), i


@pytest.mark.parametrize("d,kv,ratio,group,kg,first,last,q0,n,batch", [
    # more query tiles than compute units: the merge kernel
    (128, 4, 8, 16, 48, 1, 2, 13, 5, 1),
    (128, 2, 3, 32, 11, 2, 1, 7, 16, 2),
    (64, 3, 3, 8, 30, 1, 1, 7, 16, 1),
    (64, 1, 9, 16, 25, 0, 3, 8, 8, 2),
    # few query tiles and many key tiles: the merge kernel too
    (128, 1, 2, 32, 120, 1, 1, 70, 1, 1),
    (64, 2, 4, 16, 140, 2, 1, 40, 2, 1),
    # the last number of key tiles of the one-workgroup form for four query
    # tiles (10), and the first past it
    (128, 1, 2, 16, 25, 1, 1, 12, 1, 1),
    (128, 1, 2, 16, 29, 1, 1, 12, 1, 1),
    (64, 1, 2, 8, 50, 1, 1, 12, 1, 1),
    (64, 1, 2, 8, 57, 1, 1, 12, 1, 1),
])
def test_split_forms_match_oracle(d, kv, ratio, group, kg, first, last, q0, n, batch):
    """Routed rows from buffers, and gathered with and without buffers, against
    the float64 oracle; the three are the same bits."""
    t = _Case(d, kv, ratio, group, kg, first, last, q0, n, batch, seed=kg, distinct=True)
    hga, w = t.hga, t.w
    nbytes = hga.hga_attend_split_workspace(t.plan, n)
    out, lse = t.attend_split(0, n, nbytes)
    gi = t.gi.cpu().numpy()
    lim = (np.arange(q0, q0 + n) * (64 // group))[None, None, :, None]
    ref = O.attend(*(tensor_to_f64(x) for x in (t.q, t.k, t.v)), np.where(gi < lim, gi, -1),
                   list(range(q0, q0 + n)), 64, group, first, last, w.force_prev)
    assert np.abs(tensor_to_f64(out) - ref[0]).max() <= OUT_TOL["bf16"]
    assert np.abs(tensor_to_f64(lse) - ref[1]).max() <= LSE_TOL["bf16"]
    for buffers in (False, True):
        kr, vr = torch.full_like(t.kr, float("nan")), torch.full_like(t.vr, float("nan"))
        o2, l2 = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        ws = torch.full((nbytes // 4,), float("nan"), device="cuda")
        hga.hga_gather_attend_split(t.plan, t.q, q0, t.k, t.v, t.k, t.v, t.gi, kr if buffers else None,
                                    vr if buffers else None, o2, ws, l2)
        torch.cuda.synchronize()
        assert _same(o2, out) and _same(l2, lse), buffers
        if buffers:
            assert _same(kr, t.kr) and _same(vr, t.vr)


@pytest.mark.parametrize("d,ratio,group,kg,splits", [
    (128, 2, 16, 32, 2),     # two splits' workspace holds no 512 routed rows
    (128, 2, 8, 512, 9),
    (128, 2, 8, 512, 10),
    (128, 2, 8, 509, 11),
    (128, 2, 8, 512, 16),
    (64, 2, 16, 40, 2),
    (64, 2, 8, 509, 9),
    (64, 2, 8, 512, 16),
])
def test_host_source_bits_without_room_for_the_routed_rows(d, ratio, group, kg, splits):
    """From host memory without routed buffers, and with a workspace that holds
    the splits but not the rows, the output is still the one with buffers and
    that of hga_gather_kv and hga_attend_split, bit for bit."""
    t = _Case(d, 2, ratio, group, kg, 1, 1, 20, 2, batch=2, seed=kg)
    hga, plan = t.hga, t.plan
    kh, vh = t.k.cpu().pin_memory(), t.v.cpu().pin_memory()
    for i, n in ((1, 1), (0, 2)):
        nbytes = splits * t.split_bytes(n)
        assert nbytes < 2 * t.kr[:, :, :n].numel() * 2
        q = t.q[:, :, i * 64:(i + n) * 64].contiguous()
        gi = t.gi[:, :, i:i + n].contiguous()
        want = t.attend_split(i, n, nbytes)
        for buffers in (False, True):
            kr, vr = (torch.full_like(x[:, :, i:i + n], float("nan")) for x in (t.kr, t.vr))
            out = torch.full_like(q, float("nan"))
            lse = torch.full(q.shape[:3], float("nan"), device="cuda")
            ws = torch.empty(nbytes // 4, device="cuda")
            hga.hga_gather_attend_split(plan, q, t.q0 + i, t.k, t.v, kh, vh, gi,
                                        kr if buffers else None, vr if buffers else None, out, ws,
                                        lse, src_on_host=True)
            torch.cuda.synchronize()
            assert _same(out, want[0]) and _same(lse, want[1]), (i, n, buffers)
            if buffers:
                assert _same(kr, t.kr[:, :, i:i + n]) and _same(vr, t.vr[:, :, i:i + n])


@pytest.mark.parametrize("d,kv,ratio,kg,q0,n", [
    (128, 2, 2, 16, 20, 1),     # one workgroup a unit, few query tiles: gathered by the splits
    (128, 8, 2, 16, 20, 4),     # more of them: gathered ahead
    (128, 4, 8, 24, 20, 1),     # two workgroups a unit: ahead, then by query tile
    (128, 4, 8, 120, 40, 1),    # ... or, many key tiles, by the splits
    (64, 4, 2, 16, 20, 1),
    (64, 2, 5, 12, 20, 2),
    (64, 2, 5, 120, 40, 1),
])
def test_host_source_forms(d, kv, ratio, kg, q0, n):
    """From host memory: the bits of the two calls that it stands for, with
    buffers and without, whatever the workspace holds (everything; the rows
    behind the partial results, exactly; the rows and no more; not the rows)."""
    t = _Case(d, kv, ratio, 16, kg, 1, 1, q0, n, seed=kg + d)
    hga = t.hga
    kh, vh = t.k.cpu().pin_memory(), t.v.cpu().pin_memory()
    rows = 2 * t.kr.numel() * 2
    most = hga.hga_attend_split_workspace(t.plan, n)
    for nbytes in sorted({most, most + rows, rows, rows - 16, 3 * t.split_bytes(n) + rows,
                          3 * t.split_bytes(n) + rows - 16, 2 * t.split_bytes(n)}):
        want = t.attend_split(0, n, nbytes)
        for buffers in (False, True):
            kr, vr = torch.full_like(t.kr, float("nan")), torch.full_like(t.vr, float("nan"))
            out, lse = torch.full_like(want[0], float("nan")), torch.full_like(want[1], float("nan"))
            # (a guard behind the workspace)
            ws = torch.full((nbytes // 4 + 1024,), 7.0, device="cuda")
            hga.hga_gather_attend_split(t.plan, t.q, q0, t.k, t.v, kh, vh, t.gi,
                                        kr if buffers else None, vr if buffers else None, out,
                                        ws[:nbytes // 4], lse, src_on_host=True)
            torch.cuda.synchronize()
            assert _same(out, want[0]) and _same(lse, want[1]), (nbytes, buffers)
            assert bool((ws[nbytes // 4:] == 7).all())
            if buffers:
                assert _same(kr, t.kr) and _same(vr, t.vr)


@pytest.mark.parametrize("key,kw,splits", [
    # one tile of routed rows: block 0 has one split, the others two or three
    ("qwen32k", dict(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=64 * 12, topk_groups=4,
                     topk_chunks=3), 16),
    # more query tiles than compute units, a workspace for five splits, ragged rows
    ("qwen32k", dict(n_q_heads=16, n_kv_heads=2, seq_len=64 * 24, topk_groups=45, keep_last=3), 5),
    # up to nine and ten splits, one a wavefront
    ("qwen32k", dict(n_q_heads=8, n_kv_heads=2, seq_len=64 * 33, group=32, topk_groups=29,
                     keep_last=1), 16),
    # up to sixteen, two a wavefront
    ("qwen32k", dict(n_q_heads=8, n_kv_heads=4, seq_len=64 * 40, group=32, topk_chunks=40,
                     topk_groups=61), 16),
    ("smalllm", dict(batch=2, n_q_heads=6, n_kv_heads=2, seq_len=64 * 21, group=8, topk_groups=21,
                     topk_chunks=4), 16),
    ("smalllm", dict(batch=1, n_q_heads=16, n_kv_heads=1, seq_len=64 * 40, group=32,
                     topk_chunks=40, topk_groups=60), 16),
    # below two splits, without a workspace, one head per KV head, fp32: unsplit
    ("qwen32k", dict(n_q_heads=8, n_kv_heads=2, seq_len=64 * 9, topk_groups=9), 1),
    ("smalllm", dict(batch=1, n_q_heads=4, n_kv_heads=2, seq_len=64 * 9), 0),
    ("smalllm", dict(batch=2, n_q_heads=2, n_kv_heads=2, seq_len=64 * 9), 16),
    ("tiny", dict(n_q_heads=4, n_kv_heads=2), 16),
    # more middle chunks than the resident-key routing holds
    ("smalllm", dict(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=64 * 1061), 0),
    ("qwen32k", dict(n_q_heads=2, n_kv_heads=1, seq_len=64 * 1061, topk_groups=9), 4),
])
def test_prefill_blocks_has_block_steps_bits(key, kw, splits):
    """hga_prefill_blocks writes what hga_block_step writes for each block in
    order, bit for bit, with workspaces of any size; without a split that is
    the bulk prefill."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2606_30709_amd import hga
    from paper_2606_30709_amd.pipeline import BlockPrefillPipeline, PrefillPipeline
    w = W.preset(key).with_(needle_mode="none", **kw)
    inp = W.generate(w)
    blk = BlockPrefillPipeline(w, inp)
    if splits:
        nbytes = hga.hga_attend_split_workspace(blk.plan, 1) // 16 * splits
        blk.attend_ws = torch.full((nbytes // 4,), float("nan"), device="cuda")
    names = ("qbar", "chunk_idx", "group_idx", "k_routed", "v_routed", "out", "lse")
    for x in ("qbar", "k_routed", "v_routed", "out", "lse", "chunk_sum", "group_sum"):
        getattr(blk, x).fill_(float("nan"))
    blk.step()
    step = {x: torch.zeros_like(getattr(blk, x)) for x in names}
    cs, gs = torch.full_like(blk.chunk_sum, float("nan")), torch.full_like(blk.group_sum, float("nan"))
    for c in range(w.n_chunks):
        hga.hga_block_step(blk.plan, blk.q_blocks[c], c, blk.k, blk.v, cs, gs,
                           *(step[x][c] for x in names), workspace=blk.attend_ws)
    torch.cuda.synchronize()
    assert _same(cs, blk.chunk_sum) and _same(gs, blk.group_sum)
    for x in names:
        for c in range(w.n_chunks):
            assert _same(getattr(blk, x)[c], step[x][c]), (x, c)
    if splits < 2 or w.gqa_ratio == 1 or w.dtype == "f32":
        bulk = PrefillPipeline(w, inp)
        bulk.step()
        out = bulk.out.view(w.batch, w.n_q_heads, w.n_chunks, 64, w.head_dim).permute(2, 0, 1, 3, 4)
        assert _same(blk.out, out)
