"""The fp32 attention against the float64 oracle where its tiling has edges:
routed rows that end inside a 32-key sub-tile, sub-tiles of one, two and four
groups, chunks with fewer sub-tiles than wavefronts, invalid group ids, and
resident chunks behind a slot map (valid and not)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import hga_oracle as O
from paper_2606_30709_amd import workloads as W
from paper_2606_30709_amd.pipeline import PrefillPipeline

from parity_util import LSE_TOL, OUT_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,group,kg,ratio,first,last", [
    (64, 8, 3, 1, 1, 0),      # 24 routed rows: one partial sub-tile
    (64, 32, 1, 3, 1, 2),     # one group fills a sub-tile
    (64, 16, 7, 2, 2, 1),     # 112 rows: the last sub-tile half full
    (128, 8, 13, 2, 1, 0),
    (128, 32, 2, 1, 0, 0),
    (128, 16, 4, 5, 1, 3),
])
def test_f32_attention_tile_edges(d, group, kg, ratio, first, last):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2606_30709_amd import hga
    w = W.preset("tiny").with_(batch=2, n_q_heads=2 * ratio, n_kv_heads=2, head_dim=d,
                               seq_len=64 * 9, group=group, topk_groups=kg, topk_chunks=3,
                               keep_first=first, keep_last=last, needle_mode="none")
    inp = W.generate(w, seed=77)
    pipe = PrefillPipeline(w, inp, routed_out=False)
    pipe.step()
    torch.cuda.synchronize()
    q, k, v = (inp[x].astype(np.float64) for x in "qkv")
    args = (w.chunk, w.group, w.keep_first, w.keep_last, w.force_prev)
    gi = pipe.group_idx.cpu().numpy()
    ids = list(range(w.n_chunks))

    def check(out, lse, gi):
        ro, rl = O.attend(q, k, v, gi, ids, *args)
        assert np.abs(out.double().cpu().numpy() - ro).max() <= OUT_TOL["f32"]
        assert np.abs(lse.double().cpu().numpy() - rl).max() <= LSE_TOL["f32"]

    check(pipe.out, pipe.lse, gi)
    ref = pipe.out.clone()
    # ids that are padded in the middle of the list or in the causal future
    # count like absent rows, from the routed buffers and from the source
    bad = pipe.group_idx.clone()
    bad[:, :, 5, 0] = -1
    bad[:, :, 6, -1] = 6 * (64 // group)
    want = bad.cpu().numpy().copy()
    want[:, :, 6, -1] = -1
    kr = torch.full((2, 2, 9, kg * group, d), float("nan"), device="cuda")
    vr = kr.clone()
    for buffers in (False, True):
        out, lse = torch.empty_like(pipe.out), torch.empty_like(pipe.lse)
        hga.hga_gather_attend(pipe.plan, pipe.q, 0, pipe.k, pipe.v, bad, kr if buffers else None,
                              vr if buffers else None, out, lse)
        torch.cuda.synchronize()
        check(out, lse, want)
    # the same attention with the resident chunks in another order
    order = torch.randperm(9, generator=torch.Generator().manual_seed(5))
    kp, vp = (x.view(2, 2, 9, 64, d)[:, :, order].reshape(x.shape).contiguous()
              for x in (pipe.k, pipe.v))
    slot = torch.empty(9, dtype=torch.int32)
    slot[order] = torch.arange(9, dtype=torch.int32)
    slot = slot.cuda()
    hga.hga_gather_kv(pipe.plan, pipe.group_idx, 0, pipe.k, pipe.v, kr, vr)
    out = torch.empty_like(pipe.out)
    hga.hga_attend(pipe.plan, pipe.q, 0, kp, vp, kr, vr, pipe.group_idx, out, None, res_slot=slot)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    slot[8] = 9  # past the resident buffer: that chunk's rows are NaN, no others
    hga.hga_attend(pipe.plan, pipe.q, 0, kp, vp, kr, vr, pipe.group_idx, out, None, res_slot=slot)
    torch.cuda.synchronize()
    rows = out.view(2, 2 * ratio, 9, 64, d)
    assert bool(rows[:, :, 8].isnan().all()) and torch.equal(rows[:, :, :8], ref.view(rows.shape)[:, :, :8])
