"""The short form of the estimate (bands side by side, calibration and compaction without launches of their own) against
the general one, which a workspace without room for the row counts selects: the same bits, at the edges of a strip (16
blocks), of a row's registers (128, 256, 512 columns), with every option, with equal elements at the cut and with more
columns selected than the list has room for."""
import numpy as np
import pytest
import torch

from oracle import prism_oracle as orc
from paper_2602_08426_amd import binding as pb
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

AXIS = ([(0, 8), (16, 32), (72, 32)], [(0, 16), (36, 36), (92, 36)])


@pytest.mark.parametrize("h,hkv,N,tail,B,d,bands,p,flags,kind", [
    (1, 1, 1, 5, 128, 128, (64, 96), 0.95, 0, "noise"),
    (2, 1, 16, 64, 64, 128, (64, 96), 0.95, 0, "noise"),
    (7, 1, 17, 1, 128, 128, (64, 96), 0.9, 0, "noise"),
    (4, 2, 64, 128, 128, 64, (32, 48), 0.95, 0, "noise"),
    (4, 2, 65, 100, 128, 256, (128, 192), 0.95, 0, "noise"),
    (3, 1, 128, 64, 64, 128, (64, 96), 0.95, 0, "topics"),
    (3, 1, 129, 33, 64, 128, (0, 96), 0.95, 0, "topics"),
    (3, 3, 257, 64, 64, 128, (64, 0), 0.93, pb.PRISM_FLAG_NO_CALIBRATION, "topics"),
    (10, 2, 512, 64, 64, 64, (32, 48), 0.95, 0, "topics"),                        # 320 strips
    (2, 2, 200, 9, 64, 128, AXIS, 0.9, pb.PRISM_FLAG_BIDIRECTIONAL, "topics"),
    (2, 1, 90, 64, 64, 128, (64, 96), 0.95, pb.PRISM_FLAG_FORCE_DIAGONAL | pb.PRISM_FLAG_FORCE_SINK, "topics"),
    (2, 1, 90, 64, 64, 128, (64, 96), 1.0, 0, "noise"),
    (2, 1, 70, 64, 64, 128, (64, 96), 0.5, 0, "equal"),                           # every logit of a row the same: ties
    (2, 1, 70, 64, 64, 128, (64, 96), 0.95, 0, "zero"),                           # no energy
])
def test_same_bits_as_the_general_form(h, hkv, N, tail, B, d, bands, p, flags, kind):
    L = (N - 1) * B + tail
    print(f"case h={h}/{hkv} L={L} B={B} d={d} bands={bands} p={p} flags={flags:#x} {kind}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N * d + h)
    q, k = (torch.randn((n, L, d), generator=g, device="cuda") for n in (h, hkv))
    if kind == "topics":                                  # blocks that differ from one another
        for x in (q, k):
            x += torch.randn((x.shape[0], N, d), generator=g, device="cuda").repeat_interleave(B, 1)[:, :L] * 0.7
    elif kind == "equal":
        q, k = torch.ones_like(q), torch.ones_like(k)
    elif kind == "zero":
        q, k = torch.zeros_like(q), torch.zeros_like(k)
    q, k = q.bfloat16(), k.bfloat16()
    slices = isinstance(bands[0], list)
    params = pb.make_params(h, hkv, L, B, *((0, 0) if slices else bands), p, flags, d)
    need = pb.prism_estimate_workspace_bytes(params)
    outs = []
    for room in (need, need - (h * N * 4 + 255) // 256 * 256):
        for cap in (None, 37):
            mask, rp, ci, info = pb.alloc_estimate_outputs(params)
            ci.fill_(-7)
            n = ci.numel() if cap is None else min(cap, ci.numel())
            ws = pb.alloc_workspace(room)[:max(room, 1)]
            if slices:
                pb.prism_estimate_bands(params, pb.make_bands(*bands), q, k, mask, rp, ci, n, info, ws)
            else:
                pb.prism_estimate(params, q, k, mask, rp, ci, n, info, ws)
            outs.append((mask, rp, ci, info))
    torch.cuda.synchronize()
    for i in (0, 1):
        for a, b in zip(outs[i], outs[2 + i]):
            assert torch.equal(a, b)
    assert int(outs[0][3][0]) == int(outs[0][1][-1]) and int(outs[0][3][0]) >= h * N
    with pytest.raises(pb.PrismError):
        ws = pb.alloc_workspace(need)[:need - (h * N * 4 + 255) // 256 * 256 - 1]
        pb.prism_estimate(params, q, k, *outs[0][:3], 1, outs[0][3], ws)


@pytest.mark.parametrize("h,N,tail,flags", [
    (50, 256, 64, 0), (47, 257, 1, 0),             # 800 and 799 strips: four waves of four rows
    (48, 256, 64, 0),                              # 768: eight of two
    (24, 512, 9, pb.PRISM_FLAG_BIDIRECTIONAL),
    (26, 497, 64, 0),                              # 832 strips of rows of up to eight registers
    (8, 513, 64, 0), (7, 513, 5, 0),               # 264: eight of two; 231: sixteen of one
    (5, 1024, 64, 0), (2, 1024, 3, pb.PRISM_FLAG_BIDIRECTIONAL),
    (3, 1025, 64, 0), (2, 1100, 7, 0),             # beyond 1024 blocks
])
def test_forms_of_the_general_selection(h, N, tail, flags):
    """Every head of a call has the bits of a call on that head and one other, which takes the short form or sixteen waves of one
    row, and the lists are those of the bits.  Calls that have sixteen waves of one row themselves (7 heads of 513 blocks, 2 of 1024,
    and all beyond 1024) are held against the oracle in the test below."""
    B, L = 64, (N - 1) * 64 + tail
    g = torch.Generator(device="cuda").manual_seed(N + h)
    q, k = (torch.randn((n, L, 128), generator=g, device="cuda") for n in (h, 1))
    for x in (q, k):
        x += torch.randn((x.shape[0], N, 128), generator=g, device="cuda").repeat_interleave(B, 1)[:, :L] * 0.6
    q, k = q.bfloat16(), k.bfloat16()

    def run(heads):
        params = pb.make_params(len(heads), 1, L, B, flags=flags)
        mask, rp, ci, info = pb.alloc_estimate_outputs(params)
        pb.prism_estimate(params, q[heads].contiguous(), k, mask, rp, ci, ci.numel(), info,
                          pb.alloc_workspace(pb.prism_estimate_workspace_bytes(params)))
        rp2, ci2, info2 = torch.empty_like(rp), torch.empty_like(ci), torch.empty_like(info)
        pb.prism_mask_to_csr(params, mask, rp2, ci2, ci2.numel(), info2)
        torch.cuda.synchronize()
        n = int(info[0])
        assert torch.equal(rp, rp2) and torch.equal(info, info2) and torch.equal(ci[:n], ci2[:n])
        return mask.view(len(heads), -1)

    mask = run(list(range(h)))
    for i in sorted({0, (h - 2) // 2, h - 2}):
        assert torch.equal(mask[i:i + 2], run([i, i + 1])), i


@pytest.mark.parametrize("h,N,tail,d,flags", [
    (50, 250, 9, 256, 0),                                   # 800 strips: four waves of four rows
    (30, 300, 64, 256, pb.PRISM_FLAG_BIDIRECTIONAL),        # 570: eight of two
    (8, 600, 64, 64, 0), (8, 520, 3, 256, 0),               # 304 and 264: eight of two rows of up to 1024
    (7, 513, 5, 128, 0), (2, 1024, 3, 128, pb.PRISM_FLAG_BIDIRECTIONAL), (2, 700, 64, 256, 0),      # sixteen of one
    (3, 1025, 64, 128, 0), (2, 1100, 7, 128, 0), (2, 1040, 64, 64, pb.PRISM_FLAG_BIDIRECTIONAL), (2, 1030, 1, 256, 0),
])
def test_general_selection_agrees_with_the_oracle(h, N, tail, d, flags):
    """The first and the last head: the blocks that the oracle selects, outside its margin at the cut."""
    B, L = 64, (N - 1) * 64 + tail
    g = torch.Generator(device="cuda").manual_seed(N + h)
    q, k = (torch.randn((n, L, d), generator=g, device="cuda") for n in (h, 1))
    for x in (q, k):
        x += torch.randn((x.shape[0], N, d), generator=g, device="cuda").repeat_interleave(B, 1)[:, :L] * 0.6
    q, k = q.bfloat16(), k.bfloat16()
    bands = {64: (32, 48), 128: (64, 96), 256: (128, 192)}[d]
    res = gu.gpu_estimate(pb.make_params(h, 1, L, B, *bands, 0.95, flags, d), q, k)
    sel = orc.prism_select(q[[0, h - 1]].double().cpu().numpy(), k.double().cpu().numpy(), *bands, B, 0.95,
                           causal=not flags & pb.PRISM_FLAG_BIDIRECTIONAL)
    tol = orc.selection_tolerance(sel, 0.95)
    mask = res["mask"][[0, h - 1]]
    assert not (tol.must & ~mask).any() and not (tol.must_not & mask).any()
    assert tol.dont_care_fraction < 0.02
