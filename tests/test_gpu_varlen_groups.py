"""Packed batches whose sequences share launches: the same bits as one call per sequence, for batches of more sequences than a group (16) or a packing window (64) holds, with the workspace the library
asks for and with a larger one (larger groups), odd and even block counts, a sequence with a list entry to skip or with
values beyond fp16, which must not change the others."""
import numpy as np
import pytest
import torch

from paper_2602_08426_amd import binding as pb
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,h,hkv,B,d,bidir,extra,dirty", [
    ([1 + 37 * i % 700 for i in range(70)], 4, 2, 128, 128, False, 0, False),
    ([1 + 37 * i % 700 for i in range(70)], 4, 2, 128, 128, False, 64 << 20, False),
    ([3000, 129, 5, 1024, 1025, 2000, 640, 1], 8, 2, 128, 128, True, 64 << 20, False),
    ([3000, 129, 5, 1024, 1025, 2000, 640, 1], 8, 2, 128, 128, False, 64 << 20, True),
    ([64 * 6, 64 * 2, 64 * 10, 64 * 4], 4, 1, 64, 128, False, 64 << 20, False),      # even numbers of blocks: pairs allowed
    ([64 * 6 + 1, 64 * 2, 64 * 9, 33], 4, 1, 64, 64, False, 64 << 20, False),
    ([700, 128, 1400], 2, 2, 128, 256, False, 64 << 20, False),
    ([1024, 640, 2048, 384, 500, 128 * 9], 8, 2, 128, 128, False, 64 << 20, "list"),
    ([1024, 640, 2048, 384, 500, 128 * 9], 8, 2, 128, 128, True, 64 << 20, "value"),
    ([4096, 640, 2048, 384, 500, 128 * 90], 32, 8, 128, 128, False, 256 << 20, "list"),   # more than 4096 rows
    ([64 * 6, 64 * 2, 64 * 10, 64 * 4], 4, 1, 64, 128, False, 64 << 20, "list"),
    # 2976, 5024, 6016 and 6976 rows in one launch
    ([3000, 3500, 3001, 2049], 32, 8, 128, 128, False, 256 << 20, False),
    ([6000, 4500, 5000, 4299], 32, 8, 128, 64, False, 256 << 20, False),
    ([7000, 6500, 6000, 4400], 32, 8, 128, 64, True, 256 << 20, False),
    ([7000, 7900, 7000, 5801], 32, 8, 128, 64, False, 256 << 20, False),
    # the general form of the estimate over several sequences: 384 strips, 624 strips and bidirectional, N > 1024
    ([8192, 2048, 4096, 3000, 5000], 32, 8, 128, 128, False, 256 << 20, False),
    ([64 * 300, 64 * 299 + 1, 64 * 5], 16, 4, 64, 64, True, 128 << 20, False),
    ([64 * 1030, 64 * 20 + 3, 64 * 100, 64 * 513], 2, 1, 64, 128, False, 128 << 20, False),
])
def test_groups_equal_single_calls(lens, h, hkv, B, d, bidir, extra, dirty):
    print(f"case {len(lens)} sequences h={h}/{hkv} B={B} d={d} bidirectional={bidir} extra={extra}", flush=True)
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0
    if B == 64 and d == 128:
        flags |= pb.PRISM_FLAG_PAIR_KERNEL
    cu = [0] + np.cumsum(lens).tolist()
    T = cu[-1]
    g = torch.Generator(device="cuda").manual_seed(sum(lens) + d)
    q, k, v = (torch.randn((n, T, d), generator=g, device="cuda").bfloat16() for n in (h, hkv, hkv))
    bands = {64: (32, 48), 128: (64, 96), 256: (128, 192)}[d]
    if dirty == "value":
        v[0, cu[1] + 5, 3] = 1.0e5                        # the second sequence holds a value beyond fp16
    params = pb.make_params(h, hkv, T, B, *bands, 0.9, flags, d)
    mo, ro, co = pb.prism_varlen_layout(params, cu)
    mask, rp, ci, info = (torch.full((n,), -7, dtype=t, device="cuda") for n, t in (
        (mo[-1], torch.int64), (ro[-1], torch.int32), (co[-1], torch.int32), (4 * len(lens), torch.int32)))
    pb.prism_estimate_varlen(params, cu, q, k, mask, rp, ci, info,
                             pb.alloc_workspace(pb.prism_estimate_varlen_workspace_bytes(params, cu) + extra))
    if dirty in (True, "list"):
        ci[co[1]] = -1                                    # a list of the second sequence starts with an entry to skip
    out = torch.full((h, T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((h, T), float("nan"), dtype=torch.float32, device="cuda")
    pb.prism_sparse_attn_varlen(params, cu, q, k, v, rp, ci, out, lse,
                                pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu) + extra))
    torch.cuda.synchronize()
    for s, L in enumerate(lens):
        ps = pb.make_params(h, hkv, L, B, *bands, 0.9, flags, d)
        qs, ks, vs = (x[:, cu[s]:cu[s + 1]].contiguous() for x in (q, k, v))
        one = gu.gpu_estimate(ps, qs, ks)
        _, rp1, ci1, info1 = one["dev"]
        nnz = int(info1[0])
        assert torch.equal(mask[mo[s]:mo[s + 1]], one["dev"][0].view(-1)), s
        assert torch.equal(rp[ro[s]:ro[s + 1]], rp1), s
        assert torch.equal(info[4 * s:4 * s + 4], info1), s
        if dirty in (True, "list") and s == 1:
            ci1[0] = -1
        assert torch.equal(ci[co[s]:co[s] + nnz], ci1[:nnz]), s
        o1, l1 = gu.gpu_sparse_attn(ps, qs, ks, vs, rp1, ci1, nnz)
        assert torch.equal(out[:, cu[s]:cu[s + 1]].view(torch.int16), o1.view(torch.int16)), s
        assert torch.equal(lse[:, cu[s]:cu[s + 1]], l1), s


@pytest.mark.parametrize("room", [-1, 0, 1 << 20])
def test_estimate_of_a_batch_is_the_same_in_any_workspace(room):
    """In the least workspace that is taken (one without room for the row counts of the longest sequence, which goes the
    general way), in the one the library asks for and in a larger one."""
    lens, h, hkv, B = [5000, 300, 2048, 4999], 8, 2, 128
    cu = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device="cuda").manual_seed(12)
    q, k = (torch.randn((n, cu[-1], 128), generator=g, device="cuda").bfloat16() for n in (h, hkv))
    params = pb.make_params(h, hkv, cu[-1], B)
    need = pb.prism_estimate_varlen_workspace_bytes(params, cu)
    least = need - (h * 40 * 4 + 255) // 256 * 256           # ceil(5000 / 128) = 40 blocks
    mo, ro, co = pb.prism_varlen_layout(params, cu)

    def run(size):
        mask, rp, ci, info = (torch.full((n,), -7, dtype=t, device="cuda") for n, t in (
            (mo[-1], torch.int64), (ro[-1], torch.int32), (co[-1], torch.int32), (4 * len(lens), torch.int32)))
        pb.prism_estimate_varlen(params, cu, q, k, mask, rp, ci, info, pb.alloc_workspace(size)[:size])
        return mask, rp, ci, info

    for a, b in zip(run(least if room < 0 else need + room), run(need + (64 << 20))):
        assert torch.equal(a, b)
    with pytest.raises(pb.PrismError):
        run(least - 256)


@pytest.mark.parametrize("lens,h,hkv,B,d", [
    ([1024, 2048, 1024, 4096, 1024, 512], 8, 2, 128, 128),     # 64 blocks together fit the room of the 32 of the longest
    ([4096, 4096, 128, 300, 77], 8, 2, 128, 128),              # 65 do not
    ([1024, 2048, 1000, 4096, 1024, 64], 4, 1, 64, 64),
    ([1000, 2048, 3000, 640], 4, 4, 64, 256),
])
def test_groups_in_the_workspace_that_is_asked_for(lens, h, hkv, B, d):
    test_groups_equal_single_calls(lens, h, hkv, B, d, False, 0, False)
