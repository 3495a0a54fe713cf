"""The V image that prism_v_image and prism_sparse_attn leave for prism_sparse_attn_pre: every block and head size, whole and ragged
lengths, clean lists and lists that send a call to the general kernel, one-launch and separate preparation.  And V in places of its
own: where the outputs go, and at any alignment."""
import numpy as np
import pytest
import torch

from oracle import prism_oracle as orc
from paper_2602_08426_amd import binding as pb
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# h, h_kv, blocks, tokens of the last one, B, d, kind of lists
SHAPES = [
    (6, 3, 9, 64, 64, 64, "clean"), (6, 3, 9, 17, 64, 64, "clean"),
    (4, 2, 12, 64, 64, 128, "clean"), (5, 5, 9, 1, 64, 128, "clean"),
    (4, 2, 7, 64, 64, 256, "clean"), (4, 4, 7, 63, 64, 256, "clean"),
    (44, 44, 64, 64, 64, 256, "clean"), (44, 4, 64, 5, 64, 256, "clean"),        # 2816 rows: pairs with two buffers per tile
    (44, 4, 64, 64, 64, 256, "skip"),
    (32, 32, 128, 33, 64, 128, "clean"), (32, 4, 128, 64, 64, 128, "unsorted"),  # 4096 rows: pairs
    (6, 2, 9, 128, 128, 64, "clean"), (3, 3, 9, 100, 128, 64, "clean"),
    (6, 2, 9, 128, 128, 128, "clean"), (6, 2, 9, 128, 128, 128, "skip"), (3, 3, 9, 77, 128, 128, "clean"),
    (3, 3, 9, 128, 128, 128, "large"),                                           # V beyond fp16
    (6, 2, 5, 128, 128, 256, "clean"), (3, 3, 5, 1, 128, 256, "clean"),
    (66, 66, 125, 128, 128, 128, "skip"), (66, 66, 125, 40, 128, 64, "clean"),   # 8250 rows: separate kernels
]


def _inputs(h, hkv, N, tail, B, d, kind):
    L = (N - 1) * B + tail
    g = torch.Generator(device="cuda").manual_seed(N * B + h + tail)
    q, k, v = (torch.randn((n, L, d), generator=g, device="cuda").bfloat16() for n in (h, hkv, hkv))
    if kind == "large":
        v[-1, L // 2, 3] = 1.0e5
    rng = np.random.default_rng(h + tail)
    mask = np.tril(rng.random((h, N, N)) < 0.3)
    mask[:, np.arange(N), np.arange(N)] = True
    rp, ci, cnt = gu.csr_to_device(*orc.mask_to_csr(mask))
    at = int(rp[N])                                        # the last entries of the first q-head's last row
    if kind == "skip":
        ci[at - 1] = -1
    if kind == "unsorted":
        ci[at - 2:at] = ci[at - 2:at].flip(0)
    bands = {64: (32, 48), 128: (64, 96), 256: (128, 192)}[d]
    return pb.make_params(h, hkv, L, B, *bands, 0.9, 0, d), q, k, v, rp, ci, cnt


def _same(a, b):
    return torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                       b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32))


@pytest.mark.parametrize("h,hkv,N,tail,B,d,kind", SHAPES)
def test_image_of_either_call_serves_pre(h, hkv, N, tail, B, d, kind):
    """prism_sparse_attn leaves what prism_v_image leaves: calls of prism_sparse_attn_pre behind either have its bits, also where the
    first call took another kernel, and out and lse agree with 64-bit attention."""
    params, q, k, v, rp, ci, cnt = _inputs(h, hkv, N, tail, B, d, kind)
    need = pb.prism_sparse_attn_workspace_bytes(params)
    general = pb.make_params(h, hkv, params.seq_len, B, params.d_high, params.d_low, 0.9, pb.PRISM_FLAG_GENERAL_KERNEL, d)

    def pre(p, ws):
        out = torch.full_like(q, float("nan"))
        lse = torch.full((h, params.seq_len), float("nan"), device="cuda")
        pb.prism_sparse_attn_pre(p, q, k, ws, rp, ci, cnt, out, lse)
        torch.cuda.synchronize()
        return out, lse

    results = {}
    for p in (params, general):
        ws = torch.full((need,), 0x3c, dtype=torch.uint8, device="cuda")
        out, lse = torch.full_like(q, float("nan")), torch.full((h, params.seq_len), float("nan"), device="cuda")
        pb.prism_sparse_attn(p, q, k, v, rp, ci, cnt, out, lse, ws)
        torch.cuda.synchronize()
        results[p.flags] = (out, lse)
        for reader in (general, params, general):
            got = pre(reader, ws)
            if reader.flags in results:
                assert all(_same(a, b) for a, b in zip(got, results[reader.flags])), (p.flags, reader.flags)
            else:
                results[reader.flags] = got
    image = torch.full((need,), 0x3c, dtype=torch.uint8, device="cuda")
    pb.prism_v_image(params, v, image)
    for p in (params, general):
        assert all(_same(a, b) for a, b in zip(pre(p, image), results[p.flags])), p.flags
    rows, counts = rp.cpu().numpy(), ci.cpu().numpy()
    for i, u in {(0, N - 1), (0, 0), (h - 1, N // 2), (h - 1, N - 1)}:
        listed = counts[rows[i * N + u]:rows[i * N + u + 1]]
        t0, t1 = u * B, min((u + 1) * B, params.seq_len)
        seen = torch.from_numpy(np.isin(np.arange(t1) // B, listed)).cuda()[None, :]
        seen = seen & (torch.arange(t1, device="cuda")[None, :] <= torch.arange(t0, t1, device="cuda")[:, None])
        j = i // (h // hkv)
        x = (q[i, t0:t1].double() @ k[j, :t1].double().T / np.sqrt(d)).masked_fill(~seen, -np.inf)
        live = seen.any(1)
        ref = torch.where(live[:, None], torch.nan_to_num(torch.softmax(x, -1)) @ v[j, :t1].double(), 0.0)
        for out, lse in results.values():
            # 2e-2: the bar of the other attention tests, for values of that size
            assert ((out[i, t0:t1].double() - ref).abs() <= 2e-2 * torch.clamp(ref.abs(), min=1.0)).all(), (i, u)
            assert (lse[i, t0:t1].double() - torch.logsumexp(x, -1))[live].abs().max() <= 2e-3, (i, u)


@pytest.mark.parametrize("h,hkv,N,tail,B,d,kind", SHAPES)
def test_values_where_the_outputs_go(h, hkv, N, tail, B, d, kind):
    """V at the start of out, at its end, across its end, across lse, and at an odd address: the bits of a call with buffers apart."""
    params, q, k, v, rp, ci, cnt = _inputs(h, hkv, N, tail, B, d, kind)
    ref, ref_lse = gu.gpu_sparse_attn(params, q, k, v, rp, ci, cnt)
    ws = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(params))
    n_out, n_v, n_lse = q.numel(), v.numel(), 2 * ref_lse.numel()         # in elements of 2 bytes
    # where V starts among [out | lse | room]
    for at in {0, 1, n_out - n_v, n_out - n_v // 2 // 128 * 128, n_out, n_out + n_lse + 1}:
        buf = torch.zeros(n_out + n_lse + n_v + 8, dtype=torch.bfloat16, device="cuda")
        out = buf[:n_out].view(q.shape)
        lse = buf[n_out:n_out + n_lse].view(torch.float32).view(ref_lse.shape)
        vals = buf[at:at + n_v].view(v.shape)
        vals.copy_(v)
        pb.prism_sparse_attn(params, q, k, vals, rp, ci, cnt, out, lse, ws)
        torch.cuda.synchronize()
        assert _same(out, ref) and _same(lse, ref_lse), at


@pytest.mark.parametrize("lens,h,hkv,B,d,extra,dirty", [
    ([1024, 640, 2048, 384, 500, 128 * 9], 4, 4, 128, 128, 0, None),
    ([1024, 640, 2048, 384, 500, 128 * 9], 8, 2, 128, 128, 64 << 20, "skip"),       # one group of whole blocks, one ragged
    ([1024, 640, 2048, 384, 500, 128 * 9], 4, 4, 128, 128, 64 << 20, "large"),
    ([3000, 129, 5, 1025, 641, 1], 4, 4, 128, 64, 64 << 20, None),
    ([700, 128, 1400], 2, 2, 128, 256, 64 << 20, None),
    ([64 * 6, 64 * 2, 64 * 10, 64 * 4], 4, 1, 64, 64, 64 << 20, None),
    ([64 * 40, 64 * 2, 64 * 100, 64 * 4], 32, 32, 64, 128, 256 << 20, None),        # 4672 rows: pairs
    ([64 * 40 - 9, 64 * 2, 64 * 50, 64 * 4], 32, 8, 64, 256, 256 << 20, None),      # 2944 rows of whole blocks: pairs
    ([128 * 130, 1000, 128 * 3], 66, 66, 128, 128, 0, "skip"),                      # 8580 rows of one sequence: separate kernels
])
def test_values_where_the_outputs_of_a_packed_batch_go(lens, h, hkv, B, d, extra, dirty):
    """V at the start of out and at an odd address: the bits of a call with buffers apart."""
    cu = [0] + np.cumsum(lens).tolist()
    T = cu[-1]
    g = torch.Generator(device="cuda").manual_seed(T + d)
    q, k, v = (torch.randn((n, T, d), generator=g, device="cuda").bfloat16() for n in (h, hkv, hkv))
    if dirty == "large":
        v[0, cu[1] + 5, 3] = 1.0e5
    bands = {64: (32, 48), 128: (64, 96), 256: (128, 192)}[d]
    params = pb.make_params(h, hkv, T, B, *bands, 0.9, 0, d)
    _, ro, co = pb.prism_varlen_layout(params, cu)
    rp = torch.zeros(ro[-1], dtype=torch.int32, device="cuda")
    ci = torch.zeros(co[-1], dtype=torch.int32, device="cuda")
    for s, L in enumerate(lens):
        pb.prism_causal_csr(pb.make_params(h, hkv, L, B, *bands, 0.9, 0, d), rp[ro[s]:], ci[co[s]:], co[s + 1] - co[s])
    if dirty == "skip":
        ci[co[0]] = -1
    ws = pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu) + extra)
    ref, ref_lse = torch.full_like(q, float("nan")), torch.full((h, T), float("nan"), device="cuda")
    pb.prism_sparse_attn_varlen(params, cu, q, k, v, rp, ci, ref, ref_lse, ws)
    torch.cuda.synchronize()
    assert not torch.isnan(ref.float()).any()
    n_out, n_v = q.numel(), v.numel()
    for at in (0, n_out + 1):
        buf = torch.zeros(n_out + n_v + 8, dtype=torch.bfloat16, device="cuda")
        out, vals, lse = buf[:n_out].view(q.shape), buf[at:at + n_v].view(v.shape), torch.zeros_like(ref_lse)
        vals.copy_(v)
        pb.prism_sparse_attn_varlen(params, cu, q, k, vals, rp, ci, out, lse, ws)
        torch.cuda.synchronize()
        assert _same(out, ref) and _same(lse, ref_lse), at


@pytest.mark.parametrize("h,hkv,N,tail,B,d,kind", [s for s in SHAPES if s[3] < s[4] and s[1] > 1])
def test_nothing_behind_a_ragged_end_of_a_head_is_read(h, hkv, N, tail, B, d, kind):
    """The workspace full of NaN, V of every other kv head NaN or infinite: the other heads keep their bits."""
    params, q, k, v, rp, ci, cnt = _inputs(h, hkv, N, tail, B, d, kind)
    ref, ref_lse = gu.gpu_sparse_attn(params, q, k, v, rp, ci, cnt)
    out, lse = torch.empty_like(ref), torch.empty_like(ref_lse)
    for first, value in ((0, float("nan")), (1, float("inf"))):
        vals = v.clone()
        vals[first::2] = value
        ws = torch.full((pb.prism_sparse_attn_workspace_bytes(params),), 0xff, dtype=torch.uint8, device="cuda")
        pb.prism_sparse_attn(params, q, k, vals, rp, ci, cnt, out, lse, ws)
        torch.cuda.synchronize()
        clean = torch.arange(h, device="cuda") // (h // hkv) % 2 != first
        assert _same(out[clean], ref[clean]) and _same(lse, ref_lse)


@pytest.mark.parametrize("lens,h,hkv,B,d", [
    ([64 * 39 + 5, 64 * 47 + 63, 64 * 2 - 1], 32, 8, 64, 256),      # 2880 rows in one group: pairs with two buffers per tile
    ([64 * 79 + 5, 64 * 47 + 63, 64 * 2 - 1], 32, 8, 64, 128),      # 4160: pairs
    ([64 * 20 + 5, 64 * 30, 64 * 7 - 1], 16, 4, 64, 256),           # plain
])
def test_nothing_behind_a_ragged_end_of_a_sequence_is_read(lens, h, hkv, B, d):
    """V of every other sequence NaN or infinite, read as it is given and by way of the copy: the other sequences keep their bits."""
    cu = [0] + np.cumsum(lens).tolist()
    T = cu[-1]
    g = torch.Generator(device="cuda").manual_seed(T)
    q, k, v = (torch.randn((n, T, d), generator=g, device="cuda").bfloat16() for n in (h, hkv, hkv))
    bands = {128: (64, 96), 256: (128, 192)}[d]
    params = pb.make_params(h, hkv, T, B, *bands, 0.9, 0, d)
    _, ro, co = pb.prism_varlen_layout(params, cu)
    rp, ci = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in (ro[-1], co[-1]))
    for s, L in enumerate(lens):
        pb.prism_causal_csr(pb.make_params(h, hkv, L, B, *bands, 0.9, 0, d), rp[ro[s]:], ci[co[s]:], co[s + 1] - co[s])
    need = pb.prism_sparse_attn_varlen_workspace_bytes(params, cu) + (256 << 20)

    def run(vals):
        out = torch.full_like(q, float("nan"))
        ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")
        pb.prism_sparse_attn_varlen(params, cu, q, k, vals, rp, ci, out, None, ws)
        torch.cuda.synchronize()
        return out

    ref = run(v)
    for first, value in ((0, float("nan")), (1, -float("inf"))):
        for at in (0, 1):
            buf = torch.zeros(v.numel() + 8, dtype=torch.bfloat16, device="cuda")
            vals = buf[at:at + v.numel()].view(v.shape)
            vals.copy_(v)
            for s in range(first, len(lens), 2):
                vals[:, cu[s]:cu[s + 1]] = value
            out = run(vals)
            for s in range(1 - first, len(lens), 2):
                assert _same(out[:, cu[s]:cu[s + 1]].contiguous(), ref[:, cu[s]:cu[s + 1]].contiguous()), (s, at)
