"""Ragged last blocks at B = 128, d = 128: tails of one token, around the 32 queries of a wave and one short of a block;
causal and bidirectional; nothing written past the last row; V of any magnitude; one V image for several calls."""
import numpy as np
import pytest
import torch

from oracle import prism_oracle as orc
from paper_2602_08426_amd import binding as pb
from paper_2602_08426_amd import workloads as wl

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# one bf16 rounding of |o| <= 4 (2^-7) plus that of P; the bars of the other attention tests
OUT_TOL, LSE_TOL = 2e-2, 2e-3


@pytest.mark.parametrize("h", [64, 128])
@pytest.mark.parametrize("tail,bidir", [(1, False), (32, True), (63, False), (64, True), (65, False), (65, True), (97, False),
                                        (127, True), (1, True)])
def test_ragged_last_block(tail, bidir, h):
    hkv, B, N = 2, 128, 33
    L = (N - 1) * B + tail
    print(f"case h={h} L={L} bidirectional={bidir}", flush=True)
    rng = np.random.default_rng(100 + tail + bidir)
    Qb, Kb, Vb = (wl.f32_to_bf16_bits(rng.standard_normal((n, L, 128)).astype(np.float32) * a)
                  for n, a in ((h, 1.5), (hkv, 1.5), (hkv, 1.0)))
    mask = rng.random((h, N, N)) < 0.5
    mask[:, N - 1, N - 1] = True                            # the ragged block meets itself
    mask[0, 2, :] = False                                   # an empty row, and (bidirectional) one that starts at
    mask[1, N - 1, :] = False                               # the ragged block
    mask[2, 3, :] = False
    mask[2, 3, N - 1 if bidir else 3] = True
    if not bidir:
        mask = np.tril(mask)
    params = pb.make_params(h, hkv, L, B, flags=pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0)
    rp_d, ci_d, cnt = gu.csr_to_device(*orc.mask_to_csr(mask))
    qd, kd, vd = (pb.bf16_bits_to_device(x) for x in (Qb, Kb, Vb))
    need = pb.prism_sparse_attn_workspace_bytes(params)
    # guard elements behind the outputs
    out_g = torch.full((h * L * 128 + 4096,), 7.0, dtype=torch.bfloat16, device="cuda")
    lse_g = torch.full((h * L + 128,), 7.0, dtype=torch.float32, device="cuda")
    out, lse = out_g[:h * L * 128].view(h, L, 128), lse_g[:h * L].view(h, L)
    pb.prism_sparse_attn(params, qd, kd, vd, rp_d, ci_d, cnt, out, lse, pb.alloc_workspace(need))
    torch.cuda.synchronize()
    assert (out_g[h * L * 128:] == 7.0).all() and (lse_g[h * L:] == 7.0).all()
    o, s = out.float().cpu().numpy(), lse.cpu().numpy()
    Q, K, V = (orc.bf16_to_f64(x) for x in (Qb, Kb, Vb))
    for i in (0, 1, 2, 31, h - 1):
        seen = mask[i].repeat(B, 0).repeat(B, 1)[:L, :L]
        if not bidir:
            seen = np.tril(seen)
        x = np.where(seen, Q[i] @ K[i // (h // 2)].T / np.sqrt(128.0), -np.inf)
        m = x.max(1, keepdims=True)
        e = np.exp(x - np.where(np.isfinite(m), m, 0.0))
        t = e.sum(1)
        ref = np.where(t[:, None] > 0, e @ V[i // (h // 2)] / np.where(t > 0, t, 1.0)[:, None], 0.0)
        assert np.abs(o[i] - ref).max() <= OUT_TOL
        live = t > 0
        assert np.abs(s[i][live] - (m[live, 0] + np.log(t[live]))).max() <= LSE_TOL
        assert (s[i][~live] == -np.inf).all()


def test_one_image_for_calls_with_other_query_heads():
    """A V image of a ragged length serves attention calls on any of the q-heads of its kv heads."""
    hkv, B, L = 2, 128, 128 * 20 + 17
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((n, L, 128), generator=g, device="cuda").bfloat16() for n in (16, hkv, hkv))
    full = pb.make_params(16, hkv, L, B)
    image = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(full))
    pb.prism_v_image(full, v, image)
    for n in (16, 8, 2):
        part = pb.make_params(n, hkv, L, B)
        _, rp, ci, _ = pb.alloc_estimate_outputs(part)
        pb.prism_causal_csr(part, rp, ci, ci.numel())
        qs = q.view(hkv, 16 // hkv, L, 128)[:, :n // hkv].reshape(n, L, 128).contiguous()
        out, lse = torch.empty_like(qs), torch.empty((n, L), device="cuda")
        pb.prism_sparse_attn_pre(part, qs, k, image, rp, ci, ci.numel(), out, lse)
        ref, ref_lse = gu.gpu_sparse_attn(part, qs, k, v, rp, ci, ci.numel())
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse), n


def test_image_calls_are_right_whatever_the_buffer_holds():
    """An image written for some number of q-heads, then attention with others, in buffers of several sizes: every call that
    is accepted gives what one call with a workspace of its own gives, before and after calls with other q-heads."""
    hkv, L = 2, 128 * 20 + 17
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((n, L, 128), generator=g, device="cuda").bfloat16() for n in (16, hkv, hkv))
    calls = {}
    for n in (2, 8, 16):
        p = pb.make_params(n, hkv, L, 128)
        _, rp, ci, _ = pb.alloc_estimate_outputs(p)
        pb.prism_causal_csr(p, rp, ci, ci.numel())
        qs = q[:n].contiguous()
        calls[n] = (p, qs, rp, ci, gu.gpu_sparse_attn(p, qs, k, v, rp, ci, ci.numel()))
    need = {n: pb.prism_sparse_attn_workspace_bytes(calls[n][0]) for n in calls}
    image = hkv * 21 * 128 * 128 * 2
    accepted = 0
    for size in (need[2], need[8], need[16] - 256, need[16], need[8] + image, need[16] + image):
        buf = pb.alloc_workspace(size)[:size]
        for writer in calls:
            buf.fill_(0x3c)                                # 1.06 as fp16, a set flag as a word
            try:
                pb.prism_v_image(calls[writer][0], v, buf)
            except pb.PrismError:
                continue
            for reader in (16, 8, 2, 8, 16):
                p, qs, rp, ci, (ref, ref_lse) = calls[reader]
                out, lse = torch.zeros_like(qs), torch.zeros_like(ref_lse)
                try:
                    pb.prism_sparse_attn_pre(p, qs, k, buf, rp, ci, ci.numel(), out, lse)
                except pb.PrismError:
                    continue
                torch.cuda.synchronize()
                assert torch.equal(out, ref) and torch.equal(lse, ref_lse), (size, writer, reader)
                accepted += 1
    assert accepted >= 40


def _check_small_values(q, k, v, out):
    """One head of causal attention in 64 bits; every output within one bf16 rounding (2^-8) of P and one of itself."""
    L = q.shape[0]
    x = (q.double() @ k.double().T) / np.sqrt(128.0)
    p = torch.softmax(x.masked_fill(torch.ones(L, L, dtype=torch.bool, device="cuda").triu(1), -np.inf), -1)
    ref, size = p @ v.double(), p @ v.double().abs()
    assert ((out.double() - ref).abs() <= 1.02 * 2.0 ** -8 * (size + ref.abs())).all()


@pytest.mark.parametrize("h,hkv,L", [(2, 2, 128 * 5 + 100), (8, 2, 128 * 21 - 1), (65, 1, 128 * 63 + 77)])
def test_values_of_any_magnitude(h, hkv, L):
    """V is used as it is given: dims of 1 down to 2^-30 (below 2^-24 fp16 has nothing left), and a token of tiny values."""
    print(f"case h={h} L={L}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn((n, L, 128), generator=g, device="cuda") for n in (h, hkv, hkv))
    v = v * 2.0 ** -(torch.arange(128, device="cuda") % 31).float()
    v[:, 7] *= 2.0 ** -20
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    params = pb.make_params(h, hkv, L, 128)
    _, rp, ci, _ = pb.alloc_estimate_outputs(params)
    pb.prism_causal_csr(params, rp, ci, ci.numel())
    out, _ = gu.gpu_sparse_attn(params, q, k, v, rp, ci, ci.numel())
    for i in {0, h - 1}:
        _check_small_values(q[i], k[i // (h // hkv)], v[i // (h // hkv)], out[i])


@pytest.mark.parametrize("h,hkv,lens", [(8, 2, [128 * 20 + 5, 256, 77, 128 * 9 + 64]), (48, 2, [128 * 60 + 5, 128 * 25, 777])])
def test_values_of_any_magnitude_in_a_packed_batch(h, hkv, lens):
    """The same for the ragged sequences of a batch that holds others too."""
    print(f"case h={h} lens={lens}", flush=True)
    cu = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device="cuda").manual_seed(cu[-1])
    q, k, v = (torch.randn((n, cu[-1], 128), generator=g, device="cuda") for n in (h, hkv, hkv))
    small = v * 2.0 ** -(torch.arange(128, device="cuda") % 31).float()
    for s, L in enumerate(lens):
        if L % 128:
            v[:, cu[s]:cu[s + 1]] = small[:, cu[s]:cu[s + 1]]
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    params = pb.make_params(h, hkv, cu[-1], 128)
    _, ro, co = pb.prism_varlen_layout(params, cu)
    rp = torch.zeros(ro[-1], dtype=torch.int32, device="cuda")
    ci = torch.zeros(co[-1], dtype=torch.int32, device="cuda")
    for s, L in enumerate(lens):
        one = pb.make_params(h, hkv, L, 128)
        pb.prism_causal_csr(one, rp[ro[s]:], ci[co[s]:], co[s + 1] - co[s])
    out = torch.full((h, cu[-1], 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu) + (64 << 20))
    pb.prism_sparse_attn_varlen(params, cu, q, k, v, rp, ci, out, None, ws)
    torch.cuda.synchronize()
    for s in range(len(lens)):
        at = slice(cu[s], cu[s + 1])
        for i in (0, h - 1):
            _check_small_values(q[i, at], k[i // (h // hkv), at], v[i // (h // hkv), at], out[i, at])


@pytest.mark.parametrize("B,d", [(64, 64), (64, 128), (64, 256), (128, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("lens", [[200, 65, 127, 1], [129, 64, 190, 250]])
def test_values_behind_a_ragged_end_are_not_read(B, d, lens):
    """V of every other sequence of a packed batch, and of every other head, is NaN or infinite: what lies behind the last token of
    a sequence leaves no trace in it."""
    h = 3
    cu = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device="cuda").manual_seed(B + d)
    q, k, v = (torch.randn((h, cu[-1], d), generator=g, device="cuda").bfloat16() for _ in range(3))
    bad = torch.tensor([float("nan"), float("inf"), -float("inf")], device="cuda").bfloat16()
    for i in range(h):
        for s in range(len(lens)):
            if (i + s) % 2:
                v[i, cu[s]:cu[s + 1]] = bad[(i + s) % 3]
    bands = {64: (32, 48), 128: (64, 96), 256: (128, 192)}[d]
    params = pb.make_params(h, h, cu[-1], B, *bands, 0.9, 0, d)
    _, ro, co = pb.prism_varlen_layout(params, cu)
    rp = torch.zeros(ro[-1], dtype=torch.int32, device="cuda")
    ci = torch.zeros(co[-1], dtype=torch.int32, device="cuda")
    for s, L in enumerate(lens):
        pb.prism_causal_csr(pb.make_params(h, h, L, B, *bands, 0.9, 0, d), rp[ro[s]:], ci[co[s]:], co[s + 1] - co[s])
    out = torch.empty_like(q)
    ws = pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu))
    pb.prism_sparse_attn_varlen(params, cu, q, k, v, rp, ci, out, None, ws)
    torch.cuda.synchronize()
    for s in range(len(lens)):
        at = slice(cu[s], cu[s + 1])
        for i in range(h):
            if (i + s) % 2 == 0:
                x = (q[i, at].double() @ k[i, at].double().T) / np.sqrt(d)
                n = cu[s + 1] - cu[s]
                p = torch.softmax(x.masked_fill(torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1), -np.inf), -1)
                assert (out[i, at].double() - p @ v[i, at].double()).abs().max() <= OUT_TOL, (i, s)
