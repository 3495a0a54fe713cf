"""Ragged last blocks at B = 128, d = 128 on the hand-scheduled kernel: tails of one token, around the 32 or 64
queries of a wave and one short of a block; causal and bidirectional; nothing written past the last row."""
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


# 64 heads x 33 blocks: four waves of 32 queries (a wave of the last block may start past the end); 128 heads: two of 64
@pytest.mark.parametrize("h,small_workspace", [(64, False), (64, True), (128, False)])
@pytest.mark.parametrize("tail,bidir", [(1, False), (32, True), (63, False), (64, True), (65, False), (65, True), (97, False),
                                        (127, True), (1, True)])
def test_ragged_last_block(tail, bidir, h, small_workspace):
    hkv, B, N = 2, 128, 33
    L = (N - 1) * B + tail
    print(f"case h={h} L={L} bidirectional={bidir} small workspace={small_workspace}", flush=True)
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
    if small_workspace:                                     # without room for the second V image: the general kernel
        need -= hkv * N * B * 128 * 2
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
    for n in (16, 8, 2):                                   # 336 and 168 rows, and 42, which the general kernel takes
        part = pb.make_params(n, hkv, L, B)
        _, rp, ci, _ = pb.alloc_estimate_outputs(part)
        pb.prism_causal_csr(part, rp, ci, ci.numel())
        qs = q.view(hkv, 16 // hkv, L, 128)[:, :n // hkv].reshape(n, L, 128).contiguous()
        out, lse = torch.empty_like(qs), torch.empty((n, L), device="cuda")
        pb.prism_sparse_attn_pre(part, qs, k, image, rp, ci, ci.numel(), out, lse)
        ref, ref_lse = gu.gpu_sparse_attn(part, qs, k, v, rp, ci, ci.numel())
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(lse, ref_lse), n
