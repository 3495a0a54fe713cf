"""Performance cases: calls of the public entry points as a prefill program makes them.

A pass is one attention layer's prefill (block-importance estimation, then block-sparse attention over
the lists it wrote) or, for kind "rope", the estimation fused with the producer of the rotated tensors.
Inputs come from paper_2602_08426_amd.workloads (planted sink / local / slash / stripe structure after
RoPE), buffers and workspaces are allocated once as a serving program would, and no call waits for the
device.  Nothing here is used by the library.

Kinds
  layer   prism_estimate + prism_sparse_attn
  video   prism_estimate_bands (axis-wise bands) + prism_sparse_attn, bidirectional
  varlen  prism_estimate_varlen + prism_sparse_attn_varlen over a packed batch
  rope    prism_rope_estimate (rotation, pooling and selection in one call; no attention)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_08426_amd import binding as pb
from paper_2602_08426_amd import workloads as wl

# three axis subspaces of 16, 56 and 56 dims: the first 8 / 32 / 32 and the last 16 / 36 / 36 of each
AXIS_HIGH = ((0, 8), (16, 32), (72, 32))
AXIS_LOW = ((0, 16), (36, 36), (92, 36))
# NTK-by-parts frequencies: native length, scale, alpha, beta
YARN = (32768, 4.0, 1.0, 32.0)
# bands of each head dim (first d_high, last d_low dims)
BANDS = {64: (32, 48), 128: (64, 96), 256: (128, 192)}


def _case(kind, h, h_kv, seq_len, block, *, head_dim=128, top_p=0.95, base=5.0e5, sigma=0.0, amp=0.7,
          recipe="mixed", lse=True, lens="", yarn=False):
    return dict(kind=kind, h=h, h_kv=h_kv, seq_len=seq_len, block=block, head_dim=head_dim, top_p=top_p,
                base=base, sigma=sigma, amp=amp, recipe=recipe, lse=lse, lens=lens, yarn=yarn)


def listed():
    lens = "8192,1500,4096,77,12288,3001,640,5000"
    return [
        # the smallest call of the test workloads: one head, 2K tokens; launches and latency are all there is
        dict(_case("layer", 1, 1, 2048, 64, base=1.0e4, amp=1.0, recipe="slash16"), name="layer_2k_1head_b64"),
        # one layer of a 32 / 8 head decoder at a short, an ordinary and the longest prompt
        dict(_case("layer", 32, 8, 8192, 128, amp=0.8), name="layer_8k"),
        dict(_case("layer", 32, 8, 32768, 128), name="layer_32k"),
        dict(_case("layer", 32, 8, 131072, 128, amp=0.6), name="layer_128k"),
        # a 28 / 4 head decoder (groups of seven) with heavy-tailed keys
        dict(_case("layer", 28, 4, 65536, 128, top_p=0.93, base=1.0e6, sigma=0.75, amp=0.55), name="layer_64k_28_4"),
        # a prompt of no particular length: ragged last block, as prompts mostly are
        dict(_case("layer", 32, 8, 20011, 128, amp=0.75), name="layer_20011"),
        # the finer block size of the block-size study
        dict(_case("layer", 32, 8, 32768, 64), name="layer_32k_b64"),
        # the smaller and the larger head size
        dict(_case("layer", 32, 8, 12345, 128, head_dim=64, amp=0.75), name="layer_12345_d64"),
        dict(_case("layer", 16, 4, 16384, 64, head_dim=256, amp=0.75, lse=False), name="layer_16k_d256_b64"),
        # a packed batch of prompts of unequal lengths
        dict(_case("varlen", 32, 8, sum(map(int, lens.split(","))), 128, amp=0.75, lens=lens), name="varlen_8_prompts"),
        # estimation fused with a YaRN-extended rotary embedding
        dict(_case("rope", 28, 4, 65536, 128, top_p=0.93, base=1.0e6, amp=0.55, yarn=True), name="rope_64k_yarn"),
        # bidirectional attention with axis-wise bands, one kv head per q-head (video generation)
        dict(_case("video", 16, 16, 19290, 128, top_p=0.9, amp=0.7, lse=False), name="video_19290"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: kind, heads, block, head size, options and a length spread over its logarithm."""
    kind = rng.choice(["layer", "layer", "layer", "varlen", "rope", "video"])
    h, h_kv = rng.choice([(1, 1), (8, 2), (7, 1), (16, 4), (28, 4), (32, 8)])
    block = rng.choice([64, 128, 128])
    head_dim = rng.choice([64, 128, 128, 128, 256]) if kind in ("layer", "varlen") else 128
    lse = rng.random() < 0.5
    top_p = rng.choice([0.9, 0.93, 0.95, 0.95])
    if kind == "video":
        h = h_kv = rng.choice([4, 8, 16])
    # a drawn case costs no more than the longest listed one: 128K tokens at 32 heads of 128 dims
    most = 131072 if kind in ("layer", "rope") and head_dim == 128 else 32768
    lens = ""
    if kind == "varlen":
        parts = [_log_uniform(rng, 64, 16384) for _ in range(rng.randint(2, 12))]
        lens, seq_len = ",".join(map(str, parts)), sum(parts)
    else:
        seq_len = _log_uniform(rng, 1024, most)
        if rng.random() < 0.4:                     # whole blocks: a padded or chunked prompt
            seq_len = -(-seq_len // block) * block
    amp = min(0.8, max(0.6, 0.8 - 0.05 * math.log2(max(seq_len, 1) / 8192)))
    return _case(kind, h, h_kv, seq_len, block, head_dim=head_dim, top_p=top_p, base=rng.choice([5.0e5, 1.0e6]),
                 sigma=rng.choice([0.0, 0.0, 0.75]), amp=round(amp, 3), lse=lse, lens=lens,
                 yarn=kind == "rope" and rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------------------------------
def _workload(case, seq_len, seed):
    d_high, d_low = BANDS[case["head_dim"]]
    return wl.Workload("perf", case["h"], case["h_kv"], seq_len, case["block"], case["base"], case["top_p"],
                       int(seed) % (1 << 31), case["recipe"], head_dim=case["head_dim"], d_high=d_high, d_low=d_low,
                       k_lognormal_sigma=case["sigma"], amp_scale=case["amp"], yarn=YARN if case["yarn"] else None)


def _tensors(case, seed):
    """(q, k, v) on the device; before the rotation for kind "rope"."""
    if case["kind"] != "varlen":
        bits = wl.generate(_workload(case, case["seq_len"], seed), n_threads=16, rotate=case["kind"] != "rope")
        return tuple(pb.bf16_bits_to_device(b) for b in bits)
    parts = []
    for i, n in enumerate(map(int, case["lens"].split(","))):
        w = _workload(case, max(n, 256), (int(seed) + 7919 * i))          # the planted patterns need some length
        parts.append([pb.bf16_bits_to_device(np.ascontiguousarray(b[:, :n])) for b in wl.generate(w, n_threads=16)])
    return tuple(torch.cat([p[j] for p in parts], dim=1) for j in range(3))


def _params(case):
    d_high, d_low = BANDS[case["head_dim"]]
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if case["kind"] == "video" else 0
    return pb.make_params(case["h"], case["h_kv"], case["seq_len"], case["block"], d_high, d_low, case["top_p"],
                          flags, case["head_dim"])


def prepare(case, seed):
    q, k, v = _tensors(case, seed)
    params = _params(case)
    s = dict(kind=case["kind"], params=params, q=q, k=k, v=v)
    if case["kind"] == "varlen":
        cu = [0]
        for n in map(int, case["lens"].split(",")):
            cu.append(cu[-1] + n)
        s["cu"] = cu
        mo, ro, co = pb.prism_varlen_layout(params, cu)
        s["mask"] = torch.zeros(mo[-1], dtype=torch.int64, device="cuda")
        s["row_ptr"] = torch.zeros(ro[-1], dtype=torch.int32, device="cuda")
        s["col_idx"] = torch.zeros(co[-1], dtype=torch.int32, device="cuda")
        s["info"] = torch.zeros(4 * (len(cu) - 1), dtype=torch.int32, device="cuda")
        s["est_ws"] = pb.alloc_workspace(pb.prism_estimate_varlen_workspace_bytes(params, cu))
        s["attn_ws"] = pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu))
    else:
        s["mask"], s["row_ptr"], s["col_idx"], s["info"] = pb.alloc_estimate_outputs(params)
        s["col_idx"].zero_()                       # the lists fill only a part of it; the rest stays as it is here
        s["est_ws"] = pb.alloc_workspace(pb.prism_estimate_workspace_bytes(params))
    if case["kind"] == "rope":
        s["rope"] = pb.make_rope(case["base"], 0, *(YARN if case["yarn"] else ()))
        s["q_out"], s["k_out"] = torch.empty_like(q), torch.empty_like(k)
        return s
    if case["kind"] != "varlen":
        s["attn_ws"] = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(params))
    if case["kind"] == "video":
        s["bands"] = pb.make_bands(AXIS_HIGH, AXIS_LOW)
    s["out"] = torch.empty_like(q)
    s["lse"] = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda") if case["lse"] else None
    return s


def run(s):
    p, q, k, v = s["params"], s["q"], s["k"], s["v"]
    mask, row_ptr, col_idx, info = s["mask"], s["row_ptr"], s["col_idx"], s["info"]
    r = dict(mask=mask, row_ptr=row_ptr, col_idx=col_idx, info=info)
    if s["kind"] == "varlen":
        pb.prism_estimate_varlen(p, s["cu"], q, k, mask, row_ptr, col_idx, info, s["est_ws"])
        pb.prism_sparse_attn_varlen(p, s["cu"], q, k, v, row_ptr, col_idx, s["out"], s["lse"], s["attn_ws"])
        return dict(r, out=s["out"], lse=s["lse"])
    cap = col_idx.numel()
    if s["kind"] == "rope":
        pb.prism_rope_estimate(p, s["rope"], None, q, k, s["q_out"], s["k_out"], mask, row_ptr, col_idx, cap, info,
                               s["est_ws"])
        return dict(r, q_out=s["q_out"], k_out=s["k_out"])
    if s["kind"] == "video":
        pb.prism_estimate_bands(p, s["bands"], q, k, mask, row_ptr, col_idx, cap, info, s["est_ws"])
    else:
        pb.prism_estimate(p, q, k, mask, row_ptr, col_idx, cap, info, s["est_ws"])
    # the number of entries stays on the device: the capacity bounds it
    pb.prism_sparse_attn(p, q, k, v, row_ptr, col_idx, cap, s["out"], s["lse"], s["attn_ws"])
    return dict(r, out=s["out"], lse=s["lse"])


# ---- what a pass cannot do without ------------------------------------------------------------------
# Share of the admissible block pairs that the selection keeps on these inputs (0.09 - 0.2 over the
# lengths and heads above); the true share depends on the data.
DENSITY = 0.15


def work(case):
    h, h_kv, d, B = case["h"], case["h_kv"], case["head_dim"], case["block"]
    lens = [int(n) for n in case["lens"].split(",")] if case["lens"] else [case["seq_len"]]
    d_high, d_low = BANDS[d]
    n_bytes = flops = 0.0
    for L in lens:
        N = -(-L // B)
        pairs = h * N * N if case["kind"] == "video" else h * N * (N + 1) / 2
        kept = max(DENSITY * pairs, h * N)                  # at least one block per row
        row = 2.0 * L * d
        n_bytes += row * (h + h_kv)                         # q, k in
        n_bytes += h * N * (8 * -(-N // 64) + 4) + 4 * kept  # bit rows and lists out
        flops += 2.0 * pairs * (d_high + d_low) + 2.0 * L * d * (h + h_kv)
        if case["kind"] == "rope":
            n_bytes += row * (h + h_kv)                     # rotated q, k out
        else:
            n_bytes += row * (h + h_kv) + (4 * h * L if case["lse"] else 0)   # v in, o out
            flops += 4.0 * B * B * d * kept
    return dict(bytes=n_bytes, flops=flops)


def tolerance(case):
    # Lists and bits are whole numbers and stay the same.  out is bf16 with P rounded to bf16 or fp16
    # in front of the P V product (8 or 11 significant bits), lse is fp32.
    return dict(rel=1.0e-2, max=0.05)


# ---- the same in 64 bits ------------------------------------------------------------------------------
def _rotate64(x, case):
    """Adjacent pairs (2j, 2j+1) of x [heads, L, d] turned by position * theta_j, in 64 bits."""
    d = x.shape[-1]
    theta = case["base"] ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    if case["yarn"]:
        native, scale, alpha, beta = YARN
        keep = ((native * theta / (2 * math.pi) - alpha) / (beta - alpha)).clamp(0.0, 1.0)
        theta = (1.0 - keep) * theta / scale + keep * theta
    ang = torch.arange(x.shape[1], dtype=torch.float64, device=x.device)[:, None] * theta[None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    out = torch.empty(x.shape, dtype=torch.float64, device=x.device)
    for i in range(x.shape[0]):
        a, b = x[i, :, 0::2].double(), x[i, :, 1::2].double()
        out[i, :, 0::2] = a * c - b * s
        out[i, :, 1::2] = a * s + b * c
    return out


def _pool64(x, B):
    L, d = x.shape
    N = -(-L // B)
    y = torch.zeros((N * B, d), dtype=torch.float64, device=x.device)
    y[:L] = x.double()
    count = torch.full((N, 1), float(B), dtype=torch.float64, device=x.device)
    count[-1] = L - (N - 1) * B
    return y.view(N, B, d).sum(1) / count


def _select64(q, k, case, bands, causal):
    """[N, N] bool: blocks kept for one q-head and its kv head."""
    B, p = case["block"], case["top_p"]
    qp, kp = _pool64(q, B), _pool64(k, B)
    N, d = qp.shape
    rms = lambda t: t.square().mean().sqrt()                                   # noqa: E731
    keep = torch.zeros((N, N), dtype=torch.bool, device=q.device)
    for dims in bands:
        qz, kz = qp[:, dims], kp[:, dims]
        dz = len(dims)
        tau = math.sqrt(dz / d) * (rms(qz) / rms(qp)) * (rms(kz) / rms(kp))
        s = (qz @ kz.T) / (math.sqrt(dz) * tau)
        if causal:
            s = s.masked_fill(torch.ones_like(keep).triu(1), -math.inf)
        w, order = torch.sort(torch.softmax(s, -1), dim=-1, descending=True, stable=True)
        take = (w.cumsum(-1) - w < p) & (w > 0)
        keep |= torch.zeros_like(keep).scatter(1, order, take)
    return keep


def _attend64(q, k, v, keep, case, causal, out, lse):
    """out [L, d], lse [L] (or None) of one head; a strip of query blocks at a time."""
    L, d = q.shape
    B = case["block"]
    k64, v64 = k.double(), v.double()
    rows = max(B, min(L, (1 << 27) // L) // B * B)
    for r0 in range(0, L, rows):
        r1 = min(L, r0 + rows)
        c1 = r1 if causal else L
        s = (q[r0:r1].double() @ k64[:c1].T) / math.sqrt(d)
        allowed = keep[r0 // B:-(-r1 // B), :-(-c1 // B)]
        allowed = allowed.repeat_interleave(B, 0)[:r1 - r0].repeat_interleave(B, 1)[:, :c1]
        if causal:
            at = torch.arange(r0, r1, device=q.device)[:, None] >= torch.arange(c1, device=q.device)[None, :]
            allowed = allowed & at
        s.masked_fill_(~allowed, -math.inf)
        m = s.amax(-1, keepdim=True)
        e = s.sub_(m).exp_()
        total = e.sum(-1, keepdim=True)
        out[r0:r1] = (e @ v64[:c1]) / total
        if lse is not None:
            lse[r0:r1] = (m + total.log())[:, 0]


def exact(case, seed):
    q, k, v = _tensors(case, seed)
    h, h_kv, d = case["h"], case["h_kv"], case["head_dim"]
    none = dict(mask=None, row_ptr=None, col_idx=None, info=None)
    if case["kind"] == "rope":
        return dict(none, q_out=_rotate64(q, case), k_out=_rotate64(k, case))
    causal = case["kind"] != "video"
    if causal:
        d_high, d_low = BANDS[d]
        bands = [list(range(d_high)), list(range(d - d_low, d))]
    else:
        bands = [[i for a, n in seg for i in range(a, a + n)] for seg in (AXIS_HIGH, AXIS_LOW)]
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=q.device) if case["lse"] else None
    at = 0
    for n in map(int, case["lens"].split(",")) if case["lens"] else [case["seq_len"]]:
        for i in range(h):
            j = i // (h // h_kv)
            span = slice(at, at + n)
            keep = _select64(q[i, span], k[j, span], case, bands, causal)
            _attend64(q[i, span], k[j, span], v[j, span], keep, case, causal, out[i, span],
                      lse[i, span] if lse is not None else None)
        at += n
    return dict(none, out=out, lse=lse)
