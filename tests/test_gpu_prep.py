"""The one-launch preparation of the attention (queue plan by a single workgroup, list check, V image): numbers of rows
at the edges of its steps (a multiple of 1024 up to 8192 rows) and just past them, up to where the separate kernels take over."""
import numpy as np
import pytest
import torch

from oracle import prism_oracle as orc
from paper_2602_08426_amd import binding as pb
from tests import gpu_util as gu
from tests.test_gpu_queues import test_every_row_is_queued_once_and_the_queues_are_balanced as check_queues
from tests.test_gpu_queues import _counters as queue_counters
from tests.test_gpu_queues import _layout as queue_layout
from tests.test_gpu_queues import test_pair_plan_at_block_64 as check_pair_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,hkv,L,B,bidir", [
    (8, 8, 128 * 128, 128, False),       # 1024 rows
    (5, 1, 128 * 205, 128, True),        # 1025
    (8, 2, 128 * 256, 128, False),       # 2048
    (3, 1, 64 * 683, 64, False),         # 2049, an odd number of 64-token blocks
    (17, 1, 128 * 241, 128, False),      # 4097
    (32, 8, 128 * 256, 128, False),      # 8192
    (33, 11, 128 * 249, 128, False),     # 8217: separate kernels
])
def test_queues_at_the_edges(h, hkv, L, B, bidir):
    check_queues(h, hkv, L, B, bidir, 7)


@pytest.mark.parametrize("h,hkv,N", [(12, 4, 256), (7, 1, 439), (20, 4, 256), (3, 1, 1707), (24, 8, 256), (5, 1, 1229), (28, 4, 256),
                                     (67, 1, 107)])
def test_queues_at_the_edges_of_the_rows_per_wave(h, hkv, N):
    check_queues(h, hkv, 128 * N, 128, False, 11)   # 3072, 3073, 5120, 5121, 6144, 6145, 7168 and 7169 rows


@pytest.mark.parametrize("h,hkv,N,dirty", [(16, 4, 256, False), (17, 1, 242, True), (32, 8, 256, False)])
def test_pair_queues_at_the_edges(h, hkv, N, dirty):
    check_pair_plan(h, hkv, N, dirty)    # 4096, 4114 and 8192 rows


@pytest.mark.parametrize("tail,bidir", [(64, False), (1, False), (33, True), (63, True)])
def test_rows_beyond_one_launch_have_the_bits_of_fewer(tail, bidir):
    """B = 64, an odd number of blocks: a call of 8385 rows has the bits of calls on its halves, whose masks another
    instance of the kernel forms, and agrees with the oracle."""
    h, N, B = 129, 65, 64
    L = (N - 1) * B + tail
    rng = np.random.default_rng(tail)
    g = torch.Generator(device="cuda").manual_seed(tail)
    q, k, v = (torch.randn((n, L, 128), generator=g, device="cuda").bfloat16() for n in (h, 1, 1))
    mask = rng.random((h, N, N)) < 0.3
    mask[:, np.arange(N), np.arange(N)] = True
    mask[:, N // 2, N - 1] = True                          # the ragged block (bidirectional rows)
    if not bidir:
        mask = np.tril(mask)
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0

    def run(heads):
        params = pb.make_params(len(heads), 1, L, B, flags=flags)
        rp, ci, cnt = gu.csr_to_device(*orc.mask_to_csr(mask[heads]))
        return gu.gpu_sparse_attn(params, q[heads].contiguous(), k, v, rp, ci, cnt)

    out, lse = run(range(h))
    for part in (range(64), range(64, h)):
        o, s = run(part)
        assert torch.equal(out[part].view(torch.int16), o.view(torch.int16)) and torch.equal(lse[part], s)
    Q, K, V = (t.float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    rows = {(i, u) for i in (0, h - 1) for u in (0, N // 2, N - 1)}
    ref = orc.block_sparse_attention(Q, K, V, mask, B, rows, causal=not bidir)
    for (i, u), (ro, _) in ref.items():                    # 2e-2: the bar of the other attention tests
        assert np.abs(gu.bf16_out_to_f64(out[i, u * B:(u + 1) * B]) - ro).max() <= 2e-2, (i, u)


@pytest.mark.parametrize("h,bidir", [(43, False), (44, False), (44, True)])
def test_wide_rows_beyond_one_workgroup_per_cu(h, bidir):
    """d = 256, B = 64, an odd number of blocks, 2795 and 2860 rows: the first call has a workgroup per CU, the others two.
    Every head has the bits of a call on a few heads, and agrees with the oracle."""
    N, B, d = 65, 64, 256
    L = (N - 1) * B + 7
    rng = np.random.default_rng(h)
    g = torch.Generator(device="cuda").manual_seed(h)
    q, k, v = (torch.randn((n, L, d), generator=g, device="cuda").bfloat16() for n in (h, 1, 1))
    mask = rng.random((h, N, N)) < 0.2
    mask[:, np.arange(N), np.arange(N)] = True
    if not bidir:
        mask = np.tril(mask)
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0

    def run(heads):
        params = pb.make_params(len(heads), 1, L, B, 128, 192, 0.9, flags, d)
        rp, ci, cnt = gu.csr_to_device(*orc.mask_to_csr(mask[heads]))
        return gu.gpu_sparse_attn(params, q[heads].contiguous(), k, v, rp, ci, cnt)

    out, lse = run(range(h))
    for part in (range(8), range(h - 5, h)):
        o, s = run(part)
        assert torch.equal(out[part].view(torch.int16), o.view(torch.int16)) and torch.equal(lse[part], s)
    Q, K, V = (t.float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    rows = {(i, u) for i in (0, h - 1) for u in (0, N // 2, N - 1)}
    ref = orc.block_sparse_attention(Q, K, V, mask, B, rows, causal=not bidir)
    for (i, u), (ro, _) in ref.items():                    # 2e-2: the bar of the other attention tests
        assert np.abs(gu.bf16_out_to_f64(out[i, u * B:(u + 1) * B]) - ro).max() <= 2e-2, (i, u)


@pytest.mark.parametrize("h,bidir", [(15, False), (16, True)])
def test_wide_rows_of_short_calls(h, bidir):
    """975 and 1040 rows: one workgroup per CU, and two or one by the lists."""
    test_wide_rows_beyond_one_workgroup_per_cu(h, bidir)


@pytest.mark.parametrize("h,tail,bidir", [(43, 64, False), (44, 64, False), (44, 7, False), (45, 1, True)])
def test_wide_pairs(h, tail, bidir):
    """d = 256, B = 64, 64 blocks: 2752 rows in the plain form, 2816 and 2880 in pairs, whose unions have from one block to all.
    Every head has the bits of a call on a few heads, which is plain, and agrees with the oracle."""
    N, B, d = 64, 64, 256
    L = (N - 1) * B + tail
    rng = np.random.default_rng(h + tail)
    g = torch.Generator(device="cuda").manual_seed(h)
    q, k, v = (torch.randn((n, L, d), generator=g, device="cuda").bfloat16() for n in (h, 1, 1))
    mask = rng.random((h, N, N)) < np.array([0.0, 0.03, 0.2, 0.9])[np.arange(h) % 4, None, None]
    mask[:, np.arange(N), np.arange(N)] = True
    mask[1, :, N - 1] = True
    mask[5, 10] = False                                    # an empty list beside a full one, and two empty ones
    mask[5, 20:22] = False
    if not bidir:
        mask = np.tril(mask)
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0

    def run(heads):
        params = pb.make_params(len(heads), 1, L, B, 128, 192, 0.9, flags, d)
        rp, ci, cnt = gu.csr_to_device(*orc.mask_to_csr(mask[heads]))
        return gu.gpu_sparse_attn(params, q[heads].contiguous(), k, v, rp, ci, cnt)

    out, lse = run(range(h))
    for part in (range(8), range(h - 5, h)):
        o, s = run(part)
        assert torch.equal(out[part].view(torch.int16), o.view(torch.int16)) and torch.equal(lse[part], s)
    Q, K, V = (t.float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    rows = {(i, u) for i in (0, 1, 2, 3, h - 1) for u in (0, 1, N // 2, N - 1)}
    ref = orc.block_sparse_attention(Q, K, V, mask, B, rows, causal=not bidir)
    for (i, u), (ro, _) in ref.items():                    # 2e-2: the bar of the other attention tests
        assert np.abs(gu.bf16_out_to_f64(out[i, u * B:(u + 1) * B]) - ro).max() <= 2e-2, (i, u)


@pytest.mark.parametrize("dirty", [False, True])
def test_pair_queues_of_the_separate_kernels(dirty):
    check_pair_plan(33, 11, 250, dirty)  # 8250 rows: the counters of both plans are written by the last launch that fills one


@pytest.mark.parametrize("tail,longest", [(128, 4), (128, None), (5, 4)])
def test_rows_that_have_a_cu_to_themselves(tail, longest):
    """576 rows at B = 128, whole blocks (four waves of 32 queries) and ragged (general kernel).  With one head of full
    lists its longest rows are marked and the workgroups that would share their CUs end at once: every row is still done
    once, with the bits of calls on single heads, which mark none, and the oracle's values.  Without it no row is marked."""
    h, N, B = 9, 64, 128
    L = (N - 1) * B + tail
    rng = np.random.default_rng(3)
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((n, L, 128), generator=g, device="cuda").bfloat16() for n in (h, 1, 1))
    mask = rng.random((h, N, N)) < 0.03
    mask[:, np.arange(N), np.arange(N)] = True
    if longest is not None:
        mask[longest] = True
    mask = np.tril(mask)

    def run(heads):
        params = pb.make_params(len(heads), 1, L, B)
        rp, ci, cnt = gu.csr_to_device(*orc.mask_to_csr(mask[heads]))
        out = torch.full_like(q[heads], float("nan"))
        lse = torch.full((len(heads), L), float("nan"), device="cuda")
        ws = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(params))
        pb.prism_sparse_attn(params, q[heads].contiguous(), k, v, rp, ci, cnt, out, lse, ws)
        torch.cuda.synchronize()
        at = queue_layout(len(heads), 1, N, B, L)["plan"]
        return out, lse, ws[at:at + 160].cpu().numpy().view(np.uint32)

    out, lse, plan = run(list(range(h)))
    marked = sum(bin(int(w)).count("1") for w in plan[32:40])
    lens = mask.sum(-1)
    line = 1.4 * (lens.sum() + 3 * h * N) / (2 * torch.cuda.get_device_properties(0).multi_processor_count)
    assert marked == (lens > line).sum() and (marked >= 32 if longest is not None else marked == 0)
    for i in range(h):
        o, s, alone = run([i])
        assert (alone[32:40] == 0).all()                   # 64 rows: one workgroup each
        assert torch.equal(out[i].view(torch.int16), o[0].view(torch.int16)) and torch.equal(lse[i], s[0]), i
    Q, K, V = (t.float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    rows = {(i, u) for i in (0, 4) for u in (0, N // 2, N - 1)}
    ref = orc.block_sparse_attention(Q, K, V, mask, B, rows)
    for (i, u), (ro, _) in ref.items():                    # 2e-2: the bar of the other attention tests
        assert np.abs(gu.bf16_out_to_f64(out[i, u * B:(u + 1) * B]) - ro).max() <= 2e-2, (i, u)


def _marks(raw, lay, row_ptr, h, N, cus):
    """The marks of a plan, and those it should have by its queues and lists: bit p of queue x where its p-th row is longer
    than 1.4 times the work of an average workgroup, in queues with no more such rows than 5/8 of the CUs of an XCD."""
    plan = raw[lay["plan"]:lay["plan"] + 160].view(np.int32)
    items = raw[lay["items"]:lay["items"] + h * N * 16].view(np.int32).reshape(-1, 4)
    lens = np.diff(row_ptr)
    line = np.float32(1.4) * np.float32(lens.sum() + 3 * h * N) / np.float32(2 * cus)
    want = []
    for x in range(8):
        rows = items[plan[x]:plan[x] + plan[8 + x]]
        long = lens[rows[:, 0] * N + (rows[:, 1] & 0xffff)] > line
        want.append(sum(1 << p for p in np.nonzero(long[:cus // 8])[0]) if long.sum() <= cus // 8 * 5 // 8 else 0)
    return plan[32:40].view(np.uint32).tolist(), want


@pytest.mark.parametrize("h,N,tail,d,n_long,some,dirty", [
    (8, 100, 128, 128, 300, False, False),      # three heads of full lists: more long rows than CUs; four waves of 32 queries
    (8, 100, 128, 128, 96, True, False),
    (8, 100, 128, 128, 96, True, True),         # the general kernel with the second set of counters
    (8, 100, 9, 128, 300, False, False),        # the general kernel alone
    (8, 100, 9, 128, 96, True, False),
    (14, 300, 128, 128, 264, False, False),     # two waves of 64 queries
    (14, 300, 128, 128, 160, True, False),      # 20 a queue
    (14, 300, 128, 128, 40, True, True),
    (8, 100, 9, 64, 300, False, False),
    (8, 100, 9, 64, 96, True, True),
    (32, 40, 128, 64, 8, True, False),
])
def test_long_rows_share_their_cus_where_they_are_many(h, N, tail, d, n_long, some, dirty):
    """Bidirectional calls of n_long lists of N blocks among lists of one: the plan marks the long rows that it should, and
    every row has the bits of calls on single heads, which mark none."""
    B, L = 128, (N - 1) * 128 + tail
    rng = np.random.default_rng(h + n_long)
    lens = np.ones(h * N, np.int64)
    lens[rng.choice(h * N, n_long, replace=False) if some else np.arange(n_long)] = N
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col_idx = np.concatenate([np.arange(N) if n > 1 else [r % N] for r, n in enumerate(lens)]).astype(np.int32)
    if dirty:
        col_idx[row_ptr[np.nonzero(lens == N)[0][3]]] = -1
    g = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn((n, L, d), generator=g, device="cuda").bfloat16() for n in (h, 1, 1))
    bands = {64: (32, 48), 128: (64, 96)}[d]

    def run(heads):
        # one head's lists may be clean where the call's are not: then the same kernel by the flag
        flags = pb.PRISM_FLAG_BIDIRECTIONAL | (pb.PRISM_FLAG_GENERAL_KERNEL if dirty and len(heads) < h else 0)
        params = pb.make_params(len(heads), 1, L, B, *bands, 0.9, flags, d)
        at = row_ptr[heads[0] * N]
        rp, ci = row_ptr[heads[0] * N:(heads[-1] + 1) * N + 1] - at, col_idx[at:row_ptr[(heads[-1] + 1) * N]]
        out = torch.full_like(q[heads], float("nan"))
        ws = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(params))
        pb.prism_sparse_attn(params, q[heads].contiguous(), k, v, *gu.csr_to_device(rp, ci), out, None, ws)
        torch.cuda.synchronize()
        return out, ws.cpu().numpy()

    out, raw = run(list(range(h)))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    got, want = _marks(raw, queue_layout(h, 1, N, B, L, d), row_ptr, h, N, cus)
    assert got == want and any(want) == some, (got, want)
    for i in range(h):
        assert torch.equal(out[i].view(torch.int16), run([i])[0][0].view(torch.int16)), i


@pytest.mark.parametrize("h,hkv,N,tail,bidir,ratio,halved", [
    (16, 8, 177, 7, False, 1.19, True), (16, 8, 177, 7, False, 1.21, False),
    (16, 2, 177, 33, True, 1.19, True), (16, 2, 177, 64, True, 1.21, False),
])
def test_wide_rows_bound_by_the_longest_have_a_cu_to_themselves(h, hkv, N, tail, bidir, ratio, halved):
    """d = 256, B = 64, 2832 rows: two workgroups per CU, the second of which end at once where the longest row bounds the
    call.  Every row is done once, with the bits of calls on a few heads, and of the oracle in value."""
    B, d, L = 64, 256, (N - 1) * 64 + tail
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(h)
    # one list of N blocks, the others up to 40, until a CU's average work is `ratio` times N
    lens = np.ones((h, N), np.int64)
    most = np.minimum(40, np.full(N, N) if bidir else np.arange(N) + 1)
    lens[3, N - 1] = N
    spare = int(ratio * N * cus) - 3 * h * N - int(lens.sum())
    for r in rng.permutation(h * N):
        i, u = divmod(int(r), N)
        if lens[i, u] == 1:
            more = min(int(most[u]) - 1, spare)
            lens[i, u] += more
            spare -= more
    assert spare == 0
    lens = lens.reshape(-1)
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    mask = np.zeros((h, N, N), bool)
    for r, n in enumerate(lens):
        i, u = divmod(r, N)
        top = N if bidir else u + 1
        mask[i, u, (u - np.arange(n)) % top] = True        # the row's own block among them
    row_ptr, col_idx = orc.mask_to_csr(mask)
    assert (np.diff(row_ptr) == lens).all()
    g = torch.Generator(device="cuda").manual_seed(h)
    q, k, v = (torch.randn((n, L, d), generator=g, device="cuda").bfloat16() for n in (h, hkv, hkv))
    flags = pb.PRISM_FLAG_BIDIRECTIONAL if bidir else 0

    def run(heads, kv):
        params = pb.make_params(len(heads), len(kv), L, B, 128, 192, 0.9, flags, d)
        out = torch.full_like(q[heads], float("nan"))
        ws = pb.alloc_workspace(pb.prism_sparse_attn_workspace_bytes(params))
        pb.prism_sparse_attn(params, q[heads].contiguous(), k[kv].contiguous(), v[kv].contiguous(),
                             *gu.csr_to_device(*orc.mask_to_csr(mask[heads])), out, None, ws)
        torch.cuda.synchronize()
        at = queue_layout(len(heads), len(kv), N, B, L, d)["plan"]
        return out, ws[at:at + 160].cpu().numpy().view(np.uint32)[32:40]

    out, alone = run(list(range(h)), list(range(hkv)))
    assert (alone == (0xffffffff >> (32 - cus // 8) if halved else 0)).all(), alone
    for i in (0, 3, h - 1):
        o, few = run([i], [i // (h // hkv)])
        assert (few == 0).all() and torch.equal(out[i].view(torch.int16), o[0].view(torch.int16)), i
    assert not torch.isnan(out).any()
    Q, K, V = (t.float().cpu().numpy().astype(np.float64) for t in (q, k, v))
    rows = {(3, N - 1), (0, 0), (h - 1, N // 2)}
    ref = orc.block_sparse_attention(Q, K, V, mask, B, rows, causal=not bidir)
    for (i, u), (ro, _) in ref.items():                    # 2e-2: the bar of the other attention tests
        assert np.abs(gu.bf16_out_to_f64(out[i, u * B:(u + 1) * B]) - ro).max() <= 2e-2, (i, u)


@pytest.mark.parametrize("dirty", [0, 1])
def test_rows_that_another_kernel_takes_hold_no_cu(dirty):
    """A packed batch of two, 752 rows: the first holds the long rows, and one of the two has a list with an entry to skip.
    Where the launch does not take the long rows, the workgroups on their CUs go on: every workgroup pulls its queue to the end."""
    h, B, Ns = 8, 128, [64, 30]
    flat = [np.arange(u + 1) if i == 5 else np.array([u]) for i in range(h) for u in range(Ns[0])]
    short = [np.arange(max(0, u - 2), u + 1) for i in range(h) for u in range(Ns[1])]
    cu = [0, 128 * Ns[0], 128 * sum(Ns)]
    g = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn((n, cu[-1], 128), generator=g, device="cuda").bfloat16() for n in (h, 2, 2))
    params = pb.make_params(h, 2, cu[-1], B)
    mo, ro, co = pb.prism_varlen_layout(params, cu)
    rp, ci = np.zeros(ro[-1], np.int32), np.zeros(co[-1], np.int32)
    csr = []
    for s, lists in enumerate((flat, short)):
        lists = [c.astype(np.int32) for c in lists]
        if s == dirty:
            lists[7] = np.concatenate([[-1], lists[7]]).astype(np.int32)
        row_ptr = np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int32)
        csr.append((row_ptr, np.concatenate(lists)))
        rp[ro[s]:ro[s] + len(row_ptr)] = row_ptr
        ci[co[s]:co[s] + row_ptr[-1]] = csr[s][1]
    out = torch.full_like(q, float("nan"))
    lse = torch.full(q.shape[:2], float("nan"), device="cuda")
    ws = pb.alloc_workspace(pb.prism_sparse_attn_varlen_workspace_bytes(params, cu) + (64 << 20))
    pb.prism_sparse_attn_varlen(params, cu, q, k, v, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), out, lse, ws)
    torch.cuda.synchronize()
    for s in range(2):
        ps = pb.make_params(h, 2, cu[s + 1] - cu[s], B)
        o, l = gu.gpu_sparse_attn(ps, *(x[:, cu[s]:cu[s + 1]].contiguous() for x in (q, k, v)), *gu.csr_to_device(*csr[s]))
        assert torch.equal(out[:, cu[s]:cu[s + 1]].view(torch.int16), o.view(torch.int16)), s
        assert torch.equal(lse[:, cu[s]:cu[s + 1]], l), s
    lay, raw = queue_layout(h, 2, sum(Ns), B), ws.cpu().numpy()
    plan = raw[lay["plan"]:lay["plan"] + 160].view(np.uint32)
    length, marks = plan[8:16].astype(int), [bin(int(w)).count("1") for w in plan[32:40]]
    assert sum(marks) >= 32 and plan[24] == 1
    each = 2 * torch.cuda.get_device_properties(0).multi_processor_count // 8
    assert (length >= each).all()
    # a workgroup that goes on meets the end of its queue once, by a pull; the others end without one
    for n, done in enumerate(queue_counters(raw, lay)):
        ended = marks if n == 0 and dirty == 1 else [0] * 8    # only beside long rows that the first kernel takes
        for x in range(8):
            assert done[x] >= length[x] + each - ended[x], (n, x, done, length, marks)
