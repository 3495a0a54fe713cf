"""The one-launch preparation of the attention (queue plan by a single workgroup, list check, V image): numbers of rows
at the edges of its steps (1024, 2048, 4096, 8192 rows) and just past them, up to where the separate kernels take over."""
import pytest

from tests.test_gpu_queues import test_every_row_is_queued_once_and_the_queues_are_balanced as check_queues
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


@pytest.mark.parametrize("h,hkv,N,dirty", [(16, 4, 256, False), (17, 1, 242, True), (32, 8, 256, False)])
def test_pair_queues_at_the_edges(h, hkv, N, dirty):
    check_pair_plan(h, hkv, N, dirty)    # 4096, 4114 and 8192 rows
