"""What hc_create takes of the device's memory.  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc

pytestmark = pytest.mark.gpu


def create(B, max_ctx, max_k):
    return hc.hc_create(hc.hc_config(B=B, Hq=32, Hkv=8, D=128, max_ctx=max_ctx, max_k=max_k, window=1, metric=0, tau_num=1, tau_den=2, agg=0, window_mode=0))


@pytest.mark.parametrize("B,max_ctx,max_k", [(1, 4096, 512), (1, 229376, 8192), (16, 131072, 8192), (16, 229376, 8192), (64, 131072, 8192), (4, 1 << 20, 40000)])
def test_context_memory(B, max_ctx, max_k):
    """At most what the header states: 4.5 B Hkv workspaces of 140 KB (131 KB of histograms, 8 KB) and max_ctx / 4 bytes, tables
    of 64 B Hkv max_k bytes, and 4 MB for what the allocator rounds up."""
    print("footprint", B, max_ctx, max_k, flush=True)
    hc.hc_destroy(create(1, 64, 1))                  # what the first context of a process loads
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = create(B, max_ctx, max_k)
    taken = before - torch.cuda.mem_get_info()[0]
    hc.hc_destroy(ctx)
    assert taken <= 4.5 * B * 8 * (140 * 1024 + max_ctx / 4) + 64 * B * 8 * max_k + (4 << 20), taken / 1e6
