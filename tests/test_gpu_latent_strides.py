"""Latent attention over caches whose slots and pages are not packed, against
the fp64 oracle: the kernels form their own row addresses and load bounds from
the strides."""
import numpy as np
import pytest
import torch

import oracle.attention as OA
from paper_2606_04415_amd.workloads import WORKLOADS

from gpu_common import check_close, custom_batch, device_inputs, log, run

pytestmark = pytest.mark.gpu

MLA = WORKLOADS["mla"]


def padded(k):
    """Slots of 640 elements, three more slots a page; what no row holds is NaN."""
    big = torch.full((k.shape[0], k.shape[1] + 3, 1, 640), float("nan"), dtype=k.dtype)
    view = big[:, :k.shape[1], :, :576]
    view.copy_(k)
    return big, view


def slot_major(k):
    """The same slot of all pages side by side: the slot stride is far larger than the page stride."""
    big = k.permute(1, 0, 2, 3).contiguous()
    return big, big.permute(1, 0, 2, 3)


def overlapping(k):
    """A slot every 64 elements, so that a row shares all but 64 of them with the next."""
    pages, P = k.shape[:2]
    size = (pages * P - 1) * 64 + 576
    big = torch.randn(size, generator=torch.Generator().manual_seed(7)).to(k.dtype)
    return big, big.as_strided((pages, P, 1, 576), (P * 64, 64, 576, 1))


@pytest.mark.parametrize("hq", [64, 128])
@pytest.mark.parametrize("page", [16, 64])
@pytest.mark.parametrize("layout", [padded, slot_major, overlapping])
def test_strides(layout, page, hq):
    # one tile, a tile's end inside a wave's 8 rows, several tiles; prompts with cached keys
    ns, ls = [1, 1, 1, 1, 33, 130], [1, 29, 64, 203, 70, 150]
    b = custom_batch(MLA, ns, ls, seed=44, page_size=page, num_q_heads=hq)
    log(f"latent {layout.__name__} cache, page {page}, {hq} heads")
    big, _ = layout(b.k_cache)
    d = device_inputs(b)
    dev = big.cuda()
    host = big
    if layout is padded:
        k, b.k_cache = dev[:, :page, :, :576], host[:, :page, :, :576].contiguous()
    elif layout is slot_major:
        k, b.k_cache = dev.permute(1, 0, 2, 3), host.permute(1, 0, 2, 3).contiguous()
    else:
        shape, stride = b.k_cache.shape, (page * 64, 64, 576, 1)
        k, b.k_cache = dev.as_strided(shape, stride), host.as_strided(shape, stride).contiguous()
    d["k_cache"] = k
    out, lse, _ = run(b, d)
    w = b.workload
    ref_o, ref_l = OA.paged_attention(b.q, b.k_cache, None, b.block_table, b.seq_lens, b.query_start_loc, w.sm_scale,
                                      num_kv_heads=1, page_size=page, head_dim_v=512, v_aliases_k=True)
    rows = ~np.isnan(ref_l[:, 0])
    check_close(out, ref_o, "out", rows)
    check_close(lse, ref_l, "lse", rows)
