"""Long contexts and the largest decode ranges, on the GPU through the C ABI.

Prefill rows and latent decode pieces stage the block table in LDS windows
of 512 entries (8192 keys at page 16, 32768 at page 64), latent rows in groups
of 128 in windows of 2048, and drain the tile pipeline at each window's end;
grouped-query decode stages a whole balanced range, up to 8192 pages. These
cases cross windows and use one range for the whole batch (cus_total = 1 in
the plan options), against the fp64 oracle.
"""
import math

import numpy as np
import pytest

import oracle.attention as OA
from paper_2606_04415_amd import flexattn as F
from paper_2606_04415_amd.workloads import WORKLOADS

from gpu_common import check_close, custom_batch, log, run

pytestmark = pytest.mark.gpu

QW = WORKLOADS["decode"]
MLA = WORKLOADS["mla"]


def full_check(b, opts, what):
    w = b.workload
    out, lse, pa = run(b, opts=opts)
    ref_o, ref_l = OA.paged_attention(b.q, b.k_cache, b.v_cache, b.block_table, b.seq_lens, b.query_start_loc,
                                      w.sm_scale, num_kv_heads=w.num_kv_heads, page_size=w.page_size,
                                      head_dim_v=w.head_dim_v, v_aliases_k=w.v_aliases_k)
    rows = ~np.isnan(ref_l[:, 0])
    check_close(out, ref_o, f"{what} out", rows)
    check_close(lse, ref_l, f"{what} lse", rows)
    return pa


def favour_keys(b, s, first, units):
    """Raises the scores of sequence s's keys from `first` on by `units` (log2),
    through the last 64 columns of latent keys, which are no part of the
    values: so few keys past a window's edge then make up much of the result."""
    w = b.workload
    per = 64 * w.sm_scale * math.log2(math.e)
    b.q[:, :, 512:] = 1.0
    for t in range(int(b.seq_lens[s])):
        if t >= first or t % w.page_size == 0:   # keys before: their page is enough to clear once
            page, slot = int(b.block_table[s, t // w.page_size]), t % w.page_size
            if t >= first:
                b.k_cache[page, slot, :, 512:] = units / per
            else:
                b.k_cache[page, :, :, 512:] = 0.0


def test_prefill_across_page_windows():
    # 70 new tokens after 19930 cached ones: 1250 pages, three LDS windows;
    # plus decodes over 20000 and 8193 keys
    ns, ls = [70, 1, 1], [20000, 20000, 8193]
    b = custom_batch(QW, ns, ls, seed=31)
    log("GQA prefill over 20000 keys (3 block-table windows) + long decodes")
    full_check(b, None, "long-prefill")


def test_one_decode_range_for_the_batch():
    # cus_total = 1: a single balanced range holds every decode page
    ns, ls = [1, 1, 1, 1], [30000, 5000, 17, 80]
    pages = sum(-(-L // QW.page_size) for L in ls)      # 1875 + 313 + 2 + 5 = 2195
    b = custom_batch(QW, ns, ls, seed=32)
    log(f"GQA decode, one range of {pages} pages")
    pa = full_check(b, F.make_opts(cus_total=1), "one-range")
    assert pa.plan.info["n_decode_ranges"] == 1 and pa.plan.info["pages_per_split"] == pages


@pytest.mark.parametrize("hq, keys, windows", [(64, 40000, 2), (128, 40000, 1), (128, 131100, 2)])
def test_latent_decode_across_page_windows(hq, keys, windows):
    # page 64: 625 pages are two windows of a 64-head piece and one of a 128-head piece, 2049 pages two of the latter
    ns, ls = [1, 1], [keys, 300]
    b = custom_batch(MLA, ns, ls, seed=33, num_q_heads=hq)
    entries = 2048 if hq == 128 else 512
    assert -(-(-(-keys // 64)) // entries) == windows
    if windows > 1:
        favour_keys(b, 0, entries * 64, 10.0)
    log(f"latent decode over {keys} keys, {hq} heads ({windows} block-table windows), one range")
    pa = full_check(b, F.make_opts(cus_total=1, wg_per_cu=1), "latent-long")
    assert pa.plan.info["n_decode_ranges"] == 1 and pa.plan.info["n_split_seqs"] == 0


@pytest.mark.parametrize("bm, window", [(128, 2048 * 16), (64, 512 * 16)])
def test_latent_prefill_across_page_windows(bm, window):
    """A ragged tile whose waves end before, inside and after the first keys of
    the second window: some waves have no key there, some a part of a tile."""
    n, L = 70, window + 20
    b = custom_batch(MLA, [n], [L], seed=34, page_size=16, num_q_heads=64)
    favour_keys(b, 0, window, 10.0)
    log(f"latent prefill of {n} tokens over {L} keys at page 16 in {bm}-row tiles (2 block-table windows)")
    out, lse, pa = run(b, opts=F.make_opts(bm=bm))
    assert pa.plan.info["bm"] == bm
    w = b.workload
    picks = [(0, i) for i in (0, 15, 16, 31, 32, 48, 49, 50, 51, 63, 64, 69)]   # token 50 is the first to see the second window
    ref_o, ref_l = OA.attention_rows(b.q, b.k_cache, None, b.block_table, b.seq_lens, b.query_start_loc, w.sm_scale,
                                     picks, num_kv_heads=1, page_size=16, head_dim_v=512, v_aliases_k=True)
    idx = [i for _, i in picks]
    check_close(out[idx], ref_o, "out")
    check_close(lse[idx], ref_l, "lse")
