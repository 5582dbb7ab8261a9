"""Latent attention over 128 query rows (four waves of 32) at the edges of its
tiles, waves, block-table windows and rescaling, against the fp64 oracle."""
import pytest

from paper_2606_04415_amd import flexattn as F
from paper_2606_04415_amd.workloads import WORKLOADS

from gpu_common import custom_batch, log
from test_gpu_long import full_check

pytestmark = pytest.mark.gpu

MLA = WORKLOADS["mla"]

CASES = {
    # key counts around the 32-key tile, the 8 rows a wave loads and a page; one tile to many
    "decode-edges": ([1] * 12, [1, 7, 8, 9, 31, 32, 33, 63, 65, 96, 97, 129], 16),
    # rows around a wave's 32 and a tile's 128, with and without cached keys
    "prefill-edges": ([1, 31, 32, 33, 127, 128, 129, 2], [1, 31, 37, 33, 130, 128, 200, 95], 128),
    # 2, 3, 5 and 9 pieces of one sequence: every step of the merge
    "merge-steps": ([1, 1, 1, 1], [128, 192, 320, 1100], 64),
}


@pytest.mark.parametrize("hq", [64, 128])
@pytest.mark.parametrize("page", [16, 64])
@pytest.mark.parametrize("name", CASES)
def test_edges(name, page, hq):
    ns, ls, split = CASES[name]
    log(f"latent {name}, page {page}, {hq} heads")
    b = custom_batch(MLA, ns, ls, seed=41, page_size=page, num_q_heads=hq)
    full_check(b, F.make_opts(min_split_tokens=split), f"latent-{name}-p{page}-h{hq}")


def test_decode_across_page_windows():
    # 33000 keys at page 16: 2063 pages, two windows of 2048
    b = custom_batch(MLA, [1], [33000], seed=42, page_size=16)
    log("latent decode over 33000 keys at page 16 (2 block-table windows), one range")
    pa = full_check(b, F.make_opts(cus_total=1, wg_per_cu=1), "latent-windows")
    assert pa.plan.info["n_split_seqs"] == 0


def test_maximum_moves_past_the_rescale_threshold():
    """Keys of each third score 64 * 4 * sm_scale = 18.5 above those of the
    third before, 26.7 in log2 units: more than the 24 by which a maximum may
    be stale, so every row rescales twice. The offset sits in the last 64
    columns, which are no part of the values."""
    ns, ls = [1, 70], [600, 400]
    b = custom_batch(MLA, ns, ls, seed=43)
    b.q[:, :, 512:] = 1.0
    for s, L in enumerate(ls):
        for t in range(L):
            b.k_cache[int(b.block_table[s, t // 64]), t % 64, :, 512:] = 4.0 * (3 * t // L)
    log("latent rows whose maximum rises by 26.7 twice")
    full_check(b, F.make_opts(cus_total=1, wg_per_cu=1), "latent-rescale")
