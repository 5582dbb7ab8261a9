"""Latent attention over 128 query rows (four waves of 32) at the edges of its
tiles, waves, block-table windows and rescaling, against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle.attention as OA
from paper_2606_04415_amd import flexattn as F
from paper_2606_04415_amd.workloads import WORKLOADS

from gpu_common import check_close, custom_batch, log, run
from test_gpu_long import full_check

pytestmark = pytest.mark.gpu

MLA = WORKLOADS["mla"]

CASES = {
    # key counts around the 32-key tile, the 8 rows a wave loads and a page; one tile to many
    "decode-edges": ([1] * 12, [1, 7, 8, 9, 31, 32, 33, 63, 65, 96, 97, 129], 16),
    # rows around a wave's 32 and a tile's 128, with and without cached keys
    "prefill-edges": ([1, 31, 32, 33, 127, 128, 129, 2], [1, 31, 37, 33, 130, 128, 200, 95], 128),
    # around the tiles that take 16 rows a wave: up to 64 rows and 256 keys
    "prefill-spread": ([15, 16, 17, 47, 49, 64, 65, 64, 64], [15, 30, 17, 60, 49, 64, 65, 256, 257], 128),
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
    third before, 26.7 in log2 units: far more than a maximum may be stale, so
    every row rescales twice. The offset sits in the last 64 columns, which are
    no part of the values."""
    ns, ls = [1, 70], [600, 400]
    b = custom_batch(MLA, ns, ls, seed=43)
    b.q[:, :, 512:] = 1.0
    for s, L in enumerate(ls):
        for t in range(L):
            b.k_cache[int(b.block_table[s, t // 64]), t % 64, :, 512:] = 4.0 * (3 * t // L)
    log("latent rows whose maximum rises by 26.7 twice")
    full_check(b, F.make_opts(cus_total=1, wg_per_cu=1), "latent-rescale")


def set_offsets(b, ls, row_factor, offset):
    """Adds row_factor(row) * offset(key, L) log2 units to the scores, through the
    last 64 columns (no part of the values): query columns of row_factor,
    key columns of offset / 64 units."""
    per = 64 * b.workload.sm_scale * math.log2(math.e)
    T, H = b.q.shape[:2]
    b.q[:, :, 512:] = torch.tensor([row_factor(r) for r in range(T * H)]).reshape(T, H, 1).to(b.q.dtype)
    P = b.workload.page_size
    for s, L in enumerate(ls):
        for t in range(L):
            b.k_cache[int(b.block_table[s, t // P]), t % P, :, 512:] = offset(t, L) / per


@pytest.mark.parametrize("hq", [64, 128])
@pytest.mark.parametrize("page", [16, 64])
def test_staircase_of_maxima(page, hq):
    """Scores rise by up to 2 log2 units every 40 keys, by another amount in each
    row: a maximum is stale for several steps, then moves at another tile in
    each row, and the keys before the move keep a visible share (2^-2 a step),
    so a wrong factor, or another row's, is far outside the tolerance."""
    ns, ls = [1, 1, 45], [900, 610, 500]
    b = custom_batch(MLA, ns, ls, seed=45, page_size=page, num_q_heads=hq)
    b.q[:, :, :512] *= 0.25   # leaves the rise in charge: the noise is about half a unit
    set_offsets(b, ls, lambda r: 0.4 + 0.6 * (r * 7 % 32) / 31, lambda t, L: 2.0 * (t // 40))
    log(f"latent rows whose maximum climbs in steps of 2, page {page}, {hq} heads")
    full_check(b, F.make_opts(cus_total=1, wg_per_cu=1), f"latent-staircase-p{page}-h{hq}")


@pytest.mark.parametrize("hq", [64, 128])
def test_large_values_stay_finite(hq):
    """Values near 2^112 with scores that rise by 16 log2 units: sums of values
    times probabilities of up to 2^8 stay below 2^128, the largest float (a
    maximum that may be more than 14 units stale overflows)."""
    ns, ls = [1, 40], [700, 300]
    b = custom_batch(MLA, ns, ls, seed=46, num_q_heads=hq)
    scale = 2.0 ** 112
    b.q[:, :, :512] = 0.0
    b.k_cache[..., :512] *= scale
    set_offsets(b, ls, lambda r: 1.0, lambda t, L: 16.0 * t / L)
    log(f"latent values near 2^112, {hq} heads")
    out, lse, _ = run(b, opts=F.make_opts(cus_total=1, wg_per_cu=1))
    b.k_cache[..., :512] /= scale
    ref_o, ref_l = OA.paged_attention(b.q, b.k_cache, None, b.block_table, b.seq_lens, b.query_start_loc,
                                      b.workload.sm_scale, num_kv_heads=1, page_size=64, head_dim_v=512, v_aliases_k=True)
    check_close(out.double() / scale, ref_o, "out")
    check_close(lse, ref_l, "lse")


def rounded_sums(z, stale, tile=32):
    """Log-sum-exp (log2 units) of the rows of z as fp32 sums of bf16
    probabilities, tile by tile, against a maximum that moves when a tile
    raises it by more than `stale`."""
    m = np.full((z.shape[0], 1), -np.inf, np.float32)
    l = np.zeros((z.shape[0], 1), np.float32)
    for k in range(0, z.shape[1], tile):
        c = z[:, k:k + tile]
        top = c.max(1, keepdims=True)
        new = np.where(top > m + stale, top, m)
        l *= np.exp2(m - new)
        m = new
        p = torch.from_numpy(np.exp2(c - m)).to(torch.bfloat16).float().numpy()
        l += p.sum(1, keepdims=True, dtype=np.float32)
    return (m + np.log2(l))[:, 0]


@pytest.mark.parametrize("hq", [64, 128])
@pytest.mark.parametrize("what", ["prefill", "decode"])
def test_log_sum_exp_precision(what, hq):
    """The probabilities are rounded to bf16 before they are summed; the
    largest of a row is exact only while the maximum is fresh. The error
    against 64 bits is held to that of the same sums in numpy with a maximum
    at most 8 units stale (5% for the sampled rows; 24 units give 1.3 times)."""
    n, seqs, L = (64, 1, 2304) if what == "prefill" else (1, 24, 2304)
    b = custom_batch(MLA, [n] * seqs, [L] * seqs, seed=47, num_q_heads=hq)
    b.q *= 2   # scores spread over 5 log2 units
    _, lse, _ = run(b, opts=F.make_opts(cus_total=1, wg_per_cu=1))   # one range
    unit = b.workload.sm_scale * math.log2(math.e)
    err = {"kernel": [], 8.0: [], 24.0: []}
    for s in range(seqs):
        k = b.k_cache[b.block_table[s, :L // 64].long()].reshape(L, 576).double().numpy()
        z = b.q[s * n:(s + 1) * n].double().numpy().reshape(n * hq, 576) @ k.T * unit
        hidden = np.arange(L)[None, :] > (L - n + np.arange(n * hq) // hq)[:, None]
        z[hidden] = -np.inf
        top = z.max(1, keepdims=True)
        ref = (top + np.log2(np.exp2(z - top).sum(1, keepdims=True)))[:, 0]
        err["kernel"].append(lse[s * n:(s + 1) * n].double().numpy().reshape(-1) / math.log(2) - ref)
        for stale in (8.0, 24.0):
            err[stale].append(rounded_sums(z.astype(np.float32), stale).astype(np.float64) - ref)
    rms = {key: float(np.sqrt(np.mean(np.square(np.concatenate(v))))) for key, v in err.items()}
    log(f"  lse error (log2 units) {what}, {hq} heads: " + ", ".join(f"{key} {v:.3e}" for key, v in rms.items()))
    assert rms["kernel"] <= 1.05 * rms[8.0]
