"""Parity at the edges of kernel variants and dispatch rules: sizes on either side of a tile, of a remainder and of
the line between two kernels, against the oracle with the tolerances of test_gpu_parity."""
import math

import numpy as np
import pytest
import torch

from paper_2603_08055_amd import workloads
from tests.parity_util import (compare_windows_with_oracle, compare_with_oracle, log, run_device, special_row_splits,
                               to_host_f32)
from tests.test_gpu_parity import TOL, assert_close, compress_topk_case, draw, layer_case, s3r  # noqa: F401  (s3r: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,block,views,tpv,special,heads", [
    ("bf16", 16, 1, 530, 6, 2),       # 33 blocks = 8 units and a quarter: the last split ends in a short unit and the special one
    ("bf16", 16, 2, 250, 3, 1),       # 8 + 1 units, two splits; the second ends in the special-token segment
    ("bf16", 32, 3, 434, 2, 3),       # blocks of 32, an odd number of them (41): half a unit in the last split
    ("bf16", 16, 5, 611, 61, 2),      # 305 special rows: three row groups, five special units
    ("bf16", 64, 2, 700, 1, 1),       # one row group of two rows over many splits
    ("f32", 32, 2, 411, 2, 2),        # fp32 operand parts
])
def test_special_rows_in_key_splits(s3r, oracle, dtype, block, views, tpv, special, heads):  # noqa: F811
    wl = workloads.Workload(f"splits_{dtype}_{block}_{views}x{tpv}_{special}", views, tpv, heads, 64, dtype, block, 3,
                            93, "normal")
    assert special_row_splits(s3r, views, tpv, special, heads, block, dtype) > 1
    layer_case(s3r, oracle, wl, special, with_gate=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("views,special,grid", [
    (4, 3, (13, 11, 4)),              # 48 windows of 16, 12, 4 and 3 cells: the lengths of units past the first split
    (6, 1, (9, 11, 4)),               # 54 windows: half a unit at the end
    (2, 5, (37, 37, 4)),              # 200 windows over many splits
    (4, 3, (13, 11, 8)),              # 8 x 8 windows
])
def test_special_rows_in_key_splits_over_windows(s3r, oracle, dtype, views, special, grid):  # noqa: F811
    grid_h, grid_w, window = grid
    tpv, heads = special + grid_h * grid_w, 2
    wl = workloads.Workload(f"splits_windows_{dtype}_{views}x{grid_h}x{grid_w}_w{window}", views, tpv, heads, 64, dtype,
                            window * window, 3, 101, "normal")
    assert special_row_splits(s3r, views, tpv, special, heads, wl.block, dtype, grid) > 1
    q, k, v = workloads.make_inputs(wl)
    gate = workloads.make_gate_logits(wl)
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), wl.block, 3, gate=gate.cuda(), tokens_per_view=tpv,
                     special_per_view=special, grid=grid)
    log(f"{wl.name}: " + str(compare_windows_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v),
                                                         to_host_f32(gate), 3, dtype, views, tpv, special, grid,
                                                         label=wl.name)))


@pytest.mark.parametrize("dtype,block", [("bf16", 16), ("bf16", 64), ("f32", 32), ("f32", 64)])
def test_a_key_that_is_not_a_number_in_one_key_split(s3r, dtype, block):  # noqa: F811
    """The softmax of every special row runs over that key, whichever split holds it: NaN in the whole row.  The key
    is a special token's, so that the image rows and the other head never see it."""
    views, tpv, special, heads = 2, 400, 3, 2
    wl = workloads.Workload(f"nan_key_{dtype}_{block}", views, tpv, heads, 64, dtype, block, 3, 99, "normal")
    q, k, v = workloads.make_inputs(wl)
    k[tpv + 1, 1, 5] = float("nan")
    out = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), block, 3, tokens_per_view=tpv, special_per_view=special)["out"]
    is_nan = out.view(views, tpv, heads, 64).isnan()
    assert is_nan[:, :special, 1].all()
    assert not is_nan[:, :special, 0].any() and not is_nan[:, special:].any()


@pytest.mark.parametrize("dtype,block,n_tok,topk,heads", [
    ("bf16", 16, 16, 1, 1),           # one block, one entry
    ("bf16", 16, 16 * 5 - 1, 5, 3),   # a list one block longer than the four worked on at a time, short last block
    ("bf16", 16, 16 * 70 + 3, 64, 2), # a full load of the index row
    ("bf16", 16, 16 * 70 + 3, 66, 1), # ... and two entries more
    ("bf16", 32, 33, 2, 2),           # two blocks, the second of one token
    ("bf16", 32, 32 * 9 + 5, 3, 5),   # odd list, ten query blocks: the last workgroup half empty
    ("bf16", 32, 32 * 140, 131, 1),   # three loads of the index row
    ("f32", 16, 16 * 6 + 1, 5, 2),
    ("f32", 16, 16 * 90 + 9, 67, 1),
    ("f32", 32, 32 * 7 - 3, 3, 2),
    ("f32", 32, 31, 1, 1),
])
def test_selection_of_small_blocks(s3r, oracle, dtype, block, n_tok, topk, heads):
    wl = workloads.Workload(f"small_{dtype}_{block}_{n_tok}_{topk}", 1, n_tok, heads, 64, dtype, block, topk, 94, "normal")
    q, k, v = workloads.make_inputs(wl)
    gate = workloads.make_gate_logits(wl)
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), block, topk, gate=gate.cuda())
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v),
                                                 to_host_f32(gate), block, topk, dtype, label=wl.name)))


@pytest.mark.parametrize("tail", [1, 4, 5, 16, 17, 31, 32, 33, 44, 48, 49, 63, 64])
def test_dense_attention_with_a_short_last_unit(s3r, oracle, tail):
    """The keys of a unit that exist, counted in runs of 16 and of 4 of them per lane."""
    n_tok, heads = 128 + tail, 2
    q, k, v = (draw(n_tok, heads, "bf16", 3100 + i) for i in range(3))
    out = torch.full_like(q, float("nan")).cuda()
    s3r.speed3r_dense_attn(q.cuda(), k.cuda(), v.cuda(), out)
    ref = oracle.dense_attn(*(to_host_f32(x) for x in (q, k, v)), 0.125)
    assert_close(to_host_f32(out), ref, TOL["bf16"], f"dense tail={tail}")


@pytest.mark.parametrize("n_blk,heads,k", [
    (1, 1, 1), (2, 3, 2), (15, 2, 15), (16, 2, 4), (17, 2, 16), (63, 1, 64), (65, 2, 1), (128, 2, 7), (129, 1, 64),
    (256, 3, 9), (257, 2, 64), (511, 1, 64), (512, 2, 33), (513, 1, 5), (768, 2, 64), (769, 1, 7), (1023, 1, 64), (1024, 2, 1),
    (724, 16, 8), (725, 16, 8),       # either side of the line to the sweeps
])
def test_short_sequences_in_one_launch(s3r, oracle, n_blk, heads, k):  # noqa: F811
    """Integer scores with many ties: the TopK sets are the oracle's, bit for bit."""
    rng = np.random.default_rng(1000 * n_blk + k)
    qc, kc = (rng.integers(-2, 3, (heads, n_blk, 64)).astype(np.float32) for _ in range(2))
    vc = rng.standard_normal((heads, n_blk, 64)).astype(np.float32)
    scores = oracle.scores(qc.astype(np.float64), kc.astype(np.float64))
    for accurate in (False, True):
        o_comp, idx = compress_topk_case(s3r, qc, kc, vc, k, accurate)
        assert np.array_equal(idx, oracle.topk(scores, min(k, n_blk)))
        ref = oracle.compressed_attn(scores, vc.astype(np.float64), 0.125)
        in_one = n_blk <= 1024 and n_blk * n_blk * heads <= 2 ** 23
        assert_close(o_comp, ref, TOL["f32"] if accurate or in_one else TOL["bf16"], "o_comp")


@pytest.mark.parametrize("n_blk,k", [(130, 64), (500, 17)])   # (up to 512 blocks the sweeps' candidate lists hold every key)
def test_near_ties_are_decided_as_by_the_sweeps(s3r, n_blk, k):  # noqa: F811
    """Keys that differ by less than the rounding of a score: one launch for short sequences and (more heads: past the
    line) the sweeps with their candidates give the same lists, entry by entry."""
    rng = np.random.default_rng(n_blk + k)
    line = 2 ** 23 // n_blk ** 2
    base = rng.standard_normal((1, 1, 64))
    one = [np.asarray(base + 2e-7 * rng.standard_normal((2, n_blk, 64)), dtype=np.float32),
           np.asarray(base + 2e-7 * rng.standard_normal((2, n_blk, 64)), dtype=np.float32),
           rng.standard_normal((2, n_blk, 64)).astype(np.float32)]
    many = [np.concatenate([x, np.zeros((line - 1, n_blk, 64), dtype=np.float32)]) for x in one]
    _, idx = compress_topk_case(s3r, *one, k, False)
    _, want = compress_topk_case(s3r, *many, k, False)
    assert (np.diff(idx, axis=2) > 0).all()
    assert np.array_equal(idx, want[:2])


@pytest.mark.parametrize("n_blk,k", [(40, 40), (130, 64), (500, 17)])
def test_scores_that_are_no_numbers_enter_no_list(s3r, n_blk, k):  # noqa: F811
    """A NaN key (or query) in one launch for short sequences and, past the line, in the sweeps: the same lists, and
    zeros where fewer than k blocks are left."""
    rng = np.random.default_rng(n_blk + k)
    line = 2 ** 23 // n_blk ** 2
    one = [rng.standard_normal((2, n_blk, 64)).astype(np.float32) for _ in range(3)]
    one[1][0, 7, 3] = np.nan
    one[0][1, 5, 9] = np.nan
    many = [np.concatenate([x, np.zeros((line - 1, n_blk, 64), dtype=np.float32)]) for x in one]
    _, idx = compress_topk_case(s3r, *one, k, False)
    _, want = compress_topk_case(s3r, *many, k, False)
    assert np.array_equal(idx, want[:2])
    assert not (idx[0] == 7).any() and not idx[1, 5].any()


@pytest.mark.parametrize("n_blk,topk,n_forced", [(70, 64, 3), (200, 65, 1), (320, 64, 64), (90, 5, 90)])   # (65: scores through memory)
def test_forced_blocks_and_long_rows_in_one_launch(s3r, oracle, n_blk, topk, n_forced):  # noqa: F811
    wl = workloads.Workload(f"short_forced_{n_blk}_{topk}_{n_forced}", 1, 16 * n_blk - 3, 2, 64, "bf16", 16, topk, 103, "normal")
    q, k, v = workloads.make_inputs(wl)
    forced = list(range(0, n_blk, n_blk // n_forced))[:n_forced]
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 16, topk, forced=forced)
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 16,
                                                 topk, "bf16", forced=forced, label=wl.name)))


@pytest.mark.parametrize("n_tok,heads,topk,n_forced", [
    (64 * 3 + 1, 128, 3, 0), (64 * 3 + 1, 128, 4, 0),     # 512 query blocks, on either side of the shortest row of two pairs
    (64 * 27, 19, 7, 0), (64 * 27, 18, 7, 0), (64 * 27 - 60, 18, 8, 2),   # 513 and 486 of them, odd rows; forced blocks
    (64 * 40 - 1, 3, 5, 0), (64 * 9, 1, 9, 0),            # shorter odd rows: the second pair is done first
    (64 * 130, 2, 127, 0), (64 * 130, 2, 126, 2),         # 260: the longest rows
])
def test_two_pairs_of_waves_for_few_query_blocks(s3r, oracle, n_tok, heads, topk, n_forced):  # noqa: F811
    wl = workloads.Workload(f"few_{n_tok}_{heads}_{topk}", 1, n_tok, heads, 64, "bf16", 64, topk, 105, "normal")
    q, k, v = workloads.make_inputs(wl)
    forced = list(range(n_forced)) if n_forced else None
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 64, topk, forced=forced)
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 64,
                                                 topk, "bf16", forced=forced, label=wl.name)))


@pytest.mark.parametrize("dtype,block,n_tok,heads,topk", [
    ("bf16", 64, 700, 7, 3), ("bf16", 64, 64 * 512, 3, 5),     # a head's K and V of 8 MiB: the last size by whole heads
    ("bf16", 64, 64 * 513, 3, 5), ("bf16", 16, 16 * 33, 5, 4), ("bf16", 128, 128 * 9 - 1, 3, 4), ("f32", 64, 64 * 11, 9, 3),
    ("f32", 32, 32 * 19, 1, 3),
])
def test_every_head_and_query_block_is_mapped_to_an_xcd(s3r, oracle, dtype, block, n_tok, heads, topk):  # noqa: F811
    wl = workloads.Workload(f"map_{dtype}_{block}_{n_tok}_{heads}", 1, n_tok, heads, 64, dtype, block, topk, 106, "normal")
    q, k, v = workloads.make_inputs(wl)
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), block, topk)
    assert torch.isfinite(res["out"].float()).all()
    n_blk = (n_tok + block - 1) // block
    rows = sorted({0, n_blk // 3, n_blk - 1})
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, block,
                                                 topk, dtype, rows=rows, label=wl.name)))


@pytest.mark.parametrize("layout", ["one projection", "head major", "padded heads"])
# two pairs of waves per query block (few query blocks), one pair, two (long rows on long sequences)
@pytest.mark.parametrize("views,tpv,topk", [(3, 1000, 39), (20, 1281, 39), (150, 1281, 40)])
def test_strided_queries_in_the_pipelined_selection(s3r, views, tpv, topk, layout):  # noqa: F811
    heads = 3
    wl = workloads.Workload(f"pipe_strided_{views}", views, tpv, heads, 64, "bf16", 64, topk, 95, "normal")
    tensors = workloads.make_inputs(wl, device="cuda")
    if layout == "one projection":
        big = torch.stack(tensors, dim=1)
        strided = [big[:, i] for i in range(3)]
    elif layout == "head major":
        strided = [t.permute(1, 0, 2).contiguous().permute(1, 0, 2) for t in tensors]
    else:
        strided = [torch.full((wl.n_tok, heads, 80), float("nan"), dtype=t.dtype, device="cuda")[:, :, :64].copy_(t)
                   for t in tensors]
    assert not strided[0].is_contiguous()
    want = run_device(s3r, *tensors, 64, topk)
    got = run_device(s3r, *strided, 64, topk)
    for key in ("idx", "o_comp", "out", "o_sel", "lse"):   # the same arithmetic on the same values
        assert torch.equal(got[key], want[key]), key


@pytest.mark.parametrize("topk,n_forced", [(40, 0), (64, 1), (64, 23), (30, 40)])
def test_long_rows_keep_the_precision_of_two_pairs(s3r, topk, n_forced):  # noqa: F811
    """Outlier keys: a few weights make up a row, and what is left against 64 bits is the rounding of P to bf16.  In two
    pairs of waves the largest weight of each is exact: 6.4e-4 to 6.8e-4 in lse, 7.3e-4 to 7.6e-4 in one pair."""
    wl = workloads.Workload("long_rows", 150, 1374, 1, 64, "bf16", 64, topk, 107, "outliers")
    q, k, v = workloads.make_inputs(wl, device="cuda")
    res = run_device(s3r, q, k, v, 64, topk, forced=list(range(n_forced)) if n_forced else None)
    q64, k64 = q[:, 0].double(), k[:, 0].double()
    off = count = 0.0
    for b in range(0, wl.n_tok // 64, 8):
        keys = (res["idx"][0, b].long()[:, None] * 64 + torch.arange(64, device="cuda")).reshape(-1)
        keys = keys[keys < wl.n_tok]
        want = torch.logsumexp(q64[64 * b:64 * (b + 1)] @ k64[keys].T / 8.0, dim=-1)
        off += (res["lse"][0, 64 * b:64 * (b + 1)].double() - want).square().sum().item()
        count += 64
    assert math.sqrt(off / count) < 7.0e-4


@pytest.mark.parametrize("block", [16, 32])
def test_scores_of_small_fp32_blocks_are_added_up_exactly_enough(s3r, block):  # noqa: F811
    """Peaked softmaxes over outlier keys (scores of some hundred): the rounding of the scores shows.  Two bf16 parts of
    P and V leave 2.7e-6; scores that round each of their partial products at full size bring it to 3.4e-6 and more."""
    wl = workloads.Workload(f"sums_{block}", 12, 1374, 4, 64, "f32", block, 40, 100, "outliers")
    q, k, v = workloads.make_inputs(wl, device="cuda")
    q.mul_(16.0)
    res = run_device(s3r, q, k, v, block, 40)
    off = total = 0.0
    for h in range(wl.heads):
        qh, kh, vh = (x[:, h].double() for x in (q, k, v))
        for b in range(0, wl.n_tok // block, 16):
            keys = (res["idx"][h, b].long()[:, None] * block + torch.arange(block, device="cuda")).reshape(-1)
            keys = keys[keys < wl.n_tok]
            want = torch.softmax(qh[block * b:block * (b + 1)] @ kh[keys].T / 8.0, dim=-1) @ vh[keys]
            off += (res["o_sel"][block * b:block * (b + 1), h].double() - want).square().sum().item()
            total += want.square().sum().item()
    assert math.sqrt(off / total) < 3.0e-6


@pytest.mark.parametrize("dtype,block,views,tpv,special,heads,grid,fewer", [
    ("f32", 64, 40, 400, 32, 2, None, 12), ("f32", 16, 100, 400, 32, 1, None, 10), ("f32", 16, 30, 32 + 37 * 37, 32, 3, (37, 37, 4), 10),
    ("bf16", 16, 20, 5 + 37 * 37, 5, 16, (37, 37, 4), 16), ("bf16", 16, 2, 1374, 5, 1, None, 9), ("bf16", 64, 20, 1374, 5, 1, None, 24),
])
def test_special_rows_run_in_the_workspace_of_fewer_splits(s3r, dtype, block, views, tpv, special, heads, grid, fewer):  # noqa: F811
    """Special rows take more key splits than the time alone would ask for; a workspace for the leaner number will do."""
    splits = special_row_splits(s3r, views, tpv, special, heads, block, dtype, grid)
    assert splits > fewer
    n_tok = views * tpv
    q, k, v = (draw(n_tok, heads, dtype, 3200 + i).cuda() for i in range(3))
    layout = dict(tokens_per_view=tpv, special_per_view=special, grid=grid)
    need = s3r.speed3r_workspace_bytes_ex(n_tok, heads, 64, block, 4, s3r.S3R_F32 if dtype == "f32" else s3r.S3R_BF16, **layout)
    up = lambda x: (x + 255) // 256 * 256   # noqa: E731
    parts = lambda splits: up(splits * views * special * heads * 64 * 4) + up(splits * views * special * heads * 4)   # noqa: E731
    out = {}
    for n_bytes in (need, need - parts(splits) + parts(fewer)):
        out[n_bytes] = torch.full_like(q, float("nan"))
        s3r.speed3r_sparse_global_attn_ex(q, k, v, out[n_bytes], block, 4, workspace=torch.empty(n_bytes, dtype=torch.uint8, device="cuda"), **layout)
    a, b = out.values()
    rows = torch.arange(n_tok, device="cuda") % tpv < special
    assert torch.equal(a[~rows], b[~rows])
    assert_close(to_host_f32(a[rows]), to_host_f32(b[rows]), TOL[dtype], "special rows in more and in fewer splits")
    with pytest.raises(s3r.Speed3rError):
        s3r.speed3r_sparse_global_attn_ex(q, k, v, torch.empty_like(q), block, 4,
                                          workspace=torch.empty(n_bytes - 256, dtype=torch.uint8, device="cuda"), **layout)


def test_row_sums_of_long_fp32_rows_are_added_up_exactly_enough(s3r):  # noqa: F811
    """Rows over 274 800 outlier keys, whose sum one weight may dominate: added up unit by unit the sum leaves 3.5e-6 with
    the two bf16 parts of P and V, one key after the other onto the whole sum 6.3e-6."""
    views, tpv, special, heads = 200, 1374, 5, 2
    wl = workloads.Workload("long_row_sums", views, tpv, heads, 64, "f32", 64, 4, 104, "outliers")
    q, k, v = workloads.make_inputs(wl, device="cuda")
    out = run_device(s3r, q, k, v, 64, 4, want=(), tokens_per_view=tpv, special_per_view=special)["out"]
    off = total = 0.0
    for h in range(heads):
        k64, v64 = k[:, h].double(), v[:, h].double()
        for view in range(0, views, 5):
            rows = view * tpv + torch.arange(special, device="cuda")
            want = torch.softmax(q[rows, h].double() @ k64.T / 8.0, dim=-1) @ v64
            off += (out[rows, h].double() - want).square().sum().item()
            total += want.square().sum().item()
    assert math.sqrt(off / total) < 4.5e-6


def _one_large_weight(n_keys, twice=0):
    """Keys whose weights are 1 for the first and 2^-26 for the others (2^-25 for every twice-th), for queries of 8 in two
    channels: two small weights are below half of the last place of 1 (2^-24), the 32 of a lane and unit are four of
    them."""
    s = torch.full((n_keys,), -26.0 * math.log(2.0), dtype=torch.float64)
    if twice:
        s[::twice] = -25.0 * math.log(2.0)
    s[0] = 0.0
    hi = s.to(torch.bfloat16)
    k = torch.zeros((n_keys, 64), dtype=torch.bfloat16)
    k[:, 0], k[:, 1] = hi, (s - hi.to(torch.float64)).to(torch.bfloat16)
    return k


@pytest.mark.parametrize("block,kk,heads", [(64, 128, 5), (64, 128, 1), (64, 200, 2), (128, 64, 2)])   # one and two pairs of waves; long rows; blocks of 128
def test_small_weights_beside_a_large_one_stay_in_the_row_sum(s3r, block, kk, heads):  # noqa: F811
    """Added up within a unit first they all count; one after the other onto the whole sum an eighth of them is lost
    (7e-6 to 2.4e-5 in lse)."""
    n_tok = block * kk
    k = _one_large_weight(n_tok)[:, None].expand(n_tok, heads, 64).contiguous().cuda()
    q = torch.zeros_like(k)
    q[:, :, :2] = 8.0
    idx = torch.arange(kk, dtype=torch.int32, device="cuda").expand(heads, kk, kk).contiguous()
    lse = torch.full((heads, n_tok), float("nan"), device="cuda")
    s3r.speed3r_select_attn(q, k, torch.ones_like(k), idx, torch.empty_like(q), block, lse=lse)
    assert (lse.double() - math.log1p((n_tok - 1) * 2.0 ** -26)).abs().max().item() < 2e-6


def test_small_weights_beside_a_large_one_stay_in_the_sum_of_the_sweep(s3r):  # noqa: F811
    n_blk = 4096
    kc = _one_large_weight(n_blk, 63).float().numpy()[None]   # (bounds on the TopK that hold few keys: no second pass)
    qc = np.zeros_like(kc)
    qc[:, :, :2] = 8.0
    vc = np.ones_like(kc)
    vc[:, 0] = 0.0
    o_comp, _ = compress_topk_case(s3r, qc, kc, vc, 4, False)
    small = (n_blk - 1 + (n_blk - 1) // 63) * 2.0 ** -26
    want = small / (1.0 + small)
    assert np.abs(o_comp / want - 1.0).max() < 2e-6


@pytest.mark.parametrize("block,n_tok", [(0, 64 * 3 + 7), (0, 64 * 67), (64, 64 * 5 + 1), (64, 64 * 5 + 33), (64, 64), (128, 128 * 3 + 70), (128, 128 * 2 + 64)])
@pytest.mark.parametrize("spread", ["none", "keys", "channels", "blocks", "tiny queries", "zero blocks"])
def test_fp32_keys_of_all_sizes(s3r, oracle, block, n_tok, spread):  # noqa: F811
    """Entries of different sizes in a row, a block and from block to block, the other operand as much smaller where a channel
    is large.  Few keys in the last unit: one key half without work."""
    heads = 2
    wl = workloads.Workload(f"f32_{spread}_{block}_{n_tok}", 1, n_tok, heads, 64, "f32", max(block, 64), 1, 111, "normal")
    q, k, v = workloads.make_inputs(wl)
    gen = torch.Generator().manual_seed(112)
    if spread == "keys":        # logits stay ordinary: large keys have small entries where queries are not 0
        k *= torch.exp2(torch.randint(-12, 1, (n_tok, heads, 1), generator=gen).float())
    elif spread == "channels":
        size = torch.exp2(torch.randint(-9, 10, (1, heads, 64), generator=gen).float())
        q, k = q / size, k * size
    elif spread == "blocks":    # every block of keys of its own size, down to 2^-60
        k *= torch.exp2(-20.0 * ((torch.arange(n_tok) // max(block, 64)) % 4).float())[:, None, None]
    elif spread == "tiny queries":
        q, k = q * 1e-18, k * 1e18
    elif spread == "zero blocks":
        k[:40] = 0.0
        k[-3:] = 0.0
        q[1::3] = 0.0
    out = torch.full_like(q, float("nan")).cuda()
    if block == 0:
        s3r.speed3r_dense_attn(q.cuda(), k.cuda(), v.cuda(), out)
    else:
        n_blk = -(-n_tok // block)
        idx = torch.arange(n_blk, dtype=torch.int32, device="cuda").expand(heads, n_blk, n_blk).contiguous()
        s3r.speed3r_select_attn(q.cuda(), k.cuda(), v.cuda(), idx, out, block)
    ref = oracle.dense_attn(*(to_host_f32(x) for x in (q, k, v)), 0.125)
    assert_close(to_host_f32(out), ref, TOL["f32"], wl.name)


@pytest.mark.parametrize("where", ["dense", "blocks of 64", "few blocks of 64", "blocks of 128", "blocks of 32", "special, 64", "special, 128", "special, 16"])
@pytest.mark.parametrize("what,size", [("mask", 1e4), ("mask", 1e6), ("mask", 1e8), ("mask", 1e30), ("channels", 20), ("channels", 40),
                                       ("one channel", 24), ("one channel", 60), ("one key", 30), ("one key", 60), ("far apart", 80)])
def test_fp32_scores_of_ordinary_keys_beside_large_entries(s3r, oracle, where, what, size):  # noqa: F811
    """What one key or one channel holds takes no bits from the others: keys masked through a channel that is the same in
    all queries, channels scaled against each other (q / s, k s), one large key that no query sees, and the largest entries
    of q and k in channels where the other one is zero.  The scores that count are ordinary throughout."""
    special = 3 if "special" in where else 0
    block = 64 if where == "dense" else int(where.split()[-1])
    views, heads = (1, 2) if where in ("dense", "few blocks of 64", "blocks of 128", "blocks of 32") else (2, 3)
    tpv = 64 * 45 + 9 if where == "blocks of 64" else 64 * 6 + 41      # 270 query blocks; 14 and fewer
    wl = workloads.Workload(f"large_{what}_{size}_{where}", views, tpv, heads, 64, "f32", block, 1, 113, "normal")
    q, k, v = workloads.make_inputs(wl)
    rows, gen = torch.arange(views * tpv), torch.Generator().manual_seed(114)
    if what == "mask":
        q[:, :, 0] = 1.0
        k[rows % 16 == 5, :, 0] = -size
    elif what == "channels":
        s = torch.exp2(torch.randint(-size, size + 1, (1, heads, 64), generator=gen).float())
        q, k = q / s, k * s
    elif what == "one channel":
        q[:, :, 7] *= 2.0 ** -size
        k[:, :, 7] *= 2.0 ** size
    elif what == "one key":
        q[:, :, 9] = 0.0
        k[70, :, 9] = 2.0 ** size
    else:
        q[:, :, 0], q[:, :, 1] = 2.0 ** size, 0.0
        k[:, :, 0], k[:, :, 1] = 0.0, 2.0 ** size
    dev = [x.cuda() for x in (q, k, v)]
    ref = oracle.dense_attn(*(to_host_f32(x) for x in (q, k, v)), 0.125)
    if special:
        n_blk = -(-views * (tpv - special) // block)
        out = run_device(s3r, *dev, block, min(n_blk, 8), want=(), tokens_per_view=tpv, special_per_view=special)["out"]
        at = (rows % tpv < special).numpy()
        assert_close(to_host_f32(out)[at], ref[at], TOL["f32"], wl.name)
        return
    out = torch.full_like(dev[0], float("nan"))
    if where == "dense":
        s3r.speed3r_dense_attn(*dev, out)
    else:
        n_blk = -(-views * tpv // block)
        idx = torch.arange(n_blk, dtype=torch.int32, device="cuda").expand(heads, n_blk, n_blk).contiguous()
        s3r.speed3r_select_attn(*dev, idx, out, block)
    assert_close(to_host_f32(out), ref, TOL["f32"], wl.name)


# (unit, rise): in the first four units the maximum is looked at, afterwards a unit is done again; then looked at for 64 units
@pytest.mark.parametrize("block", [0, 64, 128])   # dense attention; long rows; blocks of 128
@pytest.mark.parametrize("rises", [[(2, 9)], [(4, 7.9)], [(4, 8.1)], [(5, 60), (6, 69)], [(7, 300)], [(4, 20), (68, 29), (80, 40), (150, 52)],
                                   [(5, 20), (65, 29), (66, 38), (70, 47), (131, 56)]])   # a raise 60 units after another, and soon after that
def test_units_done_again_when_the_maximum_rises(s3r, block, rises):  # noqa: F811
    """Keys of ever larger weight for the even queries only (the odd ones of a wave keep their maximum), in units whose
    probabilities were formed against the maximum before; the last unit is short."""
    n_units = max(rises[-1][0] + 3, 130 if block == 64 else 0) // 2 * 2 + 2
    n_tok = 64 * n_units - 9
    wl = workloads.Workload(f"again_{block}_{rises[0][0]}", 1, n_tok, 2, 64, "bf16", max(block, 64), 1, 110, "normal")
    q, k, v = workloads.make_inputs(wl)
    q[:, :, 0] = 8.0
    q[1::2, :, 0] = 0.0
    k[:, :, 0] = 0.0
    for unit, rise in rises:
        k[64 * unit + 11:64 * (unit + 1):19, :, 0] = rise * math.log(2.0)
    out = torch.full_like(q, float("nan")).cuda()
    if block == 0:
        s3r.speed3r_dense_attn(q.cuda(), k.cuda(), v.cuda(), out)
    else:
        n_blk = -(-n_tok // block)
        idx = torch.arange(n_blk, dtype=torch.int32, device="cuda").expand(2, n_blk, n_blk).contiguous()
        s3r.speed3r_select_attn(q.cuda(), k.cuda(), v.cuda(), idx, out, block)
    p = torch.softmax(torch.matmul(q.double().transpose(0, 1), k.double().permute(1, 2, 0)) / 8.0, dim=-1)
    assert_close(out.float().cpu().numpy(), torch.matmul(p, v.double().transpose(0, 1)).transpose(0, 1).numpy(), TOL["bf16"], wl.name)


# one pair of waves: edge iterations only; full ones.  Two pairs: few query blocks, edge and full; long rows on long sequences
@pytest.mark.parametrize("n_blk,kk", [(8, 3), (513, 8), (9, 8), (40, 24), (3000, 48)])
def test_probabilities_waiting_while_the_maximum_rises(s3r, n_blk, kk):  # noqa: F811
    """Pipelined selection: the running maximum rises by just under 9 (powers of two) while the probabilities of the
    block before still wait for their product with V.  These are 128 and the factor is 1.00385 / 512, the worst for
    a second rounding to bf16 (0.4 %), which the row sum would not share.  The weights of that block (V = 1) and of the
    one that raises the maximum (V = -1) all but cancel, so that it would show as 1.9e-3.  The single roundings
    left are below 1e-4: 128 (1 + 4e-5) to 128, 1 / 1.00385 to 0.99609."""
    n_tok, f64 = 64 * n_blk, torch.float64
    level = torch.full((n_tok,), -40.0, dtype=f64)     # log2 of a key's weight
    v_of = torch.zeros(n_tok, dtype=f64)
    two_pairs = kk >= 40 and n_blk >= 3000 or kk >= 4 and n_blk <= 512
    order = [0, 2, 4] if two_pairs else [0, 1, 2]      # two pairs take the blocks of a list in turn
    base, mid, top = (order[i] * 64 for i in range(3))
    level[base:base + 64] = 0.0
    level[mid:mid + 64], v_of[mid:mid + 64] = 7.0, 1.0
    level[top:top + 16], v_of[top:top + 16] = 9.0 - math.log2(1.00385), -1.0
    s = level * math.log(2.0)                          # q.k / 8 in two bf16 parts
    hi = s.to(torch.bfloat16)
    k = torch.zeros((n_tok, 1, 64), dtype=torch.bfloat16)
    k[:, 0, 0], k[:, 0, 1] = hi, (s - hi.to(f64)).to(torch.bfloat16)
    q = torch.zeros_like(k)
    q[:, 0, :2] = 8.0
    v = v_of.to(torch.bfloat16)[:, None, None].expand(n_tok, 1, 64).contiguous()
    idx = torch.arange(kk, dtype=torch.int32).expand(1, n_blk, kk).contiguous()
    out = torch.full_like(q, float("nan")).cuda()
    s3r.speed3r_select_attn(q.cuda(), k.cuda(), v.cuda(), idx.cuda(), out, 64)
    w = torch.exp(k[:64 * kk, 0, :2].to(f64).sum(-1))
    want = ((w * v_of[:64 * kk]).sum() / w.sum()).item()
    assert (out.double().cpu() - want).abs().max().item() < 2e-4


# two heads: one launch; 33: the sweeps, whose candidate lists cannot run over up to 512 blocks
@pytest.mark.parametrize("n_blk,heads", [(127, 2), (511, 2), (512, 2), (513, 2), (545, 2), (511, 33), (512, 33), (513, 33), (545, 33)])
def test_lists_filled_to_the_last_slot(s3r, oracle, n_blk, heads):
    """Equal keys: every block is a candidate of every row, and the smallest indices win."""
    n_tok, topk = 16 * n_blk, 64
    rows = None if heads == 2 else [0, n_blk // 2, n_blk - 1]
    wl = workloads.Workload(f"equal_keys_{n_blk}", 1, n_tok, heads, 64, "bf16", 16, topk, 96, "normal")
    q, k, v = workloads.make_inputs(wl)
    k[:] = k[:1].clone()
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 16, topk)
    assert torch.equal(res["idx"].cpu(), torch.arange(topk, dtype=torch.int32).expand(heads, n_blk, topk))
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 16,
                                                 topk, "bf16", rows=rows, label=wl.name)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_blk,n_forced", [(1030, 0), (1030, 40), (300, 40)])   # the sweeps, without and with forced blocks; one launch
def test_running_maximum_of_the_compression_rises_beside_forced_blocks(s3r, oracle, dtype, n_blk, n_forced):  # noqa: F811
    """Logits that rise by 64 over the pooled keys: the maximum is raised in most steps, while forced blocks leave the TopK
    and stay in the compression branch."""
    wl = workloads.Workload(f"rise_{dtype}_{n_blk}_{n_forced}", 1, 16 * n_blk, 2, 64, dtype, 16, 16, 108, "normal")
    q, k, v = workloads.make_inputs(wl)
    q.mul_(0.05)
    k.mul_(0.05)
    q[:, :, 0] = 8.0
    k[:, :, 0] = (torch.arange(n_blk, dtype=torch.float32) * (64.0 / n_blk)).round(decimals=0).repeat_interleave(16)[:, None]
    forced = np.sort(np.random.default_rng(109).choice(n_blk, n_forced, replace=False)).astype(np.int32) if n_forced else None
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 16, 16, forced=forced)
    rows = sorted({0, 1, n_blk // 2, n_blk - 1})
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 16, 16,
                                                 dtype, rows=rows, forced=forced, label=wl.name)))


@pytest.mark.parametrize("dtype,which", [("bf16", "q"), ("bf16", "k"), ("f32", "k")])
@pytest.mark.parametrize("n_blk,peak", [(1, 0), (33, 32), (2048, 2047), (2049, 2048), (2500, 2111), (4130, 4129)])
def test_head_maxima_wherever_they_sit(s3r, oracle, dtype, which, n_blk, peak):
    """Pooled entries that overflow fp16 unless the head's scale factor has seen them, on either side of the 2048 rows
    that the statistics kernel covers in one step.  The other operand is as much smaller: logits stay ordinary."""
    wl = workloads.Workload(f"peak_{which}_{dtype}_{n_blk}_{peak}", 1, 16 * n_blk - 5, 2, 64, dtype, 16, 5, 97, "normal")
    q, k, v = workloads.make_inputs(wl)
    large, small = (q, k) if which == "q" else (k, q)
    large[16 * peak:16 * peak + 16, 1] *= 2.0 ** 20
    small[:, 1] *= 2.0 ** -20
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 16, 5)
    rows = sorted({0, n_blk // 2, max(0, peak - 1), peak, n_blk - 1})
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 16,
                                                 5, dtype, rows=rows, label=wl.name)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_blk,topk,lean", [(100, 64, -1.0), (700, 1, -1.0), (700, 64, -1.0), (700, 64, 1.0), (700, 64, 0.0), (60, 64, -1.0),
                                               # from 1025 blocks on: the sweeps
                                               (1030, 1, -1.0), (1030, 64, -1.0), (1030, 64, 1.0), (1030, 64, 0.0)])
def test_bound_of_scores_of_one_sign(s3r, oracle, dtype, n_blk, topk, lean):  # noqa: F811
    """The bound on the k-th score where all scores are negative, positive or of both signs, and where fewer than k
    blocks exist."""
    wl = workloads.Workload(f"lean_{dtype}_{n_blk}_{topk}_{lean}", 1, 16 * n_blk, 1, 64, dtype, 16, topk, 98, "normal")
    q, k, v = workloads.make_inputs(wl)
    if lean != 0.0:
        q.add_(lean)
        k.add_(1.0)
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 16, topk)
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 16,
                                                 topk, dtype, label=wl.name)))


@pytest.mark.parametrize("heads,n_tok", [(17, 41120), (17, 41121), (17, 41137), (16, 43691)])   # 256 MiB of q, k, v in bf16 and past it
@pytest.mark.parametrize("block", [16, 32, 64, 128])
def test_pooling_with_rows_requested_at_once_and_one_by_one(s3r, heads, n_tok, block):  # noqa: F811
    wl = workloads.Workload("pool_line", 1, n_tok, heads, 64, "bf16", block, 1, 108, "outliers")
    tensors = workloads.make_inputs(wl, device="cuda")
    n_blk = (n_tok + block - 1) // block
    outs = [torch.full((heads, n_blk, 64), float("nan"), device="cuda") for _ in range(3)]
    s3r.speed3r_pool_blocks(*tensors, *outs, block)
    for x, got in zip(tensors, outs):
        x = torch.cat([x.double(), x.new_zeros((n_blk * block - n_tok, heads, 64)).double()]).view(n_blk, block, heads, 64)
        lens = torch.full((n_blk, 1, 1), float(block), device="cuda", dtype=torch.double)
        lens[-1] = n_tok - (n_blk - 1) * block
        want = (x.sum(1) / lens).permute(1, 0, 2)
        # up to 128 terms, each added with 2^-24 of the sum so far, and the division
        bound = (x.abs().sum(1) / lens).permute(1, 0, 2) * (block + 1) * 2.0 ** -24
        assert ((got.double() - want).abs() <= bound).all()


@pytest.mark.parametrize("dtype,block,n_tok,heads,topk,n_forced", [
    ("bf16", 64, 64 * 9 + 33, 2, 5, 0), ("bf16", 64, 64 * 300 + 1, 3, 7, 2),     # two pairs of waves (few query blocks), one pair
    ("bf16", 64, 64 * 200 + 5, 2, 20, 120), ("bf16", 128, 128 * 9 + 70, 3, 4, 0),  # long rows, blocks of 128
    ("bf16", 16, 16 * 37 + 3, 3, 5, 1), ("bf16", 32, 32 * 21 + 17, 3, 5, 0),
    ("f32", 16, 16 * 37 + 3, 3, 5, 0), ("f32", 32, 32 * 21 + 17, 3, 5, 0), ("f32", 64, 64 * 9 + 33, 3, 5, 0), ("f32", 128, 128 * 9 + 70, 3, 4, 0),
])
@pytest.mark.parametrize("gated", [False, True])
def test_every_channel_is_merged_with_its_own(s3r, dtype, block, n_tok, heads, topk, n_forced, gated):  # noqa: F811
    """out = g o_comp + (1 - g) o_sel channel by channel, from the outputs themselves (o_sel as it was stored)."""
    wl = workloads.Workload("merge", 1, n_tok, heads, 64, dtype, block, topk, 109, "normal")
    q, k, v = workloads.make_inputs(wl, device="cuda")
    gate = workloads.make_gate_logits(wl, device="cuda") if gated else None
    res = run_device(s3r, q, k, v, block, topk, gate=gate, forced=list(range(n_forced)) if n_forced else None)
    g = torch.sigmoid(gate.double()) if gated else torch.full(q.shape, 0.5, device="cuda", dtype=torch.double)
    comp = res["o_comp"].double().permute(1, 0, 2)[torch.arange(n_tok, device="cuda") // block]
    sel, out = res["o_sel"].double(), res["out"].double()
    # rounding of o_sel and of out to 8 significant bits (2^-8 at most, just above a power of two); fp32: the few operations of the merge
    ulp = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -22
    # the gate: e^-x to 2^-20 (hardware exponential, logits up to 6 or so) moves it by g (1 - g) 2^-20 <= 2^-22, and 1 + e, 1 / ., 1 - g
    # are rounded at a size of up to 1 (so that 1 - g is not exact to its own size)
    bound = ulp * ((1 - g) * sel.abs() + out.abs()) + 2.0 ** -21 * (comp.abs() + sel.abs())
    assert ((out - (g * comp + (1 - g) * sel)).abs() <= bound).all()


@pytest.mark.parametrize("n_tok,heads,topk,n_forced", [
    (64 * 2, 1, 2, 0), (64 * 9 + 1, 2, 1, 0), (64 * 9 + 33, 2, 3, 0), (64 * 9 + 31, 3, 4, 0), (64 * 9 + 31, 3, 5, 0), (64 * 9 + 33, 2, 6, 1), (64 * 40, 1, 33, 4), (64 * 70 + 5, 1, 64, 1),
    (64 * 85, 3, 5, 0), (64 * 85 + 1, 3, 5, 0),       # 255 and 258 query blocks: two units in work at a time, one
])
@pytest.mark.parametrize("strided", [False, True])
def test_two_units_at_a_time_for_few_fp32_query_blocks(s3r, oracle, n_tok, heads, topk, n_forced, strided):  # noqa: F811
    wl = workloads.Workload(f"few_f32_{n_tok}_{heads}_{topk}", 1, n_tok, heads, 64, "f32", 64, topk, 110, "outliers")
    tensors = workloads.make_inputs(wl)
    dev = [t.cuda() for t in tensors]
    if strided:
        dev = list(torch.stack(dev, dim=1).unbind(1))
    forced = list(range(n_forced)) if n_forced else None
    res = run_device(s3r, *dev, 64, topk, forced=forced)
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, *(to_host_f32(t) for t in tensors), None, 64, topk, "f32",
                                                 label=wl.name, forced=forced)))


@pytest.mark.parametrize("n_tok,heads,topk,n_forced", [
    (64 * 16, 16, 15, 0), (64 * 16, 16, 16, 0), (64 * 17, 16, 16, 0),     # 256 query blocks and 272; 15 and 16 blocks a row
    (64 * 21 - 1, 12, 17, 0), (64 * 21 - 60, 12, 18, 1), (64 * 40 + 5, 1, 19, 0), (64 * 128, 2, 128, 0), (64 * 130, 1, 101, 26),
])
def test_four_pairs_of_waves_for_few_query_blocks(s3r, oracle, n_tok, heads, topk, n_forced):  # noqa: F811
    wl = workloads.Workload(f"four_pairs_{n_tok}_{heads}_{topk}", 1, n_tok, heads, 64, "bf16", 64, topk, 111, "outliers")
    q, k, v = workloads.make_inputs(wl)
    forced = list(range(n_forced)) if n_forced else None
    res = run_device(s3r, q.cuda(), k.cuda(), v.cuda(), 64, topk, forced=forced)
    log(f"{wl.name}: " + str(compare_with_oracle(oracle, res, to_host_f32(q), to_host_f32(k), to_host_f32(v), None, 64,
                                                 topk, "bf16", forced=forced, label=wl.name)))


@pytest.mark.parametrize("block,views,tpv,special,grid", [
    (16, 127, 1376, 0, None), (16, 127, 1377, 0, None),    # 256 MiB of 4 heads are 174 762 rows: 174 752 and 174 879
    (32, 127, 1376, 0, None), (32, 127, 1377, 0, None), (64, 127, 1377, 0, None), (32, 128, 1374, 5, None), (64, 128, 1374, 5, None),
    (16, 128, 1374, 5, (37, 37, 4)), (16, 518, 339, 1, (13, 26, 4)),   # windows of 16, 8, 4 and 2 cells: slots that do not exist are passed over
    (64, 128, 1374, 5, (37, 37, 8)),
])
def test_pooling_past_the_line_writes_the_same_tiles(s3r, block, views, tpv, special, grid):  # noqa: F811
    """Four heads at once against the same heads two at a time, whose pooling stays below the line between its two forms: every
    output comes from the tiles and the means it writes."""
    assert 2 * views * tpv * 3 * 128 < 256 * 2 ** 20
    wl = workloads.Workload(f"pool_tiles_{block}", views, tpv, 4, 64, "bf16", block, 4, 115, "outliers")
    tensors = [*workloads.make_inputs(wl, device="cuda"), workloads.make_gate_logits(wl, device="cuda")]
    image = (torch.arange(views * tpv, device="cuda") % tpv) >= special

    def call(heads):
        q, k, v, gate = (x[:, heads].contiguous() for x in tensors)
        return run_device(s3r, q, k, v, block, 4, gate=gate, tokens_per_view=tpv, special_per_view=special, grid=grid)

    whole = call(slice(0, 4))
    for heads in (slice(0, 2), slice(2, 4)):
        part = call(heads)
        for name in ("idx", "o_comp"):
            assert torch.equal(whole[name][heads], part[name]), name
        assert torch.equal(whole["lse"][heads][:, image], part["lse"][:, image])
        for name in ("o_sel", "out"):
            assert torch.equal(whole[name][image][:, heads], part[name][image]), name
        if special:   # another number of key splits, each share's probabilities rounded against its own maximum
            assert_close(to_host_f32(whole["out"][~image][:, heads]), to_host_f32(part["out"][~image]), TOL["bf16"], wl.name)
