"""GPU parity at the edges of the kernels' tiles, lists and dispatch rules, against the oracle: the same comparisons as in
test_gpu_rows.py and test_gpu_configs.py (token ids, trees and masks bit for bit, reals within their 1e-5)."""
import numpy as np
import pytest
import torch

import workloads as W
from _harness import close, make_gpu, make_oracle, run_both, to_np, ORACLE_THREADS
from test_gpu_configs import _compare_reranked
from test_gpu_rows import adversarial_rows, test_entropy_over_the_top_m_against_oracle as top_m_against_oracle, test_rows_against_oracle as rows_against_oracle

pytestmark = pytest.mark.gpu


# fp32 rows are read in tiles of 8192 logits by a workgroup; the bound on the top K is raised at tiles 2, 4, 8
@pytest.mark.parametrize("V,K", [(8191, 1), (8192, 64), (8193, 16), (16385, 33), (40963, 64)])
def test_fp32_rows_at_tile_edges(V, K):
    rows_against_oracle("f32", V, K, 1)


# fp32: tiles without a finite logit ahead of others (they add nothing, a NaN among them still shows), and logits around the distance of 512 from the largest
# at which the exponential is cut off (e^-512 is nothing beside 1, whatever the sums hold: the tolerance is that of all rows)
@pytest.mark.parametrize("V,splits", [(16384, 1), (20001, 1), (40963, 3)])
def test_fp32_masked_tiles_and_far_logits(V, splits):
    from oracle import ref_row
    from paper_2502_13652_amd import C2TContext
    g = torch.Generator().manual_seed(V)
    x = torch.randn((7, V), generator=g)
    x[0, :8192] = x[1, :8192] = x[5, :8192] = -float("inf")
    x[1, 8192:-3] = -float("inf")                              # three finite logits in all
    x[2] = x[2].mul(100).sub(511)
    x[2, V - 1] = 0.0
    x[3] = torch.linspace(-513, -511, V)
    x[3, V // 2] = 0.0
    x[4] = x[4] * 1000                                         # the maximum is raised often, by more than 512
    x[5, 77] = float("nan")
    x[6] = -3e38
    x[6, [5, V - 2]] = torch.tensor([3e38, 3e38])
    per = torch.full((7, 1, (V + 3) // 4 * 4), float("inf")); per[:, 0, :V] = x
    ctx = C2TContext(7, V, 1, 5, 1, 1, 2, 0, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.set_row_splits(splits, splits)
    ctx.reset()
    ctx.expand_layer(per.cuda())
    c, out = to_np(ctx.candidates()), to_np(ctx.finalize_tree())
    np.testing.assert_array_equal(out["status"] & 1, [0, 0, 0, 0, 0, 1, 0])
    for b in (0, 1, 2, 3, 4, 6):
        r = ref_row(x[b].numpy(), 5)
        np.testing.assert_array_equal(c["token"][b, :5], r["ids"], err_msg=str(b))
        assert close(c["p"][b, :5], r["p"].astype(np.float32), atol=1e-37).all(), b
        assert close(c["H"][b, 0], np.float32(r["H"]), atol=V * 2.0 ** -53).all(), b


# bf16 lists of K to 2K-1 elements, ranked by four lanes or more to an element up to 128 of them
@pytest.mark.parametrize("K", [16, 17, 32, 33, 63, 64])
def test_bf16_lists_at_the_ranking_s_edges(K):
    rows_against_oracle("bf16", 8191, K, 1)


# The bound of the K-th largest bf16 logit: column maxima, the largest, four rows of them or two merged runs; the exact K-th largest above 32.  Rows shorter
# than a sweep of the workgroup, a cell and a group of four sweeps, and beyond
@pytest.mark.parametrize("V,K", [(4099, 1), (72, 2), (4097, 4), (520, 5), (32771, 15), (16385, 16), (200, 17), (65541, 17), (4099, 31), (32776, 32), (49163, 33), (8279, 31),
                                 (12280, 32), (12288, 32), (12289, 17)])
def test_bf16_rows_where_the_bound_changes(V, K):
    rows_against_oracle("bf16", V, K, 0)


# Splits of short bf16 rows that hold fewer than K logits: all of them are listed, wherever the bound comes from, and none of the cells without a chunk
@pytest.mark.parametrize("V,K,splits", [(100, 64, 2), (70, 33, 4), (1030, 64, 33), (40, 32, 3)])
def test_bf16_segments_of_fewer_than_k_logits(V, K, splits):
    rows_against_oracle("bf16", V, K, splits)


# Rows whose large logits lie next to each other: likely ids that are neighbours, a stretch of ids that is allowed, ids in order of frequency; few values
def neighbouring_rows(V, rng):
    rows = {}
    for w in (100, 400, 1000, 4000):
        at = int(rng.integers(0, V - w))
        rows["likely_%d" % w] = r = 3 * rng.standard_normal(V); r[at:at + w] += 25
        rows["allowed_%d" % w] = r = np.full(V, -np.inf); r[at:at + w] = 3 * rng.standard_normal(w)
    rows["by_frequency"] = 2 * rng.standard_normal(V) - 1.05 * np.log(np.arange(1, V + 1))
    rows["nine_values"] = 0.5 * rng.integers(0, 9, V) - 3.25
    rows["steps_of_a_quarter"] = np.round(4 * (rng.standard_normal(V) - 40)) / 4
    rows["lowest_and_masked"] = r = np.full(V, -np.inf); r[::41] = -127.5; r[V // 3] = 2.0      # the K-th largest is the lowest value of the window
    rows["few_lowest_and_masked"] = r = np.full(V, -np.inf); r[5:V:V // 70] = -127.5
    return list(rows), np.stack(list(rows.values())).astype(np.float32)


# bf16 rows dealt out to B sequences (one row each) against the oracle: every one of the equal rows
def dealt_rows_against_oracle(names, rows, K, B, M=0, splits=0, turns=1):
    from oracle import ref_entropy_top_m, ref_row
    from paper_2502_13652_amd import C2TContext
    n, V = rows.shape
    x = torch.full((n, 1, (V + 7) // 8 * 8 + 8), float("inf"), dtype=torch.bfloat16)
    x[:, 0, :V] = torch.from_numpy(rows).to(torch.bfloat16)
    ctx = C2TContext(B, V, 1, K, 1, 1, 2, 1, 0.0, entropy_top_m=M)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    print("%d rows, %d of them different, V=%d K=%d M=%d splits=%d" % (B, n, V, K, M, splits), flush=True)
    if splits:
        ctx.set_row_splits(splits, splits)
    xd = x.cuda()[torch.arange(B, device="cuda") % n].contiguous()
    bits = x[:, 0, :V].contiguous().view(torch.int16).numpy().view(np.uint16)
    refs = [ref_row(bits[b], K) for b in range(min(n, B))]
    H_refs = [ref_entropy_top_m(bits[b], M) if M else refs[b]["H"] for b in range(min(n, B))]
    for _ in range(turns):
        ctx.reset()
        ctx.expand_layer(xd)
        c = to_np(ctx.candidates())
        for b, (r, H) in enumerate(zip(refs, H_refs)):
            k, name = len(r["ids"]), names[b]
            for e in range(b, B, n):
                np.testing.assert_array_equal(c["token"][e, :k], r["ids"], err_msg=name)
                assert close(c["p"][e, :k], r["p"].astype(np.float32), atol=1e-37).all(), name
                assert close(c["H"][e, 0], np.float32(H), atol=V * 2.0 ** -53).all(), name        # (as in test_gpu_rows.py)


# ... in the kernel's builds for shared rows, rows alone on a CU, and four workgroups a CU
@pytest.mark.parametrize("V,K,B", [(128256, 32, 13), (128256, 16, 13), (128256, 33, 60), (8279, 31, 13), (32000, 10, 200), (32000, 32, 200), (32000, 64, 200),
                                   (20011, 1, 300), (32000, 16, 300), (65541, 20, 300), (32000, 32, 300), (32000, 64, 300)])
def test_rows_with_neighbouring_large_logits(V, K, B):
    names, rows = neighbouring_rows(V, np.random.default_rng(V + K))
    dealt_rows_against_oracle(names, rows, K, B)


# The rows of test_gpu_rows.py in the builds for four workgroups a CU (more rows than CUs) and for long rows alone on a CU, with the usual cache policy
# (up to 24 MB) and without: equal rows give equal results
@pytest.mark.parametrize("V,K,B,M", [(4099, 1, 300, 0), (4099, 17, 300, 0), (8191, 64, 300, 0), (71003, 16, 300, 0), (71003, 33, 300, 0), (32771, 32, 1100, 0), (5003, 4, 300, 37),
                                     (71003, 16, 300, 1000), (71003, 16, 150, 0), (71003, 32, 150, 1000), (128256, 17, 200, 0), (128256, 64, 200, 0), (128256, 1, 200, 1000)])
def test_adversarial_rows_in_the_builds_for_many_rows(V, K, B, M):
    names, rows = adversarial_rows(V, np.random.default_rng(V + K), True)
    dealt_rows_against_oracle(names, rows, K, B, M)


# Splits in thousands of workgroups, where wavefronts of one workgroup lie far apart: the count of the listed cells is read by all of them before it is
# set to 0 again (one row in 1500 came out wrong, of those outside the histogram's window or tied below it)
@pytest.mark.parametrize("V,K,B,M,splits", [(4391, 10, 600, 1, 5), (4391, 10, 600, 37, 2), (32000, 10, 300, 0, 3)])
def test_adversarial_rows_in_many_split_workgroups(V, K, B, M, splits):
    names, rows = adversarial_rows(V, np.random.default_rng(V + K), True)
    dealt_rows_against_oracle(names, rows, K, B, M, splits, turns=10)


# NaN, +inf and rows without a finite logit in these builds
@pytest.mark.parametrize("V,B", [(4104, 300), (71003, 150), (128256, 200)])
def test_bad_rows_in_the_builds_for_many_rows(V, B):
    from paper_2502_13652_amd import C2TContext
    rows = (2 * np.random.default_rng(V).standard_normal((6, V))).astype(np.float32)
    rows[1, V // 2], rows[2, V - 1], rows[3, :], rows[4, 0] = np.nan, np.inf, -np.inf, -np.nan
    x = torch.nn.functional.pad(torch.from_numpy(rows).to(torch.bfloat16), (0, -V % 8), value=float("nan"))
    ctx = C2TContext(B, V, 1, 4, 1, 4, 2, 1, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.reset()
    ctx.expand_layer(x.cuda()[torch.arange(B, device="cuda") % 6].unsqueeze(1))
    out = to_np(ctx.finalize_tree())
    bad = np.array([0, 1, 1, 1, 1, 0])[np.arange(B) % 6]
    np.testing.assert_array_equal(out["status"] & 1, bad)
    np.testing.assert_array_equal(out["n_nodes"], 1 - bad)


# Medians of the kernel times of one-row layers, a turn for each of the inputs [n][V] (bf16, dealt out to B rows)
def layer_times(B, K, inputs, turns):
    from paper_2502_13652_amd import C2TContext
    n, V = inputs[0].shape
    ctx = C2TContext(B, V, 1, K, 1, 1, 2, 1, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    xs = [torch.nn.functional.pad(x.to(torch.bfloat16), (0, -V % 8))[torch.arange(B, device="cuda") % n].unsqueeze(1) for x in inputs]
    for _ in range(2):                                       # (the first turns warm up)
        ctx.profile_enable(turns * len(xs))
        for i in range(turns * len(xs)):
            ctx.reset(); ctx.expand_layer(xs[i % len(xs)]); ctx.finalize_tree()
        torch.cuda.synchronize()
    return np.median(np.array(ctx.profile_read(turns * len(xs))).reshape(turns, len(xs)), axis=0)


# Where a row's large logits lie must not decide over its time: rows against the same values in random places, and
# tied rows against such with K larger logits in random places.  A second read of such rows took them 1.3 to 3 times as long
@pytest.mark.parametrize("B,K", [(256, 32), (512, 32), (300, 16), (40, 16), (1, 32)])
def test_the_place_of_large_logits_does_not_cost_a_second_read(B, K):
    V, n = 128256, min(B, 16)
    g = torch.Generator(device="cuda").manual_seed(5)
    noise, places = 3 * torch.randn((n, V), generator=g, device="cuda"), torch.randperm(V, generator=g, device="cuda")
    block = noise.clone(); block[:, 70000:71000] += 25
    few = noise.clone(); few[:, 5000:5400] += 25
    frequency = noise - 1.05 * torch.log(torch.arange(1, V + 1, device="cuda").float())
    ties = 0.5 * torch.randint(0, 9, (n, V), generator=g, device="cuda") - 3.25
    headed = ties.clone(); headed[:, places[:K]] = 5 + 0.125 * torch.arange(K, device="cuda")
    for x in (block, few, frequency):
        together, apart = layer_times(B, K, [x, x[:, places]], 30)
        assert together < 1.15 * apart, (together, apart)
    tied, free = layer_times(B, K, [ties, headed], 30)
    assert tied < 1.15 * free, (tied, free)


# Logits of zero (padding of the vocabulary) below K positive ones: nothing has to be counted again for them (a tenth of a short row's time)
def test_zeros_below_the_top_k_cost_nothing():
    x = 3 * torch.randn((3, 8279), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    zeros = x.clone(); zeros[:, 4000:4004] = 0
    with_zeros, without = layer_times(3, 10, [zeros, x], 200)
    assert with_zeros < 1.12 * without, (with_zeros, without)        # counted again: 1.2; the chunk of the zeros is counted out of line, a third of a microsecond in 11


# How a row's equal values are kept apart goes by its own length: a layer of fewer rows is not slower than one of more (150 rows of 80000, round -100, were
# slower by a seventh than 165)
@pytest.mark.parametrize("V,few,more", [(80000, 150, 165)])
def test_fewer_rows_with_few_values_are_not_slower(V, few, more):
    x = torch.randn((16, V), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    x = torch.round(2 * (x - 100)) / 2
    t_few, t_more = (layer_times(B, 10, [x], 60)[0] for B in (few, more))
    assert t_few < 1.06 * t_more, (t_few, t_more)


# Logits of the list that are equal are told apart by their ids, four a read: 160 equal ones took such layers 1.65 times as long as none, one id at a time
@pytest.mark.parametrize("B,V", [(4, 20011), (200, 32000)])
def test_equal_logits_of_a_list(B, V):
    x = torch.randn((4, V), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    tied = x.clone(); tied[:, 8000:8160] = 24.0              # in 20 chunks: all of them are listed
    t_tied, t_free = layer_times(B, 32, [tied, x], 100)
    assert t_tied < 1.6 * t_free, (t_tied, t_free)           # (1.38 to 1.50 in a dozen turns of both)


# The entropy's M-th largest logit among the first and the last bins of a lane, and past the row's positive values
@pytest.mark.parametrize("V,M", [(4099, 2), (4099, 9), (32771, 512), (520, 519)])
def test_top_m_at_a_lane_s_bins(V, M):
    top_m_against_oracle("bf16", V, M, 0)


# NaN is looked for in pairs of an fp32 row's logits, +inf in its maximum: each place of a chunk, the padding of the last one not among them
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_bad_fp32_logits_at_each_place_of_a_chunk(bad):
    from paper_2502_13652_amd import C2TContext
    V, places = 8197, [0, 1, 2, 3, 2047, 8190, 8191, 8192, 8195, 8196]
    x = torch.full((len(places) + 1, 1, 8200), float(bad))
    x[:, 0, :V] = torch.from_numpy(np.random.default_rng(8).standard_normal((len(places) + 1, V)).astype(np.float32))
    for r, at in enumerate(places):
        x[r, 0, at] = float(bad)
    ctx = C2TContext(len(places) + 1, V, 1, 4, 1, 4, 2, 0, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.set_row_splits(1, 1)
    ctx.reset()
    ctx.expand_layer(x.cuda())
    out = to_np(ctx.finalize_tree())
    np.testing.assert_array_equal(out["status"] & 1, [1] * len(places) + [0])
    np.testing.assert_array_equal(out["n_nodes"], [0] * len(places) + [1])


# Long fp32 rows of a launch with more rows than CUs: one workgroup each up to 196608 logits, and split above.  The rows are dealt out ten times and more: equal rows give equal results.
@pytest.mark.parametrize("V,K,per_row", [(49163, 64, 1), (131075, 16, 1), (196608, 8, 1), (196612, 8, 2)])
def test_long_fp32_rows_unsplit(V, K, per_row):
    from oracle import ref_row
    from paper_2502_13652_amd import C2TContext, C2TError
    names, rows = adversarial_rows(V, np.random.default_rng(V), False)
    n, B = len(names), 260
    stride = (V + 3) // 4 * 4 + 4
    x = torch.full((n, 1, stride), float("inf"))
    x[:, 0, :V] = torch.from_numpy(rows)
    xd = x.cuda()[torch.arange(B, device="cuda") % n].contiguous()
    ctx = C2TContext(B, V, 1, K, 1, 1, 2, 0, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    assert ctx.row_workgroups() == (per_row, per_row)
    with pytest.raises(C2TError):
        ctx.set_row_splits(1, 1)                             # a split count that is set keeps its limit of 49152 logits
    ctx.set_row_splits(0, 0)
    ctx.reset()
    ctx.expand_layer(xd)
    c = to_np(ctx.candidates())
    for b, name in enumerate(names):
        r = ref_row(x[b, 0, :V].numpy(), K)
        k = len(r["ids"])
        for e in range(b, B, n):
            np.testing.assert_array_equal(c["token"][e, :k], r["ids"], err_msg=name)
            assert close(c["p"][e, :k], r["p"].astype(np.float32), atol=1e-37).all(), name
            assert close(c["H"][e, 0], np.float32(r["H"]), atol=V * 2.0 ** -53).all(), name       # (as in test_gpu_rows.py)


# bf16 rows that mask part of their vocabulary, one workgroup each: whole groups of eight sweeps (32768 logits), a rest, a partial chunk
@pytest.mark.parametrize("V", [32768, 36865, 65549])
def test_masked_bf16_rows_alone_on_a_cu(V):
    rows_against_oracle("bf16", V, 16, 1)


# The masked loop is taken by the wavefronts of whose first eight chunks (512 logits, 4096 apart) half hold a masked logit: masked
# stretches of whole and partial sweeps of the workgroup, single tokens in them, shares around one logit a chunk
@pytest.mark.parametrize("V", [32768, 40007, 65549])
@pytest.mark.parametrize("mask", [-float("inf"), -1e9])
def test_bf16_masks_at_the_loop_s_choice(V, mask):
    rng = np.random.default_rng(V)
    names, rows = [], []
    for head in (1, 4095, 4096, 12288, 12289, 16383, 16384, 16385, 28672, 32767):
        names.append("first %d" % head); r = 2 * rng.standard_normal(V); r[:head] = mask; rows.append(r)
        names.append("but the first %d" % head); r = 2 * rng.standard_normal(V); r[head + 1:] = mask; r[:16] = rng.standard_normal(16); rows.append(r)
    for n in (1, 2, 3, 4, 5, 8):
        for at in (0, 511, 3584, 4095):
            names.append("%d chunks, token %d" % (n, at)); r = 2 * rng.standard_normal(V); r[at + 4096 * rng.choice(8, n, replace=False)] = mask; rows.append(r)
    for share in (0.0005, 0.002, 0.005, 0.01):
        names.append("share %g" % share); r = 2 * rng.standard_normal(V); r[rng.random(V) < share] = mask; rows.append(r)
    _rows_equal_oracle(names, np.stack(rows).astype(np.float32), 16, 1, torch.bfloat16)


# Rows that mask one token are counted by the usual loop (256 rows of 128256: 22 us both; 27 by the masked one), rows that mask one
# in two hundred by the masked one (30 us; 39 where some wavefronts take the usual one)
def test_bf16_layer_time_of_few_masked_tokens():
    g = torch.Generator(device="cuda").manual_seed(3)
    x = (3 * torch.randn((256, 128256), generator=g, device="cuda")).to(torch.bfloat16)
    one, few = x.clone(), x.clone()
    one[:, 0] = -float("inf")
    few[torch.rand(x.shape, generator=g, device="cuda") < 0.005] = -float("inf")
    took = [_row_layer_us(y, 16, 1) for y in (x, one, few)]
    print("none %.1f us, one %.1f us, one in 200 %.1f us" % tuple(took), flush=True)
    assert took[1] < 1.15 * took[0] and took[2] < 1.55 * took[0]


@pytest.mark.parametrize("dtype,V", [("bf16", 40000), ("f32", 20000)])
def test_bad_logits_among_masked_ones(dtype, V):
    from paper_2502_13652_amd import C2TContext
    rng = np.random.default_rng(V)
    rows = (2 * rng.standard_normal((8, V))).astype(np.float32)
    rows[rng.random((8, V)) < 0.3] = -np.inf
    at = V - 5000                                            # (a NaN with its sign set is a code of its own in the histogram pass)
    neg_nan = np.float32(np.uint32(0xFFC00000).view(np.float32))
    for r, v in ((1, np.nan), (2, neg_nan), (3, np.inf), (5, -np.inf), (6, neg_nan)):
        rows[r, at] = v
    rows[6, 3] = neg_nan
    x = torch.from_numpy(rows).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    if dtype == "bf16":
        x.view(torch.int16)[2, at] = np.int16(np.uint16(0xFFC0).view(np.int16))
        x.view(torch.int16)[6, [3, at]] = torch.tensor([-1, -64], dtype=torch.int16)      # 0xFFFF and 0xFFC0
    ctx = C2TContext(8, V, 1, 4, 1, 4, 2, 1 if dtype == "bf16" else 0, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.set_row_splits(1, 1)
    ctx.reset()
    ctx.expand_layer(x.view(8, 1, V).cuda())
    out = to_np(ctx.finalize_tree())
    np.testing.assert_array_equal(out["status"] & 1, [0, 1, 1, 1, 0, 0, 1, 0])
    np.testing.assert_array_equal(out["n_nodes"], np.where(out["status"] & 1, 0, 1))          # one frontier slot: the best child


def _layers(cfg):
    cache = {}

    def get(l):
        if l not in cache:
            x = W.logits_layer(cfg, l, device="cuda")
            per = 8 if cfg["dtype"] == "bf16" else 4
            xp = torch.full((cfg["B"], cfg["F"], (cfg["V"] + per - 1) // per * per), float("inf"), dtype=x.dtype, device=x.device)
            xp[:, :, :cfg["V"]] = x
            cache[l] = xp[:, :, :cfg["V"]]
        return cache[l]
    return get


def _cfg(**k):
    return dict(dict(idx=89, B=3, V=3001, dtype="bf16", D=4, F=8, K=8, h=8, beta=0.3, N=30, zipf_s=1.0, sigma=(1.0, 4.0), spike_frac=0.1,
                     desc="edges"), **k)


# candidates of a sequence: one a thread up to 512, several beyond; survivors ranked directly up to 64, lists of up to 128
# behind a bound, radix select beyond; classifiers from 48 hidden units on evaluated by the workgroup, in one or several blocks
@pytest.mark.parametrize("F,K,h,N,dtype", [(16, 32, 47, 60, "bf16"), (27, 19, 48, 100, "bf16"), (9, 57, 50, 64, "f32"), (64, 8, 12, 200, "f32"),
                                           (33, 62, 256, 300, "bf16"), (8, 8, 63, 20, "bf16"), (3, 64, 49, 12, "f32"), (1, 1, 64, 3, "bf16")])
def test_sequence_step_at_its_edges(F, K, h, N, dtype):
    total = 0
    for seed, beta in ((0, 0.0), (1, 0.2), (2, 0.4)):
        cfg = _cfg(F=F, K=K, h=h, N=N, dtype=dtype, beta=beta)
        go, oo, _ = run_both(cfg, W.classifier(cfg, seed), _layers(cfg), tag="F=%d K=%d h=%d seed %d" % (F, K, h, seed))
        total += int(go["n_nodes"].sum())
    assert total > 0


# live rows dealt round the CUs (more workgroups than CUs, one round): a lane a slot to the largest frontier, sets of sequences in one to four ballots, frontiers
# of any length between none and full (confidence = the path's probability, thresholds across what the layers hold); and the fixed orders beyond
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,F,K", [(5, 64, 8), (17, 60, 2), (63, 16, 4), (64, 16, 4), (65, 15, 4), (129, 7, 4), (255, 4, 4), (256, 4, 4), (300, 3, 4), (70, 33, 2)])
def test_ragged_frontiers_dealt_to_workgroups(B, F, K, dtype):
    lengths = set()
    for beta in (0.02, 0.2):
        cfg = _cfg(B=B, F=F, K=K, h=2, N=3 * F, D=5, V=520, dtype=dtype, beta=beta)
        W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
        cls = (W1, np.zeros(2, np.float32), np.array([8, 0], np.float32), -4.0)          # C = sigmoid(8 P - 4)
        go, oo, _ = run_both(cfg, cls, _layers(cfg), tag="B=%d F=%d beta %g" % (B, F, beta))
        lengths |= set(go["n_nodes"].tolist())
    assert len(lengths) > 2


# the same with several workgroups a row: the row and its split from one index, splits that are empty (68 logits in seven: two are in bf16, one in fp32) or hold fewer
# than K logits, the records of a row merged by whichever split is done last, the entropy over the M largest of the merged row, ended sequences noted by their first split alone
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,F,K,V,splits,M", [(17, 20, 8, 520, 2, 0), (5, 64, 4, 520, 3, 0), (63, 5, 4, 520, 3, 37), (9, 16, 8, 68, 7, 0), (65, 2, 4, 68, 7, 0), (256, 2, 2, 520, 2, 0)])
def test_ragged_frontiers_of_split_rows(B, F, K, V, splits, M, dtype):
    assert 256 < B * F * splits <= 1024 and B <= 256          # one round of workgroups, more of them than CUs
    chunks = -(-V // (8 if dtype == "bf16" else 4))
    assert splits < 7 or -(-chunks // splits) * (splits - 1) >= chunks          # the last split is empty
    lengths = set()
    for beta in (0.02, 0.2):
        cfg = _cfg(B=B, F=F, K=K, h=2, N=3 * F, D=5, V=V, dtype=dtype, beta=beta, entropy_top_m=M)
        W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
        cls = (W1, np.zeros(2, np.float32), np.array([8, 0], np.float32), -4.0)
        go, oo, _ = run_both(cfg, cls, _layers(cfg), splits=(splits, splits), tag="B=%d F=%d splits %d beta %g" % (B, F, splits, beta))
        lengths |= set(go["n_nodes"].tolist())
    assert len(lengths) > 2


# more than 64 survivors in one candidate a thread, of which 1 to 16 are kept: the bound from sorted maxima, and the ballots beyond
@pytest.mark.parametrize("F,K,N", [(2, 50, 12), (3, 64, 7), (15, 30, 50), (16, 31, 60), (17, 30, 60)])
def test_sequence_step_where_the_bound_changes(F, K, N):
    test_sequence_step_at_its_edges(F, K, 8, N, "bf16")


# classifiers of a multiple of four units by four lanes a candidate, up to 16 candidates: groups of 16, 8 and 4 units, lone rows (F = 1) too
@pytest.mark.parametrize("F,K,h,N,dtype", [(10, 16, 28, 60, "bf16"), (7, 15, 4, 60, "f32"), (1, 16, 20, 4, "bf16"), (1, 1, 12, 3, "f32"), (16, 3, 44, 60, "bf16")])
def test_classifiers_by_four_lanes(F, K, h, N, dtype):
    test_sequence_step_at_its_edges(F, K, h, N, dtype)


# classifiers of a multiple of four units, evaluated by the workgroup: one and more blocks of activations, an odd number of fours in one, one candidate
@pytest.mark.parametrize("F,K,h,N,dtype", [(4, 64, 256, 60, "bf16"), (5, 33, 52, 60, "f32"), (3, 1, 48, 8, "bf16"), (7, 20, 252, 60, "f32")])
def test_wide_classifiers_by_fours(F, K, h, N, dtype):
    test_sequence_step_at_its_edges(F, K, h, N, dtype)


# the mask is written sixteen bytes a store in slices of 16384 bytes: budgets around multiples of sixteen and slice edges
@pytest.mark.parametrize("N", [1, 15, 16, 17, 127, 128, 129, 181, 500, 1023])
def test_mask_at_store_and_slice_edges(N):
    cfg = _cfg(B=2, V=700, D=18, F=64, K=8, h=4, beta=0.0, N=N)
    go, oo, _ = run_both(cfg, W.classifier(cfg, 0), _layers(cfg), per_layer=False, tag="N=%d" % N)
    assert (go["n_nodes"] == N).all()
    # caller's buffers at any alignment
    ctx = make_gpu(cfg, W.classifier(cfg, 0))
    ctx.reset()
    for l in range(cfg["D"]):
        ctx.expand_layer(_layers(cfg)(l))
    out = ctx.new_tree_out()
    room = torch.full((2 * N * N + 8,), 7, dtype=torch.uint8, device="cuda")
    out["mask"] = room[3:3 + 2 * N * N].view(2, N, N)
    ctx.finalize_tree(out)
    np.testing.assert_array_equal(out["mask"].cpu().numpy(), go["mask"])
    assert (room[:3] == 7).all() and (room[3 + 2 * N * N:] == 7).all()


# up to 160 nodes out behind a bound, radix select beyond; the mask in the same kernel up to 256; histories beyond 8192
# candidates are not kept in LDS; F * K = 1
@pytest.mark.parametrize("D,F,K,n_outs", [(6, 16, 16, (1, 64, 159, 160, 161, 256, 257, 700)), (9, 32, 32, (60, 160, 161, 900)), (12, 1, 1, (1, 5, 12, 20))])
def test_reranking_at_its_edges(D, F, K, n_outs):
    for seed in range(2):
        cfg = _cfg(B=3, V=1500, D=D, F=F, K=K, h=4, beta=0.0, N=min(1024, D * F), rerank=1)
        cls = W.classifier(cfg, seed)
        layers = _layers(cfg)
        g, o = make_gpu(cfg, cls), make_oracle(cfg, cls)
        g.reset(); o.reset()
        for l in range(D):
            x = layers(l)
            g.expand_layer(x)
            if o.frontier()["n_frontier"].sum() > 0:
                o.expand_layer(W.as_numpy_bits(x), threads=ORACLE_THREADS)
        torch.cuda.synchronize()
        for n_out in n_outs:
            _compare_reranked(g, o, [0, 1, 2], n_out, "rerank D=%d F=%d K=%d seed %d" % (D, F, K, seed))


def _row_layer_us(x, K, splits=0, n=9):
    """Duration (the kernel's own begin and end; the least of three medians) of a layer whose rows are the sequences' root rows: x [rows][V]."""
    from paper_2502_13652_amd import C2TContext
    rows, V = x.shape
    ctx = C2TContext(rows, V, 1, K, 1, 1, 2, x.dtype, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.set_row_splits(splits, splits)
    ctx.profile_enable(n)
    us = []
    for _ in range(4):                                       # (the first to warm up)
        for _ in range(n):
            ctx.reset()
            ctx.expand_layer(x.view(rows, 1, V))
        torch.cuda.synchronize()
        us.append(float(np.median(ctx.profile_read(n))) * 1e3)
    return min(us[1:])


def _rows_equal_oracle(names, rows, K, splits, dtype=torch.float32):
    from oracle import ref_row
    from paper_2502_13652_amd import C2TContext
    B, V = rows.shape
    ctx = C2TContext(B, V, 1, K, 1, 1, 2, dtype, 0.0)
    W1 = np.zeros((2, 3), np.float32); W1[0, 0] = 1
    ctx.set_classifier(W1, np.zeros(2, np.float32), np.array([1, 0], np.float32), 0.0)
    ctx.set_row_splits(splits, splits)
    x = torch.full((B, 1, (V + 7) // 8 * 8 + 8), float("inf"), dtype=dtype)
    x[:, 0, :V] = torch.from_numpy(rows).to(dtype)
    ctx.reset()
    ctx.expand_layer(x.cuda())
    c = to_np(ctx.candidates())
    bits = W.as_numpy_bits(x[:, 0, :V])
    for b, name in enumerate(names):
        r = ref_row(bits[b], K)
        k = len(r["ids"])
        np.testing.assert_array_equal(c["token"][b, :k], r["ids"], err_msg=name)
        assert close(c["p"][b, :k], r["p"].astype(np.float32), atol=1e-37).all(), name
        assert close(c["H"][b, 0], np.float32(r["H"]), atol=V * 2.0 ** -53).all(), name       # (as in test_gpu_rows.py)


# fp32 lists that do not come out with K to 128 entries: ties at and above the K-th value, from one more than the list is ranked with
# to one more than it holds; fewer finite logits than K; logits that follow a masked tile, which overflow it; maxima in fewer
# lanes than K (a period of 2048 logits), up to the general path.  V: one tile, several, rows split by the caller
@pytest.mark.parametrize("V,splits", [(4000, 1), (16387, 1), (49152, 1), (131075, 3)])
@pytest.mark.parametrize("K", [1, 10, 64])
def test_fp32_lists_that_are_long_or_short(V, splits, K):
    rng = np.random.default_rng(V + K)
    names, rows = [], []

    def add(name, r):
        names.append(name); rows.append(r.astype(np.float32))

    def noise():
        return 2 * rng.standard_normal(V)

    for n in (127, 128, 129, 511, 513, 1000, 4095, 4096, 4097):
        for value in (17.3, 16.0):                           # (a value whose low bits the bound keeps or drops)
            if n < V:
                r = noise(); r[rng.choice(V, n, replace=False)] = value; add("%d tied at %g" % (n, value), r)
                r = r.copy(); r[rng.choice(V, 5, replace=False)] = 17.5; add("the same below five", r)
    for mask in (-np.inf, -1e9, -3.4028234663852886e38):
        for n in (1, 3, 9, 10, 63, 64, 200):
            r = np.full(V, mask); r[rng.choice(V, n, replace=False)] = rng.standard_normal(n); add("%d not masked by %g" % (n, mask), r)
        for head in (1, 2047, 8192, 16384, 24576):
            if head < V:
                r = noise(); r[:head] = mask; add("%d masked by %g ahead" % (head, mask), r)
    add("ascending", np.sort(noise()))
    add("ascending integers", np.floor(np.sort(8 * rng.standard_normal(V))))
    for lanes in (1, 9, 30, 63):
        r = noise(); r[(np.arange(V) // 4) % 512 < lanes] += 30.0; add("maxima in %d lanes" % lanes, r)
    print("V=%d splits=%d K=%d: %d rows" % (V, splits, K, len(rows)), flush=True)
    _rows_equal_oracle(names, np.stack(rows), K, splits)


# fp32: how many lanes of a wavefront reach the bound in a chunk (one adds to the list's length for itself, several at once): one, two and all of them, with one
# to four logits each, in the first wavefront's chunk, a later one's and the row's last, which may be partial or narrower than a wavefront
@pytest.mark.parametrize("V", [255, 4097, 20003, 40962])
@pytest.mark.parametrize("K", [1, 10, 64])
def test_fp32_lanes_that_reach_the_bound(V, K):
    rng = np.random.default_rng(V + K)
    names, rows = [], []
    for at in sorted({0, 37 * 256 % max(V // 1024 * 1024, 256), (V - 1) // 256 * 256}):
        for lanes in ([0], [63], [0, 1], [5, 62], [1, 2, 3, 40], range(64)):
            for each in ([0], [3], [0, 1, 2, 3]):
                ids = np.array([at + 4 * i + j for i in lanes for j in each])
                ids = ids[ids < V]
                r = rng.standard_normal(V); r[ids] = 8 + np.round(rng.standard_normal(len(ids)))
                names.append("%d lanes, %d each, at %d" % (len(lanes), len(each), at)); rows.append(r.astype(np.float32))
    _rows_equal_oracle(names, np.stack(rows), K, 1)


# 256 rows of 128256 equal logits took 2.26 times as long as rows of which few reach the bound where every logit took its place by itself (88.9 us, 39.3), 2.00 times so
def test_fp32_layer_time_of_equal_logits():
    g = torch.Generator(device="cuda").manual_seed(3)
    x = 3 * torch.randn((256, 128256), generator=g, device="cuda")
    equal, usual = _row_layer_us(torch.ones_like(x), 16), _row_layer_us(x, 16)
    print("equal %.1f us, usual %.1f us" % (equal, usual), flush=True)
    assert equal < 2.13 * usual


# Such rows take little longer than others: 320 rows of 32000 take 24 us, 23 to 51 us if they are tied, masked or sorted.  The bound is
# what the second read of an overflowed segment and the search for ties can cost: before there were rows of 2300 us (3000 tied) and
# of 70 (three finite logits); ten rows of 4000 took 3400 us where 11 are usual (18 now).
@pytest.mark.parametrize("rows,V", [(10, 4000), (320, 32000)])
def test_fp32_layer_time_of_tied_and_masked_rows(rows, V):
    g = torch.Generator(device="cuda").manual_seed(1)
    base = 3 * torch.randn((rows, V), generator=g, device="cuda")
    usual = _row_layer_us(base, 10)
    few = torch.full((rows, V), -float("inf"), device="cuda")
    few[:, [0, V // 2, V - 1]] = torch.tensor([1.0, 2.0, 2.0], device="cuda")
    tied = base.clone()
    tied[:, torch.randperm(V, generator=g, device="cuda")[:3000]] = 17.3
    ahead = base.clone()
    ahead[:, :V // 2] = -float("inf")
    took = {}
    for name, x, most in (("three finite", few, 1.6), ("three above -1e9", few.clamp_min(-1e9), 2.5), ("3000 tied", tied, 2.5),
                          ("all equal", torch.ones_like(base), 2.5), ("half masked ahead", ahead, 2.0), ("ascending", base.sort(1).values, 2.2)):
        took[name] = (_row_layer_us(x, 10) / usual, most)
    print("usual %.1f us," % usual, ", ".join("%s %.2f" % (k, v[0]) for k, v in took.items()), flush=True)
    assert all(t < most for t, most in took.values())


# What a layer of fp32 rows takes depends little on K (320 rows of 32000: 24 us with K = 10, 35 us with K = 64): the logits that
# reach the bound on the top K, which are ranked, stay few.  With a bound from 64 columns 300 of them did at K = 64: 88 us.
def test_fp32_layer_time_at_large_k():
    g = torch.Generator(device="cuda").manual_seed(1)
    x = 3 * torch.randn((320, 32000), generator=g, device="cuda")
    small, large = _row_layer_us(x, 10), _row_layer_us(x, 64)
    print("K=10 %.1f us, K=64 %.1f us" % (small, large), flush=True)
    assert large < 2 * small


# Equal confidences are usual deep in a tree, and rows share tokens: ten rows of ten such candidates take little longer than others
# (14 and 16 us; 23 where each tied candidate's rank was counted by one lane).
def test_layer_time_of_equal_confidences():
    V, F, K = 8000, 10, 10
    g = torch.Generator(device="cuda").manual_seed(1)
    bias = -1.05 * torch.log(torch.rand((1, 1, V), generator=g, device="cuda") * V + 1)
    x = [(3 * torch.randn((1, F, V), generator=g, device="cuda") + bias).to(torch.bfloat16) for _ in range(2)]
    took = []
    for w2 in (1.0, 0.0):
        from paper_2502_13652_amd import C2TContext
        ctx = C2TContext(1, V, F, K, 2, 100, 4, 1, 0.0)
        W1 = np.zeros((4, 3), np.float32); W1[0, 0] = 1
        ctx.set_classifier(W1, np.zeros(4, np.float32), np.array([w2, 0, 0, 0], np.float32), 0.0)
        ctx.profile_enable(30)
        us = []
        for _ in range(4):                                   # (the first to warm up)
            for _ in range(15):
                ctx.reset()
                for l in x:
                    ctx.expand_layer(l)
            torch.cuda.synchronize()
            us.append(float(np.median(ctx.profile_read(30)[1::2])) * 1e3)
        took.append(min(us[1:]))
    print("varied %.1f us, equal %.1f us" % tuple(took), flush=True)
    assert took[1] < 1.4 * took[0]


# Few nodes out of many candidates with equal scores cost no more than many: 60 of 1536 17 us, 161 of them 15 us (46 and 15 when
# everything that reached the bound was ranked).
def test_reranking_time_with_ties():
    from paper_2502_13652_amd import C2TContext
    B, D, F, K = 32, 6, 16, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    ctx = C2TContext(B, 2000, F, K, D, 96, 4, 1, 0.0, rerank=1)
    W1 = np.zeros((4, 3), np.float32); W1[0, 0] = 1; W1[1, 1] = -0.1
    ctx.set_classifier(W1, np.full(4, 0.5, np.float32), np.array([1, 1, 0, 0], np.float32), 0.0)
    ctx.reset()
    for _ in range(D):
        ctx.expand_layer((3 * torch.randn((B, F, 2000), generator=g, device="cuda")).to(torch.bfloat16))
    took = []
    for n_out in (60, 161):
        out, us = ctx.new_tree_out(n_out), []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                ctx.finalize_tree_reranked(n_out, out)
            b.record()
            torch.cuda.synchronize()
            us.append(a.elapsed_time(b) * 50)
        took.append(float(np.median(us)))
    print("60 out %.1f us, 161 out %.1f us" % tuple(took), flush=True)
    assert took[0] < 2 * took[1]


# Candidates of equal confidence whose rows hold the same few tokens: hundreds of equal keys are left to rank, by one, two or four lanes each
@pytest.mark.parametrize("B,V,F,K,D", [(20, 34, 32, 33, 2), (20, 33, 17, 31, 2), (20, 60, 32, 33, 2), (20, 100, 32, 33, 2), (20, 65, 32, 64, 2), (9, 33, 64, 32, 3), (20, 33, 16, 32, 2),
                                       (2, 34, 32, 33, 2)])
@pytest.mark.parametrize("dtype,M", [("bf16", 0), ("bf16", 37), ("f32", 0)])
def test_equal_confidences_of_the_same_tokens(B, V, F, K, D, dtype, M):
    cfg = dict(B=B, V=V, F=F, K=K, D=D, N=512, h=2, beta=0.3, dtype=dtype, entropy_top_m=M)
    cls = np.zeros((2, 3), np.float32), np.zeros(2, np.float32), np.zeros(2, np.float32), 0.1
    g = torch.Generator(device="cuda").manual_seed(3)
    x = 2 * torch.randn((D, B, F, V), generator=g, device="cuda")
    x = torch.nn.functional.pad(x, (0, -V % 8), value=float("inf")).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    run_both(cfg, cls, lambda l: x[l], tag="equal")
