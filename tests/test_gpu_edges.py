"""GPU: sizes at which a kernel changes the way it works (edges of tiles, of register-
resident runs, of the ranges of a launch rule), through the C ABI against the fp64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import test_gpu_block as PB                       # noqa: E402
import test_gpu_parity as P                       # noqa: E402
from gpu_progress import say as _say              # noqa: E402
from oracle import sample_attention as O           # noqa: E402
from test_gpu_block import _block_case            # noqa: E402
from test_gpu_parity import _check_out, _dev, _f64, _inputs, _score_tol, _select_case, _sparse_case   # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [63, 64, 65, 1023, 1025, 16383, 16384, 16385, 17408])
def test_select_around_the_register_resident_size(S):
    """Up to 16384 candidates are read once and kept in registers, 1024 candidates are one per
    thread; whole and partial batches of sixteen groups take different loops."""
    _say(f"select sizes S={S}")
    rng = np.random.default_rng(S)
    a = np.exp(rng.standard_normal((2, S)) * 2).astype(np.float32)
    b = (np.round(rng.random((2, S)) ** 4 * 64) / 64).astype(np.float32)      # ties and exact zeros
    for alpha in (0.3, 0.95, 0.9999):
        _select_case(a, b, alpha, alpha)


def test_sparse_attn_bitmap_in_several_segments():
    """Above 1M tokens a head's bitmaps are built in segments of 2^20 bits and the tile
    diagonals are listed by a launch of their own: strips on both sides of the cut, checked on
    the rows that meet them (bf16 probabilities against their fp64 softmax, as elsewhere)."""
    import paper_2406_15486_amd as sa
    S, w, cut = (1 << 20) + 3000, 64, 1 << 20
    _say(f"bitmap segments S={S}")
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, 1, S, 128, generator=g, device="cuda", dtype=torch.float32).bfloat16() for _ in range(3))
    off_max = (S + 255) // 256 * 256 - 1
    Ic = np.array([0, 31, 32, cut - 1, cut, cut + 1, S - 1])
    Is = np.array([100, off_max - cut - 1, off_max - cut, off_max - cut + 1, cut - 1, cut, S - 1])
    ci, si = (torch.zeros(1, S, dtype=torch.int32, device="cuda") for _ in range(2))
    ci[0, :len(Ic)] = torch.from_numpy(Ic.astype(np.int32))
    si[0, :len(Is)] = torch.from_numpy(Is.astype(np.int32))
    cc, sc = (torch.tensor([len(x)], dtype=torch.int32, device="cuda") for x in (Ic, Is))
    out, lse, _ = sa.sa_sparse_attn(q, k, v, ci, cc, si, sc, w, out_dtype=sa.SA_OUT_F32, want_lse=True)
    torch.cuda.synchronize()
    for i in (0, 63, 64, 2000, off_max - cut, off_max - cut + 500, cut - 1, cut, cut + 1, cut + 999, S - 257, S - 1):
        keys = np.unique(np.concatenate([Ic[Ic <= i], i - Is[Is <= i], np.arange(max(0, i - w + 1), i + 1)]))
        kk, vv = (t[0, 0, torch.from_numpy(keys).cuda()].double().cpu() for t in (k, v))
        s = kk @ q[0, 0, i].double().cpu() / np.sqrt(128.0)
        assert abs(float(torch.logsumexp(s, 0)) - float(lse[0, i])) < 2e-3, i
        assert (torch.softmax(s, 0) @ vv - out[0, 0, i].double().cpu()).abs().max() < 2e-2, i


def _fill(rng, n, share):
    return np.sort(rng.choice(n, int(round(share * n)), replace=False))


@pytest.mark.parametrize("S", [1, 63, 65, 255, 257, 320, 321, 1279, 1281])
def test_swept_heads_beside_two_pass_heads(S):
    """Heads with nearly full lists are swept once, the others take the two passes, in one
    launch: per-key lists of every mixture, at lengths around the key and query tiles."""
    _say(f"swept heads S={S}")
    wl, x = _inputs("glm8k", S=S, Hq=4, Hkv=2, n_sinks=min(8, S))
    rng = np.random.default_rng(S)
    Ic = [_fill(rng, S, f) for f in (0.9, 0.02, 1.0, 0.5)]
    Is = [_fill(rng, S, f) for f in (0.9, 0.01, 0.3, 0.97)]
    _sparse_case(wl, x, Ic, Is, 1, "swept", f32_out=S % 2 == 1)


@pytest.mark.parametrize("S,blk", [(1280, 64), (1333, 128), (2100, 256)])
def test_swept_heads_block_lists(S, blk):
    _say(f"swept heads S={S} blk={blk}")
    _, x = _inputs("glm8k", S=S, Hq=4, Hkv=2, n_sinks=8)
    nb = (S + blk - 1) // blk
    rng = np.random.default_rng(S)
    Ic = [_fill(rng, nb, f) for f in (0.9, 0.1, 1.0, 0.6)]
    Is = [_fill(rng, nb, f) for f in (0.8, 0.0, 0.3, 1.0)]
    _block_case(x, Ic, Is, 1, blk, "swept blocks")


@pytest.mark.parametrize("S,C,blk", [(1000, 3, 1), (1901, 5, 128)])
def test_swept_segments(S, C, blk):
    """Segments that end inside a query tile, full lists next to short ones."""
    import paper_2406_15486_amd as sa
    _say(f"swept segments S={S} C={C} blk={blk}")
    _, x = _inputs("glm8k", S=S, Hq=2, Hkv=1, n_sinks=8)
    n = (S + blk - 1) // blk
    rng = np.random.default_rng(S)
    lists = [[[_fill(rng, n, 0.9 if (m + h) % 2 else 0.05) for h in range(2)] for m in range(C)] for _ in range(2)]
    idx = [torch.zeros(C, 2, n, dtype=torch.int32) for _ in range(2)]
    cnt = [torch.zeros(C, 2, dtype=torch.int32) for _ in range(2)]
    for t in range(2):
        for m in range(C):
            for h in range(2):
                cnt[t][m, h] = len(lists[t][m][h])
                idx[t][m, h, :len(lists[t][m][h])] = torch.from_numpy(lists[t][m][h].astype(np.int32))
    out, lse, _ = sa.sa_sparse_attn_chunked(_dev(x["q"]), _dev(x["k"]), _dev(x["v"]), idx[0].cuda(), cnt[0].cuda(),
                                            idx[1].cuda(), cnt[1].cuda(), 1, C, granularity=blk, want_lse=True)
    torch.cuda.synchronize()
    qf, kf, vf = _f64(x["q"]), _f64(x["k"]), _f64(x["v"])
    for h in range(2):
        want, wlse = O.chunked_masked_attn(qf[h], kf[0], vf[0], [lists[0][m][h] for m in range(C)],
                                           [lists[1][m][h] for m in range(C)], 1, C, blk=blk)
        _check_out(out[0, h].float().cpu().numpy(), want, f"swept segments h{h}")
        assert np.abs(lse[h].cpu().numpy() - wlse).max() < 2e-3


@pytest.mark.parametrize("S,n_s,Hq", [(1087, 64, 1), (1088, 64, 1), (1111, 65, 2), (4224, 128, 2), (4500, 300, 2), (32896, 128, 1)])
def test_sample_scores_around_the_key_splits(S, n_s, Hq):
    """The keys of a query tile are cut into parts of eight tiles or more (S - n_s = 1024: the
    first cut; 32768: the most of them)."""
    import paper_2406_15486_amd as sa
    _say(f"key splits S={S} n_s={n_s}")
    _, x = _inputs("glm8k", S=S, Hq=Hq, Hkv=1, n_sinks=8)
    col, slash, lse = sa.sa_sample_scores(_dev(x["q"]), _dev(x["k"]), n_s, want_lse=True)
    torch.cuda.synchronize()
    qf, kf = _f64(x["q"]), _f64(x["k"])
    for h in range(Hq):
        wc, ws, wl = O.sample_scores(qf[h], kf[0], n_s)
        _score_tol(col[h].cpu().numpy(), wc, f"col h{h}")
        _score_tol(slash[h].cpu().numpy(), ws, f"slash h{h}")
        assert np.abs(lse[h].cpu().numpy() - wl).max() < 2e-3


# many heads: fewer workgroups than parts (8300 x 448 x 64 heads: four for eight parts)
@pytest.mark.parametrize("S,n_s,Hq,Hkv", [(1100, 65, 8, 2), (4224, 128, 8, 4), (8300, 448, 32, 2), (17000, 832, 8, 2),
                                          (33000, 1664, 8, 2), (33000, 128, 16, 4)])
def test_sample_scores_follow_from_the_sequence(S, n_s, Hq, Hkv):
    """A head's scores and log-sum-exps are the same bits in a batch of two, alone with its
    sequence, among half of the heads, and in passes over a small workspace."""
    import paper_2406_15486_amd as sa
    _say(f"scores by sequence S={S} n_s={n_s} Hq={Hq}")
    xs = [_inputs("glm8k", S=S, Hq=Hq, Hkv=Hkv, seed=s, n_sinks=8)[1] for s in (31, 32)]
    q, k = (torch.cat([_dev(x[t]) for x in xs]).contiguous() for t in "qk")
    both = [t.view(2, Hq, -1) for t in sa.sa_sample_scores(q, k, n_s, want_lse=True)]
    least = sa.sa_workspace_bytes(sa.binding.SA_OP_SAMPLE_SCORES_MIN, sa.Shape(2, Hq, Hkv, S), n_s)
    for size in (least, 3 * least):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        for a, b in zip(both, sa.sa_sample_scores(q, k, n_s, workspace=ws, want_lse=True)):
            assert torch.equal(a.view_as(b), b), f"workspace of {size} bytes"
    for b in range(2):
        for heads in (Hq, Hq // 2):
            one = sa.sa_sample_scores(q[b:b + 1, :heads].contiguous(), k[b:b + 1, :heads * Hkv // Hq].contiguous(), n_s,
                                      want_lse=True)
            for x, y in zip(both, one):
                assert torch.equal(x[b, :heads], y), f"sequence {b}, {heads} heads"
    col, slash, lse = (t[1, Hq - 1].cpu().numpy() for t in both)
    wc, ws, wl = O.sample_scores(_f64(xs[1]["q"])[Hq - 1], _f64(xs[1]["k"])[Hkv - 1], n_s)
    _score_tol(col, wc, "col")
    _score_tol(slash, ws, "slash")
    assert np.abs(lse - wl).max() < 2e-3


def test_heads_are_swept_where_the_bench_says():
    """bench.py counts the slots of a swept head or of the two passes by the kernel's own rule: the
    tiles that the kernel reports are those of a sweep on exactly these heads."""
    import bench
    S, w = 2900, 5
    _say(f"swept heads in the bench S={S}")
    wl, x = _inputs("glm8k", S=S, Hq=8, Hkv=1, n_sinks=8)
    rng = np.random.default_rng(1)
    Ic = [_fill(rng, S, f) for f in (0.05, 0.3, 0.3, 0.6, 0.6, 0.9, 1.0, 0.0)]
    Is = [_fill(rng, S, f) for f in (0.002, 0.001, 0.003, 0.0, 0.001, 0.005, 0.0, 1.0)]
    tiles = _sparse_case(wl, x, Ic, Is, w, "bench rule")
    last = np.minimum(256 * np.arange((S + 255) // 256) + 255, S - 1)
    rows = 256 * np.arange(len(last))[:, None] + 32 * np.arange(8)[None, :] + 31
    sweep_tiles, sweep_slots = int(np.minimum(last[:, None] // 64 + 1, rows // 64 + 1).sum()), int(8 * (last // 64 + 1).sum())
    swept = [bench.schedule_slots(S, Ic[h], Is[h], w) == sweep_slots for h in range(8)]
    assert any(swept) and not all(swept)
    for h in range(8):
        assert (int(tiles[h]) == sweep_tiles) == swept[h], h
        assert tiles[h] <= bench.schedule_slots(S, Ic[h], Is[h], w)


@pytest.mark.parametrize("copies", [16, 32, 48])
def test_sample_scores_of_many_heads(copies):
    """So many heads that two workgroups, or one, go through all parts of a query tile: the bits of
    one sequence alone, in every copy of it."""
    import paper_2406_15486_amd as sa
    S, n_s, Hq = 4224, 300, 8
    _say(f"scores of many heads, {copies} copies")
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k = (torch.randn(1, h, S, 128, generator=g, device="cuda").bfloat16() for h in (Hq, 2))
    one = sa.sa_sample_scores(q, k, n_s, want_lse=True)
    many = sa.sa_sample_scores(q.repeat(copies, 1, 1, 1), k.repeat(copies, 1, 1, 1), n_s, want_lse=True)
    for a, b in zip(one, many):
        assert torch.isfinite(a).all()
        for x in b.view(copies, Hq, -1):
            assert torch.equal(a, x)


def _bare(path, Hq, Hkv, S):
    """Bytes of an attention workspace without room for partial sums."""
    up = lambda b: (b + 255) // 256 * 256                                      # noqa: E731
    S_pad = up(S)
    if path == "dense":
        return Hkv * 256 * S_pad
    lists = sum(up(Hq * 4 * w) for w in (S_pad, S_pad // 32 + 2, S_pad // 32 + 24, S_pad // 64 + 8, 1))
    return Hkv * 256 * S_pad + lists + (up(Hq * 4) if path == "blocks" else Hq * 512 * S_pad)


# (path, S, Hq, Hkv, segments or block size): from one tile to the most parts (256), ragged last
# tiles and parts, a batch of segments
@pytest.mark.parametrize("path,S,Hq,Hkv,n", [("dense", 513, 1, 1, 0), ("dense", 1100, 3, 1, 0), ("dense", 3001, 8, 2, 0),
                                             ("strips", 700, 1, 1, 1), ("strips", 2305, 4, 2, 1), ("strips", 2600, 2, 1, 3),
                                             ("blocks", 577, 1, 1, 64), ("blocks", 1100, 4, 2, 256), ("blocks", 2049, 2, 1, 128),
                                             ("blocks", 2500, 4, 2, 64)])
def test_tiles_cut_into_parts(path, S, Hq, Hkv, n):
    """Small problems: a query tile's keys are cut into parts.  A workspace without room for the
    partial sums gives uncut tiles; both against the oracle."""
    import paper_2406_15486_amd as sa
    B = sa.binding
    _say(f"parts {path} S={S} Hq={Hq}")
    _, x = _inputs("glm8k", S=S, Hq=Hq, Hkv=Hkv, n_sinks=8)
    q, k, v = (_dev(x[t]) for t in "qkv")
    qf, kf, vf = (_f64(x[t]) for t in "qkv")
    sh, G = sa.Shape(1, Hq, Hkv, S), Hq // Hkv
    rng = np.random.default_rng(S)
    blk, C = (n, 1) if path == "blocks" else (1, max(n, 1))
    nb = (S + blk - 1) // blk
    shares = [(0.9, 0.9), (0.3, 0.01), (0.05, 0.3), (0.6, 0.002)]
    Ic = [[_fill(rng, nb, shares[(h + m) % 4][0]) for h in range(Hq)] for m in range(C)]
    Is = [[_fill(rng, nb, shares[(h + m) % 4][1]) for h in range(Hq)] for m in range(C)]
    ci, si = (torch.zeros(C, Hq, nb, dtype=torch.int32) for _ in range(2))
    for m in range(C):
        for h in range(Hq):
            ci[m, h, :len(Ic[m][h])] = torch.from_numpy(Ic[m][h].astype(np.int32))
            si[m, h, :len(Is[m][h])] = torch.from_numpy(Is[m][h].astype(np.int32))
    cc, sc = (torch.tensor([[len(a) for a in row] for row in lists], dtype=torch.int32) for lists in (Ic, Is))
    if path == "dense":
        need = sa.sa_workspace_bytes(B.SA_OP_DENSE_ATTN, sh)
    else:
        op = B.SA_OP_BLOCK_SPARSE_ATTN if path == "blocks" else B.SA_OP_SPARSE_ATTN
        need = sa.sa_workspace_bytes(op, sh, granularity=blk, n_chunks=C)
    bare = _bare(path, Hq, Hkv, S)
    assert bare < need
    got = []
    for size in (need, bare):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")         # NaN patterns
        if path == "dense":
            r = sa.sa_dense_attn(q, k, v, workspace=ws, want_lse=True)
        else:
            lists = [t.cuda() for t in (ci, cc, si, sc)]
            r = sa.sa_sparse_attn_chunked(q, k, v, *lists, 3, C, granularity=blk, workspace=ws, want_lse=True)
        torch.cuda.synchronize()
        got.append((r[0][0].float().cpu().numpy(), r[1].cpu().numpy()))
    assert not np.array_equal(got[0][1], got[1][1])                              # two routes
    for h in range(Hq):
        if path == "dense":
            want, wlse = O.dense_attn(qf[h], kf[h // G], vf[h // G])
        else:
            want, wlse = O.chunked_masked_attn(qf[h], kf[h // G], vf[h // G], [Ic[m][h] for m in range(C)],
                                               [Is[m][h] for m in range(C)], 3, C, blk=blk)
        for (out, lse), route in zip(got, ("parts", "uncut")):
            _check_out(out[h], want, f"{path} {route} h{h}")
            assert np.abs(lse[h] - wlse).max() < 2e-3


@pytest.mark.parametrize("S,Hq,Hkv,same", [(300, 4, 2, True), (512, 1, 1, True), (1300, 4, 2, True), (2100, 32, 4, True),
                                           (16400, 4, 1, True), (2305, 8, 2, False), (3001, 8, 2, False)])
def test_attention_of_a_batch_element_and_of_the_sequence_alone(S, Hq, Hkv, same):
    """Bit for bit where neither call cuts its tiles, or both cut them alike; else (a small problem
    that the larger batch cuts in another way) to the rounding of the probabilities: each is
    rounded to bf16 against another reference, 2^-9 of its value on either side, so the outputs
    lie within 2^-8 max |v|.  Selected lists are the same bits in either case."""
    import paper_2406_15486_amd as sa
    _say(f"batch element S={S} Hq={Hq}")
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(2, h, S, 128, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    n_s, w, f32 = min(128, S), 16, sa.SA_OUT_F32
    def run(q, k, v):
        sh = sa.Shape(q.shape[0], Hq, Hkv, S)
        lists = sa.sa_select_strips(*sa.sa_sample_scores(q, k, n_s), 0.9, 0.3, sh)
        blocks = sa.sa_select_blocks(*sa.sa_sample_scores(q, k, n_s, granularity=128), 0.6, 0.4, 128, sh)
        return lists, (sa.sa_dense_attn(q, k, v, out_dtype=f32)[0], sa.sa_sparse_attn(q, k, v, *lists, w, out_dtype=f32)[0],
                       sa.sa_block_sparse_attn(q, k, v, *blocks, w, 128, out_dtype=f32)[0])
    lists, outs = run(q, k, v)
    equal = True
    for b in range(2):
        lists1, outs1 = run(*(t[b:b + 1].contiguous() for t in (q, k, v)))
        torch.cuda.synchronize()
        for idx, cnt, idx1, cnt1 in zip(lists[::2], lists[1::2], lists1[::2], lists1[1::2]):
            assert torch.equal(cnt.view(2, Hq)[b], cnt1)
            for h in range(Hq):
                assert torch.equal(idx.view(2, Hq, S)[b, h, :int(cnt1[h])], idx1[h, :int(cnt1[h])])
        for x, y in zip(outs, outs1):
            equal = equal and torch.equal(x[b], y[0])
            assert (x[b] - y[0]).abs().max().item() <= v.abs().max().item() / 256
    assert equal == same


@pytest.mark.parametrize("S,Hq", [(8449, 9), (8193, 17)])
def test_launch_order_by_tile_and_by_head(S, Hq):
    """Launches of up to 32 query tiles per head go by tile, longer ones by head: 33 or 34 tiles
    of heads that do not divide over the eight XCDs, at once and in three launches."""
    import paper_2406_15486_amd as sa
    _say(f"launch order S={S} Hq={Hq}")
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, h, S, 128, generator=g, device="cuda").bfloat16() for h in (Hq, 1, 1))
    col, slash = sa.sa_sample_scores(q, k, 64)
    lists = sa.sa_select_strips(col, slash, 0.3, 0.2, sa.Shape(1, Hq, 1, S))
    want = sa.sa_sparse_attn(q, k, v, *lists, 16, want_lse=True, want_tiles=True)
    got = sa.sa_sparse_attn_partitioned(q, k, v, *lists, 16, Hq, 3, want_lse=True, want_tiles=True)
    torch.cuda.synchronize()
    assert torch.isfinite(want[1]).all()
    for a, b in zip(want, got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n_s", [31, 32, 33, 223, 224, 225, 255, 257, 1023, 1024, 1025, 1400])
def test_sample_scores_window_lengths(n_s):
    """The diagonal windows are as long as a chunk's rows, in steps of 32 up to 1024."""
    import paper_2406_15486_amd as sa
    S = 1400
    _say(f"window lengths n_s={n_s}")
    _, x = _inputs("glm8k", S=S, Hq=2, Hkv=1, n_sinks=8)
    col, slash = sa.sa_sample_scores(_dev(x["q"]), _dev(x["k"]), n_s)
    torch.cuda.synchronize()
    qf, kf = _f64(x["q"]), _f64(x["k"])
    for h in range(2):
        wc, ws, _ = O.sample_scores(qf[h], kf[0], n_s)
        _score_tol(col[h].cpu().numpy(), wc, f"col h{h}")
        _score_tol(slash[h].cpu().numpy(), ws, f"slash h{h}")


@pytest.mark.parametrize("test,args", [
    (P.test_sparse_attn_random_strips, (1024, 1, 1, 64)), (P.test_sparse_attn_random_strips, (1500, 4, 2, 128)),
    (P.test_sparse_attn_column_counts_around_the_loop_stretches, (0,)),
    (P.test_sparse_attn_column_counts_around_the_loop_stretches, (2,)),
    (P.test_sparse_attn_column_counts_around_the_loop_stretches, (40,)),
    (P.test_sparse_attn_nearly_full_lists, (1500, 0.7, 0.6)), (P.test_sparse_attn_nearly_full_lists, (1024, 0.95, 0.9)),
    (P.test_sparse_attn_nearly_full_lists, (2304, 0.5, 0.8)), (P.test_sparse_attn_degenerate_strip_sets, ()),
    (PB.test_block_sparse_attn_random_blocks, (1500, 4, 2, 128, 128)),
    (PB.test_block_sparse_attn_random_blocks, (1300, 2, 2, 1, 64)),
    (PB.test_block_sparse_attn_random_blocks, (2000, 2, 1, 300, 256)), (PB.test_block_sparse_attn_degenerate_sets, ()),
    (test_swept_heads_beside_two_pass_heads, (1279,)), (test_swept_heads_beside_two_pass_heads, (1281,)),
    (test_swept_heads_block_lists, (1280, 64)), (test_swept_heads_block_lists, (1333, 128)),
    (test_swept_heads_block_lists, (2100, 256)), (test_swept_segments, (1000, 3, 1)), (test_swept_segments, (1901, 5, 128)),
    (P.test_large_logits_exercise_the_reference_maximum, ("rising",)),
    (P.test_large_logits_exercise_the_reference_maximum, ("falling",)),
    (P.test_large_logits_exercise_the_reference_maximum, ("spiky",))])
def test_uncut_tiles(test, args, monkeypatch):
    """Cases whose point is the tile loop of a whole query tile (where its stretches meet, the
    reference maximum that rises from tile to tile) are small enough to be cut into parts: here
    on workspaces without the room for that, as the long problems run them.  Every call is made
    both ways; the log-sum-exps show that they are two routes."""
    import paper_2406_15486_amd as sa
    calls = []
    for name in ("sa_sparse_attn", "sa_block_sparse_attn", "sa_sparse_attn_chunked", "sa_dense_attn"):
        def both(q, k, v, *a, real=getattr(sa, name), name=name, **kw):
            blocks = name == "sa_block_sparse_attn" or kw.get("granularity", 1) > 1
            path = "dense" if name == "sa_dense_attn" else "blocks" if blocks else "strips"
            kw["want_lse"] = True
            ws = torch.full((_bare(path, q.shape[1], k.shape[1], q.shape[2]),), 0xFF, dtype=torch.uint8, device="cuda")
            cut, uncut = real(q, k, v, *a, **kw), real(q, k, v, *a, workspace=ws, **kw)
            calls.append(not torch.equal(cut[1], uncut[1]))
            return uncut
        monkeypatch.setattr(sa, name, both)
    test(*args)
    assert calls and all(calls)


def _picked(ws, Hq, Hkv, S):
    """What the list kernel of a strip call wrote into the entries of diagonal 0: swept, sparse (core 1) or neither."""
    up, S_pad = (lambda b: (b + 255) // 256 * 256), (S + 255) // 256 * 256
    at = Hkv * 256 * S_pad + Hq * 512 * S_pad + sum(up(Hq * 4 * n) for n in (S_pad, S_pad // 32 + 2, S_pad // 32 + 24))
    first = ws[at:at + Hq * 4 * (S_pad // 64 + 8)].view(torch.int32).view(Hq, -1)[:, 0].cpu().numpy()
    assert (first & 0x3FFFFF == 0).all()
    return ["swept" if e >> 23 & 1 else "sparse" if e >> 22 & 1 else "" for e in first]


# just below and above the lengths and the tiles of a call at which a launch changes core
@pytest.mark.parametrize("path,S,H", [("dense", 4095, 17), ("dense", 4097, 17), ("dense", 4097, 15), ("strips", 49151, 2), ("strips", 49153, 2),
                                      ("strips", 49153, 1), ("strips", 49153, 3), ("blocks", 24575, 3), ("blocks", 24577, 3), ("blocks", 24577, 2)])
def test_cores_of_the_attention_kernels(path, S, H):
    """Uncut tiles take one of the cores, by the length, the query tiles and (strips) the list of the
    head: scattered strips, every other one, nearly full lists that are swept.  With three heads a long
    launch of strips has all three kinds.  Rows around the tiles against their fp64 softmax (probabilities and
    V are bf16, as elsewhere)."""
    import paper_2406_15486_amd as sa
    _say(f"cores {path} S={S} H={H}")
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, h, S, 128, generator=g, device="cuda").bfloat16() for h in (H, 1, 1))
    rng = np.random.default_rng(S)
    blk = 128 if path == "blocks" else 1
    n, w = (S + blk - 1) // blk, 16
    Is = [np.arange(3, n, 613 if blk == 1 else 17), np.arange(0, n, 2), np.sort(rng.choice(n, n * 19 // 20, replace=False))]
    Ic = [np.sort(rng.choice(n, m, replace=False)) for m in (n // 5, n // 40, n * 9 // 10)]
    Ic, Is = ([L[(h + (H == 2)) % 3] for h in range(H)] for L in (Ic, Is))
    lists = []
    for L in (Ic, Is):
        idx = torch.zeros(H, n, dtype=torch.int32)
        for h in range(H):
            idx[h, :len(L[h])] = torch.from_numpy(L[h].astype(np.int32))
        lists += [idx.cuda(), torch.tensor([len(y) for y in L], dtype=torch.int32, device="cuda")]
    kw = dict(out_dtype=sa.SA_OUT_F32, want_lse=True, workspace=torch.full((_bare(path, H, 1, S),), 0xFF, dtype=torch.uint8, device="cuda"))
    if path == "dense":
        out, lse = sa.sa_dense_attn(q, k, v, **kw)
    elif path == "strips":
        out, lse, _ = sa.sa_sparse_attn(q, k, v, *lists, w, **kw)
    else:
        out, lse, _ = sa.sa_block_sparse_attn(q, k, v, *lists, w, blk, **kw)
    torch.cuda.synchronize()
    if (path, S, H) == ("strips", 49153, 3):
        assert _picked(kw["workspace"], H, 1, S) == ["sparse", "", "swept"]
    kk, vv = k[0, 0].double(), v[0, 0].double()
    j = torch.arange(S, device="cuda")
    for h in range(0, H, 1 if H < 4 else 5):
        cols, offs = (torch.zeros(n, dtype=torch.bool, device="cuda") for _ in range(2))
        cols[lists[0][h, :len(Ic[h])].long()] = True
        offs[lists[2][h, :len(Is[h])].long()] = True
        for i in (0, 1, 63, 64, 255, 256, 1000, 2111, S // 2, S - 258, S - 257, S - 2, S - 1):
            d = i - j
            if path == "dense":
                keep = d >= 0
            elif path == "strips":
                keep = (d >= 0) & (cols | offs[d.clamp(min=0)] | (d < w))
            else:      # block diagonals: an offset block b lies on the diagonals b and b + 1, the window on those it reaches
                t = i // blk - j // blk
                diag = torch.zeros(n + 1, dtype=torch.bool, device="cuda")
                diag[:n] |= offs
                diag[1:] |= offs
                diag[:(w + blk - 2) // blk + 1] = True
                keep = (d >= 0) & (cols[j // blk] | diag[t.clamp(min=0)])
            s = (kk @ q[0, h, i].double()) / np.sqrt(128.0)
            s = torch.where(keep, s, torch.tensor(-float("inf"), dtype=torch.float64, device="cuda"))
            assert abs(float(torch.logsumexp(s, 0)) - float(lse[h, i])) < 2e-3, (h, i)
            assert float((torch.softmax(s, 0) @ vv - out[0, h, i].double()).abs().max()) < 2e-2, (h, i)


# segments shorter than a query tile, as long as one, ragged; as many as one launch takes and one more; cut into parts and not
@pytest.mark.parametrize("S,H,C,blk", [(1301, 2, 8, 1), (1301, 2, 9, 1), (768, 1, 3, 1), (2600, 4, 3, 128), (4611, 17, 2, 1), (4611, 16, 4, 64)])
def test_segments_in_one_launch(S, H, C, blk):
    """The segments of a call go through one launch per step where the workspace holds the lists of
    all of them, and one after the other where it does not: the same scores bit for bit, and
    attention to the rounding of the probabilities (other cuts of the tiles, another core)."""
    import paper_2406_15486_amd as sa
    B = sa.binding
    _say(f"segments S={S} C={C} blk={blk}")
    g = torch.Generator(device="cuda").manual_seed(S + C)
    q, k, v = (torch.randn(2, h, S, 128, generator=g, device="cuda").bfloat16() for h in (H, 1, 1))
    sh, n_s = sa.Shape(2, H, 1, S), min(65, S // C)
    one = sa.sa_workspace_bytes(B.SA_OP_SAMPLE_SCORES, sh, n_s, granularity=blk)
    need = sa.sa_workspace_bytes(B.SA_OP_SAMPLE_SCORES, sh, n_s, n_chunks=C, granularity=blk)
    assert (need > one) == (C <= 8)
    scores = [sa.sa_sample_scores(q, k, n_s, granularity=blk, n_chunks=C,
                                  workspace=torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")) for size in (need, one)]
    for a, b in zip(*scores):
        assert torch.equal(a, b)
    lists = sa.sa_select_chunked(*scores[0], 0.8, 0.3, sh, C, blk)
    outs = []
    op = B.SA_OP_SPARSE_ATTN if blk == 1 else B.SA_OP_BLOCK_SPARSE_ATTN
    bare = _bare("strips" if blk == 1 else "blocks", 2 * H, 2, S)
    for size in (sa.sa_workspace_bytes(op, sh, n_chunks=C, granularity=blk), bare):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        outs.append(sa.sa_sparse_attn_chunked(q, k, v, *lists, 5, C, blk, out_dtype=sa.SA_OUT_F32, workspace=ws, want_lse=True, want_tiles=True))
    torch.cuda.synchronize()
    (x, lx, tx), (y, ly, ty) = outs
    assert (x - y).abs().max().item() <= v.abs().max().item() / 256 and (lx - ly).abs().max().item() < 1e-3
    assert torch.isfinite(x).all() and (S != 4611 or torch.equal(tx, ty))


# empty lists leave a query tile the four key tiles that hold its window, for up to six parts
@pytest.mark.parametrize("S,C", [(1281, 1), (1536, 1), (2600, 2), (3300, 3)])
@pytest.mark.parametrize("n_col,n_off", [(0, 0), (1, 0), (0, 1), (65, 2)])
def test_parts_without_tiles(S, C, n_col, n_off):
    """More parts than key tiles in the schedule: the parts left over must add nothing (the
    workspace holds NaN patterns), also in segments that start at a later query tile."""
    import paper_2406_15486_amd as sa
    _say(f"parts without tiles S={S} C={C} {n_col} columns {n_off} offsets")
    _, x = _inputs("glm8k", S=S, Hq=1, Hkv=1, n_sinks=8)
    rng = np.random.default_rng(S + n_col + n_off)
    Ic, Is = ([np.sort(rng.choice(S, n, replace=False)) for _ in range(C)] for n in (n_col, n_off))
    ci, si = (torch.zeros(C, 1, S, dtype=torch.int32) for _ in range(2))
    for m in range(C):
        ci[m, 0, :n_col] = torch.from_numpy(Ic[m].astype(np.int32))
        si[m, 0, :n_off] = torch.from_numpy(Is[m].astype(np.int32))
    cc, sc = (torch.full((C, 1), n, dtype=torch.int32) for n in (n_col, n_off))
    need = sa.sa_workspace_bytes(sa.binding.SA_OP_SPARSE_ATTN, sa.Shape(1, 1, 1, S), n_chunks=C)
    assert need > _bare("strips", 1, 1, S)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    lists = [t.cuda() for t in (ci, cc, si, sc)]
    out, lse, _ = sa.sa_sparse_attn_chunked(*(_dev(x[t]) for t in "qkv"), *lists, 1, C, workspace=ws, want_lse=True)
    torch.cuda.synchronize()
    want, wlse = O.chunked_masked_attn(*(_f64(x[t])[0] for t in "qkv"), Ic, Is, 1, C)
    _check_out(out[0, 0].float().cpu().numpy(), want, "parts without tiles")
    assert np.abs(lse[0].cpu().numpy() - wlse).max() < 2e-3


# dense and swept tiles of one sequence alone (289 query tiles: 32x32x16 MFMAs) and in a batch of three (867: 16x16x32);
# a query's largest logits come first, last, or now and then
@pytest.mark.parametrize("kind", ["random", "rising", "falling", "spiky"])
def test_both_shapes_of_the_mfmas_give_the_same_bits(kind):
    """A score is the same eight products after eight in either shape, and the sums of a row are kept for the
    same groups of keys: outputs and log-sum-exps are equal, whichever a launch takes."""
    import paper_2406_15486_amd as sa
    S, H, w, blk = 4097, 17, 5, 128
    _say(f"shapes of the MFMAs, {kind} logits")
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, h, S, 128, generator=g, device="cuda") for h in (H, 1, 1))
    j = torch.arange(S, device="cuda")
    if kind != "random":
        gain = {"rising": j / S, "falling": 1 - j / S, "spiky": (j % 97 == 5).float()}[kind]
        u = torch.randn(128, generator=g, device="cuda")
        q = q + 4 * u
        k = k + 6 * gain[:, None] * u
    q, k, v = (t.bfloat16() for t in (q, k, v))
    rng = np.random.default_rng(S)
    def lists(n, shares):
        idx, cnt = torch.zeros(H, n, dtype=torch.int32), torch.zeros(H, dtype=torch.int32)
        for h in range(H):
            x = _fill(rng, n, shares[h % len(shares)])
            idx[h, :len(x)], cnt[h] = torch.from_numpy(x.astype(np.int32)), len(x)
        return idx.cuda(), cnt.cuda()
    n = (S + blk - 1) // blk
    strips = (*lists(S, (0.9, 0.97, 0.6)), *lists(S, (0.9, 0.3, 0.97)))      # nearly full: swept
    blocks = (*lists(n, (0.9, 1.0, 0.7)), *lists(n, (0.9, 0.5, 1.0)))
    def run(B):
        qq, kk, vv = (t.repeat(B, 1, 1, 1) for t in (q, k, v))
        kw = dict(out_dtype=sa.SA_OUT_F32, want_lse=True)
        return (sa.sa_dense_attn(qq, kk, vv, **kw), sa.sa_sparse_attn(qq, kk, vv, *(t.repeat(B, *[1] * (t.dim() - 1)) for t in strips), w, want_tiles=True, **kw),
                sa.sa_block_sparse_attn(qq, kk, vv, *(t.repeat(B, *[1] * (t.dim() - 1)) for t in blocks), w, blk, **kw))
    one, three = run(1), run(3)
    torch.cuda.synchronize()
    last = np.minimum(256 * np.arange(17) + 255, S - 1)
    rows = 256 * np.arange(17)[:, None] + 32 * np.arange(8)[None, :] + 31
    assert (one[1][2] == int(np.minimum(last[:, None] // 64 + 1, rows // 64 + 1).sum())).all()          # every head is swept
    for a, b in zip(one, three):
        assert torch.isfinite(a[0]).all() and torch.isfinite(a[1]).all()
        for x in range(3):
            assert torch.equal(a[0][0], b[0][x]) and torch.equal(a[1], b[1].view(3, H, S)[x])
    # rows of the dense call against their fp64 softmax (bf16 probabilities and V, as elsewhere)
    for h in (0, 7, 16):
        for i in (0, 31, 64, 300, 2111, S - 2, S - 1):
            s = (k[0, 0, :i + 1].double() @ q[0, h, i].double()) / np.sqrt(128.0)
            assert abs(float(torch.logsumexp(s, 0)) - float(one[0][1].view(H, S)[h, i])) < 2e-3, (h, i)
            assert float((torch.softmax(s, 0) @ v[0, 0, :i + 1].double() - one[0][0][0, h, i].double()).abs().max()) < 2e-2, (h, i)


def test_core_of_heads_in_two_passes():
    """In long calls the list kernel picks the core of a head by its lists: what it wrote into the entry of
    diagonal 0.  Isolated offsets (with or without some columns) leave most waves of their tiles without work; columns
    alone and wide bands of offsets do not."""
    import paper_2406_15486_amd as sa
    S, w = 49153, 16
    _say("core of heads in two passes")
    a = np.arange(S)
    def share(f):
        return a[::int(1 / f)]
    def runs(r, p):
        return a[a % p < r]
    none = a[:0]
    cases = [(none, runs(1, 1000), "sparse"), (none, runs(4, 300), "sparse"), (share(0.05), runs(1, 8000), "sparse"), (share(0.1), runs(4, 1000), "sparse"),
             (none, runs(2000, 4000), ""), (share(0.2), none, ""), (share(0.9), runs(1, 2), "swept"), (none, none, "sparse")]
    H = len(cases)
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = (torch.randn(1, h, S, 128, generator=g, device="cuda").bfloat16() for h in (H, 1, 1))
    lists = []
    for t in range(2):
        idx = torch.zeros(H, S, dtype=torch.int32)
        for h in range(H):
            idx[h, :len(cases[h][t])] = torch.from_numpy(cases[h][t].astype(np.int32))
        lists += [idx.cuda(), torch.tensor([len(c[t]) for c in cases], dtype=torch.int32, device="cuda")]
    ws = torch.full((_bare("strips", H, 1, S),), 0xFF, dtype=torch.uint8, device="cuda")
    sa.sa_sparse_attn(q, k, v, *lists, w, workspace=ws)
    torch.cuda.synchronize()
    assert _picked(ws, H, 1, S) == [c[2] for c in cases]


@pytest.mark.parametrize("path", ["strips", "blocks"])
@pytest.mark.parametrize("kind", ["random", "rising", "falling", "spiky"])
def test_heads_in_two_passes_of_long_calls(path, kind):
    """The tile loop of core 0 on gathered and range tiles (the small cases run on core 1): column counts that put the
    boundaries of its stretches at the first, a middle and the last iteration, and logits whose
    maximum keeps rising, is met at once, or comes in isolated keys.  Rows against their fp64 softmax."""
    import paper_2406_15486_amd as sa
    _say(f"two passes of long calls, {path}, {kind} logits")
    blk, S, w = (1, 49153, 16) if path == "strips" else (128, 24577, 16)
    counts = [0, 1, 64, 65, 255, 257, 320, 321, 384, 640] if blk == 1 else [0, 1, 2, 3, 5, 12]
    H, n = len(counts), (S + blk - 1) // blk
    g = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(1, h, S, 128, generator=g, device="cuda") for h in (H, 1, 1))
    j = torch.arange(S, device="cuda")
    if kind != "random":
        u = torch.randn(128, generator=g, device="cuda")
        u = u / u.norm()
        q = q + 6 * u
        # (40 logits over the sequence, and 40 above the rest)
        k = k + (75 * (torch.rand(S, generator=g, device="cuda") < 1e-3) if kind == "spiky" else 75 * (j / S if kind == "rising" else 1 - j / S))[:, None] * u
    q, k, v = (t.bfloat16() for t in (q, k, v))
    rng = np.random.default_rng(S)
    Ic = [np.sort(rng.choice(n, c, replace=False)) for c in counts]
    Ic[3] = np.arange(counts[3])                              # the first keys: every query tile sees all of them
    Ic[-2] = np.arange(n - counts[-2], n)                     # the last keys: only the last tiles do
    a = np.arange(n)
    Is = [a[(a + 97 * h) % (4000 if blk == 1 else 24) < (2000 if blk == 1 else 1 + h % 3)] for h in range(H)]
    lists = []
    for L in (Ic, Is):
        idx = torch.zeros(H, n, dtype=torch.int32)
        for h in range(H):
            idx[h, :len(L[h])] = torch.from_numpy(L[h].astype(np.int32))
        lists += [idx.cuda(), torch.tensor([len(y) for y in L], dtype=torch.int32, device="cuda")]
    ws = torch.full((_bare(path, H, 1, S),), 0xFF, dtype=torch.uint8, device="cuda")
    kw = dict(out_dtype=sa.SA_OUT_F32, want_lse=True, workspace=ws)
    if blk == 1:
        out, lse, _ = sa.sa_sparse_attn(q, k, v, *lists, w, **kw)
    else:
        out, lse, _ = sa.sa_block_sparse_attn(q, k, v, *lists, w, blk, **kw)
    torch.cuda.synchronize()
    if blk == 1:
        assert _picked(ws, H, 1, S) == [""] * H
    kk, vv = k[0, 0].double(), v[0, 0].double()
    for h in range(H):
        cols, offs = (torch.zeros(n, dtype=torch.bool, device="cuda") for _ in range(2))
        cols[lists[0][h, :len(Ic[h])].long()] = True
        offs[lists[2][h, :len(Is[h])].long()] = True
        diag = torch.zeros(n + 1, dtype=torch.bool, device="cuda")
        diag[:n] |= offs
        diag[1:] |= offs
        diag[:(w + blk - 2) // blk + 1] = True
        for i in (0, 31, 64, 255, 256, 1000, 4500, S // 2, S - 322, S - 258, S - 257, S - 65, S - 2, S - 1):
            d = i - j
            if blk == 1:
                keep = (d >= 0) & (cols | offs[d.clamp(min=0)] | (d < w))
            else:
                keep = (d >= 0) & (cols[j // blk] | diag[(i // blk - j // blk).clamp(min=0)])
            x = (kk @ q[0, h, i].double()) / np.sqrt(128.0)
            x = torch.where(keep, x, torch.tensor(-float("inf"), dtype=torch.float64, device="cuda"))
            want = float(torch.logsumexp(x, 0))
            assert abs(want - float(lse[h, i])) < 2e-3 * max(1.0, abs(want) / 10), (h, i)
            assert float((torch.softmax(x, 0) @ vv - out[0, h, i].double()).abs().max()) < 2e-2, (h, i)
