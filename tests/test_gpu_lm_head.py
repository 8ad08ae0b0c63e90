"""GPU parity of lm_head_argmax (teacher head + greedy choice, logits never materialised) against the fp64 oracle.

The argmax is an integer decided by floating point: the kernel accumulates bf16 products in fp32, the oracle in
fp64.  So the index is compared exactly wherever the oracle's two best logits differ by more than the accumulation
error bound, and elsewhere the kernel's choice must be one of the near-maximal entries; exact ties (duplicated weight
rows give bit-identical logits on both sides) must resolve to the lowest index; planted winners must be found."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_08088_amd import api, synth
from gpu_helpers import bits_of, to_dev

pytestmark = pytest.mark.gpu


def _bf16(x):
    return synth.f32_to_bf16_bits(np.asarray(x, dtype=np.float32))


def _dev_bf16(bits):
    return to_dev(bits).view(torch.bfloat16) if bits.dtype == np.uint16 else to_dev(bits)


def _check(h_bits, w_bits, n, exact=None):
    B, T, D = h_bits.shape
    ref = oracle.lm_head_argmax(h_bits, w_bits, n, dtype="bf16", want_logits=True)
    dh, dw, dn = _dev_bf16(h_bits), _dev_bf16(w_bits), to_dev(np.asarray(n, dtype=np.int32))
    got = api.lm_head_argmax(dh, dw, dn)
    # the same weights packed into tiles: same arithmetic in the same order, so the same bits
    packed = api.pack_lm_head(dw)
    got2 = api.lm_head_argmax(dh, packed, dn, V=w_bits.shape[0])
    torch.cuda.synchronize()
    assert torch.equal(got["argmax"], got2["argmax"]) and torch.equal(got["maxval"], got2["maxval"])
    g, gmax = bits_of(got["argmax"]), bits_of(got["maxval"]).astype(np.float64)
    hf = synth.bf16_bits_to_f32(h_bits).astype(np.float64)
    wf = synth.bf16_bits_to_f32(w_bits).astype(np.float64)
    for b in range(B):
        nb = int(np.clip(n[b], 0, T))
        assert np.all(g[b, nb:] == -1) and np.all(np.isneginf(gmax[b, nb:]))
        for k in range(nb):
            lg = ref["logits"][b, k]
            # fp32 accumulation of D exact products: |error| <= D * 2^-24 * sum |h_c w_vc| for any order
            bound = D * 2.0 ** -24 * float(np.abs(hf[b, k]) @ np.abs(wf[int(g[b, k])])) + 1e-30
            assert 0 <= g[b, k] < w_bits.shape[0]
            assert abs(gmax[b, k] - lg[g[b, k]]) <= bound, (b, k, gmax[b, k], lg[g[b, k]], bound)
            order = np.argsort(-lg, kind="stable")
            margin = lg[order[0]] - lg[order[1]] if len(order) > 1 else np.inf
            if margin > 2 * bound:
                assert g[b, k] == ref["argmax"][b, k], (b, k, margin, bound)
            else:
                assert lg[g[b, k]] >= lg[order[0]] - 2 * bound
    if exact is not None:
        assert np.array_equal(g, exact)
    return ref, g


@pytest.mark.parametrize("B,T,D,V", [(1, 1, 128, 1), (1, 7, 128, 100), (2, 15, 128, 128), (1, 60, 256, 129),
                                      (2, 33, 384, 1000), (3, 60, 128, 700), (1, 128, 128, 513), (2, 128, 256, 300),
                                      (5, 64, 128, 257), (1, 64, 128, 200), (1, 65, 256, 190), (1, 129, 128, 64),
                                      (1, 256, 128, 450)])
def test_random_inputs_all_shapes(B, T, D, V):
    rng = np.random.default_rng(3000 + B * 1000 + T + D + V)
    h = _bf16(rng.standard_normal((B, T, D)))
    w = _bf16(rng.standard_normal((V, D)) / np.sqrt(D))
    n = [T] + [int(rng.integers(0, T + 1)) for _ in range(B - 1)]
    _check(h, w, n)


def test_random_row_counts_and_vocabularies_on_the_wide_path():
    """Seeded sweep over the shapes that exercise the 128-row workgroups: last row groups of 1..127 rows, padded
    sequences, vocabularies that end inside the first or the second half of a tile, one and several tiles."""
    rng = np.random.default_rng(3050)
    for case in range(14):
        B = int(rng.integers(1, 4))
        T = int(rng.integers(max(1, 65 // B), 140))
        D = 128 * int(rng.integers(1, 4))
        V = int(rng.choice([1, 33, 64, 65, 127, 128, 129, 191, 192, 193, 255, 300, 641]))
        h = _bf16(rng.standard_normal((B, T, D)))
        w = _bf16(rng.standard_normal((V, D)) / np.sqrt(D))
        n = [T] + [int(rng.integers(0, T + 1)) for _ in range(B - 1)]
        assert B * T > 64
        _check(h, w, n)


def _gemm_runs(B, T, V):
    """The head's choice: the GEMM tiling (256 vocabulary rows x 256 node rows per workgroup) where it needs less than half the
    rounds of 256 workgroups that the 128-row groups need."""
    tiles, rows = (V + 127) // 128, B * T
    wide, gemm = (-(-t * -(-rows // r) // 256) for t, r in ((tiles, 128), ((tiles + 1) // 2, 256)))
    return rows > 128 and 2 * gemm < wide


def test_random_row_counts_and_vocabularies_beyond_256_rows():
    """More than 256 node rows over a small vocabulary, which stay on the 128-row groups: row counts that end inside the
    first, second, third or fourth 32-row block of the last group, padded sequences, vocabularies that end inside the first
    or the second half of a tile, one and several tiles, contraction lengths of one to three packed steps."""
    rng = np.random.default_rng(3060)
    shapes = [(4, 128, 128, 513), (3, 200, 256, 300), (9, 100, 128, 129), (32, 33, 384, 1000), (2, 256, 128, 256),
              (5, 103, 256, 127), (8, 65, 128, 770), (1, 600, 128, 1), (6, 97, 384, 385), (1, 257, 128, 300),
              (8, 60, 256, 641), (3, 111, 128, 64)]
    for (B, T, D, V) in shapes:
        assert B * T > 256 and not _gemm_runs(B, T, V)
        h = _bf16(rng.standard_normal((B, T, D)))
        w = _bf16(rng.standard_normal((V, D)) / np.sqrt(D))
        n = [T] + [int(rng.integers(0, T + 1)) for _ in range(B - 1)]
        _check(h, w, n)


@pytest.mark.parametrize("B,T,D,V", [(32, 125, 128, 2177), (31, 129, 384, 2304), (10, 100, 128, 8225), (3, 100, 256, 21889), (1, 257, 128, 22017),
                                      (17, 241, 128, 2200)])
def test_gemm_tiling_where_it_saves_rounds(B, T, D, V):
    """The GEMM tiling runs where it needs less than half the rounds of workgroups: vocabularies that end inside the first and
    the second half of a 256-row tile, last row groups of 1 ... 256 rows, several panels of tiles and groups per XCD."""
    assert _gemm_runs(B, T, V)
    rng = np.random.default_rng(3070 + V)
    h = _bf16(rng.standard_normal((B, T, D)))
    w = _bf16(rng.standard_normal((V, D)) / np.sqrt(D))
    _check(h, w, [T] + [int(rng.integers(0, T + 1)) for _ in range(B - 1)])


@pytest.mark.parametrize("B,T,V,gemm", [(5, 128, 900, False), (32, 125, 2177, True)])
def test_exact_ties_beyond_256_rows_take_the_lowest_index(B, T, V, gemm):
    rng = np.random.default_rng(3110)
    D = 128
    assert _gemm_runs(B, T, V) == gemm
    hb = _bf16(rng.standard_normal((B, T, D)))
    wb = _bf16(rng.standard_normal((V, D)) / np.sqrt(D))
    hf = synth.bf16_bits_to_f32(hb)
    # node (2, 77): a clear winner duplicated in another 256-row tile, in the other 128-row half of its tile, in
    # another 32-row block of its half and in the last (partial) tile
    win = _bf16(8.0 * hf[2, 77] / float(hf[2, 77] @ hf[2, 77]))
    for v in (300, 37, 310, 420, 899, V - 1):
        wb[v] = win
    for gone, lowest in (((), 37), ((37,), 300), ((300, 310), 420)):
        for v in gone:
            wb[v] = _bf16(rng.standard_normal(D) / np.sqrt(D))
        ref, g = _check(hb, wb, [T] * B)
        assert g[2, 77] == lowest and ref["argmax"][2, 77] == lowest


def test_unsupported_width_is_rejected():
    h = torch.zeros((1, 4, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((10, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(api.EtvError):
        api.lm_head_argmax(h, w, torch.ones(1, dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("T", [40, 100])     # 100 rows: the 128-row workgroups that take a tile in two passes
def test_exact_ties_take_the_lowest_index_within_and_across_tiles(T):
    rng = np.random.default_rng(3100)
    B, D, V = 1, 128, 600
    h = rng.standard_normal((B, T, D)).astype(np.float32)
    w = (rng.standard_normal((V, D)) / np.sqrt(D)).astype(np.float32)
    hb = _bf16(h)
    wb = _bf16(w)
    hf = synth.bf16_bits_to_f32(hb)
    # make row 300 a clear winner for node 0 and duplicate it at 37 (another tile), 310 (same tile, same 32-block),
    # 350 (same tile, other block; the other half of the tile) and 599 (last tile): bit-identical logits, the
    # lowest index must win
    win = _bf16(8.0 * hf[0, 0] / float(hf[0, 0] @ hf[0, 0]))
    for v in (300, 37, 310, 350, 599):
        wb[v] = win
    ref, g = _check(hb, wb, [T])
    assert g[0, 0] == 37 and ref["argmax"][0, 0] == 37
    # and with the duplicates only above 300
    wb[37] = _bf16(w[37])
    ref, g = _check(hb, wb, [T])
    assert g[0, 0] == 300


def test_planted_winners_at_verify_step_size():
    rng = np.random.default_rng(3200)
    for (B, T, D, V) in ((1, 60, 1024, 32000), (1, 60, 4096, 2048), (2, 60, 512, 4000), (1, 128, 1024, 8000)):
        h = rng.standard_normal((B, T, D)).astype(np.float32)
        w = (rng.standard_normal((V, D)) / np.sqrt(D)).astype(np.float32)
        hb = _bf16(h)
        hf = synth.bf16_bits_to_f32(hb).astype(np.float64)
        target = rng.permutation(V)[: B * T].reshape(B, T)
        for b in range(B):
            for k in range(T):
                w[target[b, k]] = (12.0 * hf[b, k] / (hf[b, k] @ hf[b, k])).astype(np.float32)
        _check(hb, _bf16(w), [T] * B, exact=target.astype(np.int32))


def test_head_to_commit_without_logits():
    """hidden states -> lm_head_argmax -> the fused epilogue taking the per-node choice in place of logits: the
    acceptance and the commit equal the oracle's, which is given logits whose row argmax is the oracle head's."""
    from gpu_helpers import DevWorkload
    from helpers import logits_from_argmax
    rng = np.random.default_rng(3300)
    wl = synth.config2(P=300, with_logits=False)
    B, T, D, V = wl.B, wl.T_max, 512, wl.V
    h = rng.standard_normal((B, T, D)).astype(np.float32)
    w = (rng.standard_normal((V, D)) / np.sqrt(D)).astype(np.float32)
    hb = _bf16(h)
    hf = synth.bf16_bits_to_f32(hb).astype(np.float64)
    # the teacher agrees with the draft along one root-to-leaf path for three steps, then picks something else
    path = [int(x) for x in wl.retrieve[0, 5] if x >= 0]
    plant = {path[i]: int(wl.tokens[0, path[i + 1]]) for i in range(min(3, len(path) - 1))}
    free = [int(x) for x in rng.permutation(V) if int(x) not in set(plant.values())]
    for node in range(T):
        v = plant.get(node, free[node])      # distinct rows, so every node keeps its planted winner
        w[v] = (12.0 * hf[0, node] / (hf[0, node] @ hf[0, node])).astype(np.float32)
    wb = _bf16(w)
    ref_head = oracle.lm_head_argmax(hb, wb, wl.n_nodes, dtype="bf16")
    lg = np.stack([logits_from_argmax(rng, ref_head["argmax"][b].clip(0), V) for b in range(B)])
    rp = oracle.evaluate_posterior(lg, wl.tokens, wl.retrieve, wl.n_nodes)
    kc, vc = wl.k_cache[None].copy(), wl.v_cache[None].copy()
    rc = oracle.commit_accepted_kv(wl.kt[None], wl.vt[None], kc, vc, wl.prefix_len, wl.capacity, wl.n_nodes,
                                   rp["acc_nodes"], rp["accept_len"], block_table=wl.block_table)
    assert rp["accept_len"][0] >= 1

    d = DevWorkload(wl)
    head = api.lm_head_argmax(_dev_bf16(hb), api.pack_lm_head(_dev_bf16(wb)), d.n_nodes, V=V)
    dkc, dvc = d.k_cache[None].clone(), d.v_cache[None].clone()
    g, p, c = api.verify_epilogue(None, d.tokens, d.retrieve, d.n_nodes, d.kt[None], d.vt[None], dkc, dvc,
                                  d.prefix_len, d.capacity, block_table=d.block_table,
                                  post_out=dict(argmax=head["argmax"]))
    p2 = api.evaluate_posterior(None, d.tokens, d.retrieve, d.n_nodes, out=dict(argmax=head["argmax"]))
    # third way: the head stops after its weight pass and the epilogue finishes the choice per node itself
    part = api.lm_head_argmax(_dev_bf16(hb), _dev_bf16(wb), d.n_nodes, finish=False)
    dkc3, dvc3 = d.k_cache[None].clone(), d.v_cache[None].clone()
    g3, p3, c3 = api.verify_epilogue(None, d.tokens, d.retrieve, d.n_nodes, d.kt[None], d.vt[None], dkc3, dvc3,
                                     d.prefix_len, d.capacity, block_table=d.block_table,
                                     workspace=part["workspace"], head_V=V)
    p4 = api.evaluate_posterior(None, d.tokens, d.retrieve, d.n_nodes, workspace=part["workspace"], head_V=V)
    torch.cuda.synchronize()
    assert np.array_equal(bits_of(p3["argmax"])[0, :int(wl.n_nodes[0])], ref_head["argmax"][0, :int(wl.n_nodes[0])])
    assert np.all(bits_of(p3["argmax"])[0, int(wl.n_nodes[0]):] == -1)
    for key in ("len", "best", "accept_len", "acc_nodes", "bonus"):
        assert np.array_equal(bits_of(p3[key]), rp[key]) and np.array_equal(bits_of(p4[key]), rp[key]), key
    for key in rc:
        assert np.array_equal(bits_of(c3[key]), rc[key]), key
    assert np.array_equal(bits_of(dkc3), kc) and np.array_equal(bits_of(dvc3), vc)
    n = int(wl.n_nodes[0])
    assert np.array_equal(bits_of(head["argmax"])[0, :n], ref_head["argmax"][0, :n])
    for key in ("len", "best", "accept_len", "acc_nodes", "bonus"):
        assert np.array_equal(bits_of(p[key]), rp[key]), key
        assert np.array_equal(bits_of(p2[key]), rp[key]), key
    for key in rc:
        assert np.array_equal(bits_of(c[key]), rc[key]), key
    assert np.array_equal(bits_of(dkc), kc) and np.array_equal(bits_of(dvc), vc)


@pytest.mark.parametrize("T", [12, 13, 70])
@pytest.mark.parametrize("V", [2048, 2049, 8200, 32768, 32769, 70000])
def test_partials_of_the_head_are_finished_inline_or_by_a_launch(T, V):
    """The choice per node out of the head's per-tile maxima, on both sides of the rule that picks where they are reduced
    (nodes per tree, partials per node) and of the 256 partials that a wavefront reads per trip to memory: hand-made partials
    with ties, against numpy and the oracle's acceptance."""
    from helpers import logits_from_argmax, random_tree
    rng = np.random.default_rng(100 * T + V)
    B, tiles = 3, (V + 127) // 128
    n = [T, 1, max(1, T - 5)]
    parents = [random_tree(rng, x) for x in n]
    wl = synth.assemble("partials", rng, parents, [40] * B, Hq=2, Hkv=2, d=64, dtype="bf16", V=V, W=T, paged=False, T_max=T,
                        with_logits=False)
    pval = rng.integers(0, 9, size=(B, T, tiles)).astype(np.float32)            # few distinct values: ties across tiles
    pidx = np.minimum(np.arange(tiles) * 128 + rng.integers(0, 128, size=(B, T, tiles)), V - 1).astype(np.int32)
    want = np.take_along_axis(pidx, pval.argmax(axis=2)[..., None], axis=2)[..., 0]   # first maximum = lowest index
    lg = np.stack([logits_from_argmax(rng, want[b], V) for b in range(B)])
    rp = oracle.evaluate_posterior(lg, wl.tokens, wl.retrieve, wl.n_nodes)
    ws = torch.cat([to_dev(pval).reshape(-1).view(torch.uint8), to_dev(pidx).reshape(-1).view(torch.uint8)])
    tok, ret, dn = to_dev(wl.tokens), to_dev(wl.retrieve), to_dev(wl.n_nodes)
    p = api.evaluate_posterior(None, tok, ret, dn, workspace=ws, head_V=V)
    kt, vt, kc, vc = (to_dev(x)[None].clone() for x in (wl.kt, wl.vt, wl.k_cache, wl.v_cache))
    _, q, _ = api.verify_epilogue(None, tok, ret, dn, kt, vt, kc, vc, to_dev(wl.prefix_len), to_dev(wl.capacity),
                                  workspace=ws, head_V=V)
    torch.cuda.synchronize()
    for key in rp:
        assert np.array_equal(bits_of(p[key]), rp[key]) and np.array_equal(bits_of(q[key]), rp[key]), key


@pytest.mark.parametrize("T", [12, 13])
@pytest.mark.parametrize("V", [65536, 65541, 70000])
def test_partials_of_the_logits_are_finished_inline_or_by_a_launch(T, V):
    """Vocabularies around 16 chunks of the logit scan: beyond them the choice per node is finished by a launch of its own from 13
    nodes on.  Ties within a chunk and across chunks; against the oracle."""
    rng = np.random.default_rng(T + V)
    B, n = 2, [T, T - 4]
    from helpers import random_tree
    wl = synth.assemble("logits", rng, [random_tree(rng, x) for x in n], [40] * B, Hq=2, Hkv=2, d=64, dtype="bf16", V=V, W=T, paged=False,
                        T_max=T, with_logits=False)
    lg = rng.integers(0, 4, size=(B, T, V)).astype(np.float32)         # ties everywhere
    for b in range(B):
        for k in range(T):
            lg[b, k, rng.integers(0, V, size=3)] = 9.0                 # three of the largest, in any chunks
        for p in wl.retrieve[b]:                                       # and the children's tokens now and then, so that paths are accepted
            for x, y in zip(p[:-1], p[1:]):
                if 0 <= x and 0 <= y and rng.random() < 0.5:
                    lg[b, x, wl.tokens[b, y]] = 10.0
    rp = oracle.evaluate_posterior(lg, wl.tokens, wl.retrieve, wl.n_nodes)
    tok, ret, dn, dl = to_dev(wl.tokens), to_dev(wl.retrieve), to_dev(wl.n_nodes), to_dev(lg)
    p = api.evaluate_posterior(dl, tok, ret, dn)
    kt, vt, kc, vc = (to_dev(x)[None].clone() for x in (wl.kt, wl.vt, wl.k_cache, wl.v_cache))
    _, q, _ = api.verify_epilogue(dl, tok, ret, dn, kt, vt, kc, vc, to_dev(wl.prefix_len), to_dev(wl.capacity))
    torch.cuda.synchronize()
    for key in rp:
        assert np.array_equal(bits_of(p[key]), rp[key]) and np.array_equal(bits_of(q[key]), rp[key]), key
