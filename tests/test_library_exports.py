"""CPU-side checks of the boundary: the built library loads and exports every symbol the header declares."""
import ctypes
import os
import re

import numpy as np
import pytest
import torch

from paper_2603_08088_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols(header="eagletv.h", prefix="etv_"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(" + prefix + r"[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported_and_binding_lists_them_all():
    syms = _declared_symbols()
    assert len(syms) >= 10
    assert os.path.exists(api.LIB_PATH), "build the library first: python -m paper_2603_08088_amd.build"
    lib = ctypes.CDLL(api.LIB_PATH)
    for s in syms:
        assert hasattr(lib, s), s
    assert sorted(api.EXPORTS) == syms


def test_probe_library_exports_its_header_and_the_product_library_holds_no_probe():
    from paper_2603_08088_amd import probe
    syms = _declared_symbols("eagletv_probe.h", "etvp_")
    assert sorted(probe.EXPORTS) == syms and len(syms) == 5
    lib = ctypes.CDLL(probe.LIB_PATH)
    for s in syms:
        assert hasattr(lib, s), s
    assert probe.mfma_bf16_probe_flops(1) == 2048 * 4 * 16 * 2 * 32 * 32 * 16
    product = ctypes.CDLL(api.LIB_PATH)
    assert not hasattr(product, "etv_hbm_read_probe") and not hasattr(product, "etvp_hbm_read_probe")


def test_host_only_calls_need_no_gpu():
    lib = api.lib()
    assert b"gfx950" in lib.etv_version()
    assert lib.etv_status_string(0) == b"ok" and lib.etv_status_string(-3) == b"workspace too small"
    assert lib.etv_status_string(-5) == b"not implemented"
    # a replica of a contiguous cache is a defined operation that is not built: refused on the host, before any pointer is used
    cd = api.CacheDesc(B=1, Hkv=2, d=64, elem_bytes=2, n_layers=1, block_size=0, max_blocks=0, num_blocks=0, P_cap=64,
                       reserved=0, cache_layer_stride=64 * 2 * 64)
    assert lib.etv_replicate_branches(ctypes.byref(cd), None, None, None, None, None, 1, None, 0, None, None, None, None,
                                      None) == -5
    dsc = api.AttnDesc(B=1, T_max=60, Hq=32, Hkv=8, d=128, dtype=api.BF16, block_size=0, max_blocks=0, num_blocks=0,
                       P_cap=2100, P_max=2048, scale=0.0, kv_split=0, flags=0)
    ws = api.tree_verify_attention_workspace_bytes(dsc)
    assert ws >= 256
    dsc.kv_split = 64
    assert api.tree_verify_attention_workspace_bytes(dsc) >= 1 * 32 * 60 * 32 * 130 * 4
    assert api.evaluate_posterior_workspace_bytes(1, 60, 32000) == 60 * 8 * 8


def test_launch_plan_is_reported_and_follows_the_tuning_flags():
    """Host-only: the plan call shows what the cost model picks, and kv_split / the flags override it."""
    def desc(B, T, P, paged, **kw):
        return api.AttnDesc(B=B, T_max=T, Hq=32, Hkv=8, d=128, dtype=api.BF16, block_size=16 if paged else 0,
                            max_blocks=(P + T + 15) // 16 + 1, num_blocks=0, P_cap=P + T, P_max=P, scale=0.0,
                            kv_split=kw.get("kv_split", 0), flags=kw.get("flags", 0))
    big = api.tree_verify_attention_plan(desc(32, 128, 4096, True))
    assert big["mfma"] == 1 and big["n_splits"] == 1 and big["kv_split"] == 4096 and big["workgroups"] == 32 * 8 * big["row_groups"]
    assert big["wavefronts"] * (1 if not big["key_halves"] else 0.5) * big["row_groups"] >= 16      # 16 chunks of 32 rows
    c2 = api.tree_verify_attention_plan(desc(1, 60, 2048, False))
    assert c2["n_splits"] > 1 and c2["kv_split"] % 64 == 0 and c2["kv_split"] * c2["n_splits"] >= 2048
    forced = api.tree_verify_attention_plan(desc(1, 60, 2048, False, kv_split=512, flags=api.ATTN_FLAG_WHOLE_TILE | api.ATTN_FLAG_SMALL_WG))
    assert forced["kv_split"] == 512 and forced["n_splits"] == 4 and forced["key_halves"] == 0 and forced["wavefronts"] == 4
    large = api.tree_verify_attention_plan(desc(1, 60, 2048, False, flags=api.ATTN_FLAG_LARGE_WG | api.ATTN_FLAG_WHOLE_TILE))
    assert large["wavefronts"] == 8 and large["key_halves"] == 0
    # split slots follow the sequences' lengths for batches of 2 .. 64 sequences, unless the flag keeps one split size
    assert big["balanced_splits"] == 0 and c2["balanced_splits"] == 0             # no splits / one sequence
    ragged = api.tree_verify_attention_plan(desc(8, 60, 8192, True))
    assert ragged["n_splits"] > 1 and ragged["balanced_splits"] == 1
    assert ragged["workgroups"] == 8 * ragged["n_splits"] * 8 * ragged["row_groups"]
    kept = api.tree_verify_attention_plan(desc(8, 60, 8192, True, flags=api.ATTN_FLAG_UNIFORM_SPLITS))
    assert kept["balanced_splits"] == 0 and kept["n_splits"] == ragged["n_splits"]
    assert api.tree_verify_attention_plan(desc(65, 12, 8192, True, kv_split=1024))["balanced_splits"] == 0
    ws = api.tree_verify_attention_workspace_bytes(desc(8, 60, 8192, True))
    assert ws >= 8 * ragged["n_splits"] * 32 * 60 * 130 * 4 + 64 * 8                  # partials + the split table
    f32 = api.AttnDesc(B=1, T_max=15, Hq=4, Hkv=4, d=64, dtype=api.F32, block_size=0, max_blocks=0, num_blocks=0,
                       P_cap=200, P_max=128, scale=0.0, kv_split=0, flags=0)
    assert api.tree_verify_attention_plan(f32)["mfma"] == 0


def test_the_kernel_of_a_plan_is_reported():
    """Host only: each kernel by a call that takes it on its own, and by the flag that asks for it."""

    def kernel(flags=0, **kw):
        c = dict(dict(B=32, T_max=128, Hq=32, Hkv=8, d=128, dtype=api.BF16, P_cap=4096, P_max=4096, flags=flags), **kw)
        return api.tree_verify_attention_kernel(api.AttnDesc(**c))
    assert kernel() == "wide"                                           # many rows, long splits
    assert kernel(B=1, T_max=60, P_max=2048) == "key_blocks"            # a launch that fits the chip at once
    assert kernel(T_max=16) == "tile"
    assert kernel(dtype=api.F32, d=64) == kernel(dtype=api.F32) == "f32"
    assert kernel(scale=-1.0) == kernel(flags=api.ATTN_FLAG_GENERIC) == kernel(dtype=api.F32, flags=api.ATTN_FLAG_GENERIC) == "generic"
    assert kernel(flags=api.ATTN_FLAG_KEY_BLOCKS) == kernel(d=64, flags=api.ATTN_FLAG_KEY_BLOCKS) == "key_blocks"
    assert kernel(d=64) == "tile"
    for T in (1, 33, 64, 65, 256):
        for P in (0, 1, 900, 4096):
            assert kernel(T_max=T, P_max=P, flags=api.ATTN_FLAG_WIDE) == "wide", (T, P)
    # more than 128 nodes cost the wide kernel a second pass: over short splits the tile kernel is faster (99 and 81 us, 52 and 41)
    assert kernel(B=23, T_max=199, Hq=32, Hkv=32, P_max=377) == "tile" and kernel(B=12, T_max=169, P_max=428) == "tile"
    assert kernel(T_max=256) == "wide"
    # a flag for a shape of the tile kernel names that kernel, and the wide one's goes before it
    for flags in (api.ATTN_FLAG_SMALL_WG, api.ATTN_FLAG_LARGE_WG, api.ATTN_FLAG_WHOLE_TILE, api.ATTN_FLAG_KEY_HALVES,
                  api.ATTN_FLAG_LARGE_WG | api.ATTN_FLAG_WHOLE_TILE, api.ATTN_FLAG_LARGE_WG | api.ATTN_FLAG_KEY_HALVES,
                  api.ATTN_FLAG_WHOLE_TILE | api.ATTN_FLAG_KEY_HALVES):
        for kw in (dict(), dict(T_max=32), dict(B=2, T_max=32, Hq=8, Hkv=2, P_max=300, kv_split=4096), dict(B=1, P_max=32768), dict(T_max=8)):
            assert kernel(flags=flags, **kw) == "tile", (flags, kw)
            assert kernel(flags=flags | api.ATTN_FLAG_WIDE, **kw) == "wide", (flags, kw)
    # heads of 64 and fp32 have no wide kernel, and its flag changes nothing for them
    for kw in (dict(d=64), dict(d=64, B=1, T_max=60, P_max=2048), dict(d=64, B=4, T_max=48, P_max=1500), dict(dtype=api.F32)):
        c = dict(dict(B=32, T_max=128, Hq=32, Hkv=8, d=128, dtype=api.BF16, P_cap=4096, P_max=4096), **kw)
        plain, wide = api.AttnDesc(**c), api.AttnDesc(**c, flags=api.ATTN_FLAG_WIDE)
        assert api.tree_verify_attention_plan(plain) == api.tree_verify_attention_plan(wide)
    with pytest.raises(api.EtvError):
        kernel(Hq=9)


def test_struct_layouts_match_the_header():
    assert ctypes.sizeof(api.AttnDesc) == 14 * 4
    assert ctypes.sizeof(api.AttnPlan) == 8 * 4 + 8
    assert ctypes.sizeof(api.CommitDesc) == 12 * 4 + 8


@pytest.mark.parametrize("layers", [1, 3])
def test_commit_descriptor_of_the_binding_is_the_struct(layers):
    """What the binding builds from the shapes, byte for byte: paged and contiguous caches, every second layer of a larger one, and what it
    leaves to Python (rows in the cache, a width that is no int, other layers)."""
    B, T, Hkv, d, W = 2, 12, 3, 64, 5
    for dtype in (torch.bfloat16, torch.float32):
        kt = torch.zeros((layers, B, T, Hkv, d), dtype=dtype)
        paged, table = torch.zeros((2 * layers, 7, Hkv, 16, d), dtype=dtype), torch.zeros((B, 4), dtype=torch.int32)
        flat = torch.zeros((2 * layers, B, 40, Hkv, d), dtype=dtype)
        for step in (1, 2):
            pc, fc = paged[:step * layers:step], flat[:step * layers:step]
            sp, sf = (pc.stride(0), fc.stride(0)) if layers > 1 else (pc.numel(), fc.numel())
            e = dtype.itemsize
            for cache, bt, tail in ((pc, table, (16, 4, 7, 0, 0, sp)), (fc, None, (0, 0, 0, 40, 0, sf))):
                want = bytes(api.CommitDesc(B, T, Hkv, d, e, layers, W, *tail))
                assert api._native().commit_desc(kt, cache, bt, W) == want
                assert bytes(api._commit_desc(kt, cache, bt, np.int64(W))) == want and bytes(api._commit_desc(None, cache, bt, W, B, T)) == want
                assert api._native().commit_desc(None, cache, bt, W) is None and api._native().commit_desc(kt, cache, bt, np.int64(W)) is None
    assert api._native().commit_desc(kt, torch.zeros((layers + 1, B, 40, Hkv, d)), None, W) is None


def test_binding_refuses_what_is_not_a_device_tensor_or_a_descriptor():
    """The native call path checks its arguments before anything is launched; it needs no GPU to do so."""
    x = torch.zeros(8, dtype=torch.int32)
    call = api._native()
    with pytest.raises(AssertionError):          # host memory
        call.pack_lm_head(x, 1, 128, x)
    with pytest.raises(TypeError):               # neither a tensor nor None
        call.pack_lm_head([1, 2], 1, 128, None)
    with pytest.raises(TypeError):               # a size that is not an int
        call.pack_lm_head(None, 1.0, 128, None)
    with pytest.raises(TypeError):               # the C prototype's number of arguments, less the stream
        call.pack_lm_head(None, 1, 128)
    with pytest.raises(ValueError):              # shorter than the struct
        call.commit_accepted_kv(b"\0" * 8, *[None] * 13)
    with pytest.raises(ctypes.ArgumentError):    # another struct
        api.tree_verify_attention(x, x, x, x, x, x, x, x, P_max=1, desc=api.CommitDesc(), out=x, lse=x, workspace=x)
    assert call.empty_i32(x, 3, 4).shape == (3, 4) and call.empty_i32(x, 2).dtype == torch.int32


def test_binding_takes_every_integer_that_ctypes_takes():
    """Sizes come as ints, numpy integers or tensors of one element; what has no __index__ is refused.  Arguments are taken
    from left to right: the host tensor at the end is the one refused where the sizes before it are good."""
    call, x = api._native(), torch.zeros(8)
    for size in (8, True, np.int64(8), np.int32(8), np.uint8(8), torch.tensor(8), torch.tensor([8], dtype=torch.int32)):
        ctypes.c_int32.from_param(size)
        with pytest.raises(AssertionError):
            call.pack_lm_head(None, size, 128, x)
    for other in (8.0, np.float32(8), None, "8", torch.tensor(0.5), torch.tensor([0, 0])):
        with pytest.raises(TypeError):
            ctypes.c_int32.from_param(other)
        with pytest.raises(TypeError):
            call.pack_lm_head(None, other, 128, x)


def test_calls_refuse_queries_of_another_rank_and_rows_that_are_not_there():
    x, ws = torch.zeros((2, 3, 8), dtype=torch.bfloat16), torch.zeros(256, dtype=torch.uint8)
    with pytest.raises(ValueError):      # a descriptor of its own does not make up for a q that is not [B, T, Hq, d]
        api.tree_verify_attention(x, x, x, x, x, x, x, x, P_max=1, desc=api.AttnDesc(), out=x, want_lse=False, workspace=ws)
    tok, ret = torch.zeros((0, 3), dtype=torch.int32), torch.zeros((0, 2, 4), dtype=torch.int32)
    kt, kc = torch.zeros((1, 0, 3, 2, 64)), torch.zeros((1, 0, 8, 2, 64))
    with pytest.raises(IndexError):      # no first row to take the row's size from
        api.verify_epilogue(None, tok, ret, tok, kt, kt, kc, kc, tok, tok, src=tok[..., None], post_out={"argmax": tok})


def test_unforced_fp32_and_heads_of_64_plans_fit_the_fixed_array():
    """etv_tree_verify_attention_static cannot fall back on another workspace: a split that the library chooses by itself (fp32, heads
    of 64, and heads of 128) stays within its array, at every size, so that no unforced call is refused.  (Host only: the plan.)"""
    cases = [(64, api.BF16, 17, 60, 64, 8, 8192), (128, api.F32, 12, 60, 64, 8, 16384), (64, api.BF16, 8, 160, 64, 8, 4096),
             (128, api.F32, 24, 60, 28, 4, 16384)]
    cases += [(d, dt, B, T, Hq, Hkv, P) for d, dt in ((64, api.BF16), (64, api.F32), (128, api.F32), (128, api.BF16)) for B in (1, 3, 17, 40, 65, 129)
              for T in (1, 16, 60, 129, 256) for Hq, Hkv in ((4, 4), (32, 8), (64, 8), (28, 4), (257, 257)) for P in (0, 500, 8192, 100000)]
    for d, dt, B, T, Hq, Hkv, P in cases:
        dsc = api.AttnDesc(B=B, T_max=T, Hq=Hq, Hkv=Hkv, d=d, dtype=dt, P_cap=P, P_max=P)
        need = api.tree_verify_attention_workspace_bytes(dsc)
        assert need <= api.ATTN_STATIC_WORKSPACE_BYTES, (d, dt, B, T, Hq, Hkv, P, need)
        assert api.tree_verify_attention_plan(dsc)["n_splits"] >= 1


def test_key_block_launches_fit_every_xcd():
    """The key-block kernel runs where a launch fits the chip at once.  The chunks of one (split, KV head, sequence) stay on one of
    the eight XCDs, so the fullest XCD, not the sum, has to fit its 32 compute units (two workgroups on each at heads of 64)."""
    import random
    rng = random.Random(3)
    shapes = [(10, 96, 8, 2, 128, 230), (6, 107, 4, 2, 128, 2667)]
    shapes += [(rng.randint(1, 32), rng.randint(1, 256), *rng.choice([(8, 2), (4, 2), (32, 8), (32, 32), (16, 4)]), rng.choice([64, 128]),
                rng.choice([60, 230, 700, 2667, 9000])) for _ in range(600)]
    taken = 0
    for B, T, Hq, Hkv, d, P in shapes:
        plan = api.tree_verify_attention_plan(api.AttnDesc(B=B, T_max=T, Hq=Hq, Hkv=Hkv, d=d, dtype=api.BF16, P_cap=P, P_max=P))
        if plan["ring_stages"] == 0:
            taken += 1
            assert -(-B * plan["n_splits"] * Hkv // 8) * plan["row_groups"] <= (64 if d == 64 else 32), (B, T, Hq, Hkv, d, P, plan)
    assert taken > 100
