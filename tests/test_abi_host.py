"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol include/kvqp.h declares, answers its size queries, and rejects bad
arguments before anything could be launched."""
import ctypes as C
import os
import re

import pytest

from paper_2412_12706_amd import kvqp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(kvqp.LIB_PATH):
        from paper_2412_12706_amd import build
        build.build()
    return kvqp.lib()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "kvqp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kvqp_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_symbols()
    assert set(names) == set(kvqp.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_header_is_plain_c(tmp_path):
    """The boundary is a C ABI: the header must compile as C99 on its own, with no C++ or HIP types."""
    import shutil
    import subprocess
    if shutil.which("gcc") is None:
        pytest.skip("no C compiler")
    src = tmp_path / "t.c"
    src.write_text('#include "kvqp.h"\nint main(void) { kvqp_cfg c; kvqp_cache k; (void)c; (void)k; return KVQP_OK; }\n')
    r = subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", os.path.join(ROOT, "include"),
                        "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_version_and_strerror(lib):
    assert kvqp.version() >= 100
    assert kvqp.strerror(0) == "ok"
    for code in (-1, -2, -3, -4):
        assert kvqp.strerror(code) and kvqp.strerror(code) != kvqp.strerror(0)
    assert "unknown" in kvqp.strerror(-99)


def bpt(bits, G):
    return 512 if bits == 16 else 2 * (128 * bits // 8 + 4 * 128 // G)


@pytest.mark.parametrize("bits,G", [(2, 32), (2, 64), (4, 32), (4, 128), (8, 32), (16, 32)])
def test_cache_sizes_match_bytes_per_token(lib, bits, G):
    cfg = kvqp.Cfg(batch=3, n_q_heads=32, n_kv_heads=8, seq_len=4096 + 32, window=32, budget=1024, bits=bits, group_size=G)
    sizes = kvqp.cache_sizes(cfg, tail_cap=40)
    heads = 3 * 8
    assert sum(sizes[:6]) == heads * 1024 * bpt(bits, G)
    assert sizes[6] == sizes[7] == heads * 40 * 128 * 2
    # 2-bit value codes are padded to 64-token superblocks
    cfg2 = kvqp.Cfg(batch=1, n_q_heads=8, n_kv_heads=2, seq_len=1000, window=32, budget=96, bits=2, group_size=32)
    s2 = kvqp.cache_sizes(cfg2, 32)
    assert s2[0] == 2 * 96 * 128 * 2 // 8 and s2[1] == 2 * 128 * 128 * 2 // 8


def test_workspace_sizes_are_positive_and_compress_grows_with_the_problem(lib):
    small = kvqp.Cfg(batch=1, n_q_heads=32, n_kv_heads=8, seq_len=4096, window=32, budget=1024)
    big = kvqp.Cfg(batch=32, n_q_heads=32, n_kv_heads=8, seq_len=32768, window=32, budget=8192)
    (c0, d0), (c1, d1) = kvqp.workspace_bytes(small), kvqp.workspace_bytes(big)
    assert 0 < c0 < c1 and d0 > 0 and d1 > 0     # (decode: partials of the token-axis splits, few heads -> more splits)


BAD = [
    (dict(bits=3), -1), (dict(bits=0), -1), (dict(group_size=48), -1), (dict(group_size=16), -2),
    (dict(head_dim=64), -2), (dict(n_q_heads=30), -1), (dict(n_q_heads=8 * 16), -2), (dict(pool_kernel=4), -1),
    (dict(pool_kernel=0), -1), (dict(window=0), -1), (dict(window=5000), -1), (dict(budget=-1), -1),
    (dict(outlier_overflow_cap=-1), -1),
    (dict(key_axis=2), -1), (dict(batch=0), -1), (dict(window=128), -2), (dict(decode_splits=-1), -1),
    (dict(sm_scale=float("nan")), -1), (dict(decode_cache_hint=3), -1), (dict(decode_cache_hint=-1), -1),
]


@pytest.mark.parametrize("patch,code", BAD)
def test_invalid_configurations_are_rejected_on_the_host(lib, patch, code):
    base = dict(batch=1, n_q_heads=32, n_kv_heads=8, head_dim=128, seq_len=4096, window=32, pool_kernel=7, budget=1024,
                bits=4, group_size=32, key_axis=0, decode_splits=0, sm_scale=0.088)
    base.update(patch)
    cfg = kvqp.Cfg(**base)
    sizes = (C.c_size_t * 8)()
    assert lib.kvqp_cache_sizes(C.byref(cfg.struct()), max(cfg.window, 1), sizes) == code


def test_entry_points_reject_null_pointers_without_touching_the_device(lib):
    cfg = kvqp.Cfg(batch=1, n_q_heads=32, n_kv_heads=8, seq_len=4096, window=32, budget=1024)
    cs = kvqp.CacheStruct()
    st = cfg.struct()
    assert lib.kvqp_compress(C.byref(st), None, None, None, C.byref(cs), None, None, None, 0, None) == -1
    assert lib.kvqp_compress(None, None, None, None, None, None, None, None, 0, None) == -1
    assert lib.kvqp_quantize_selected(C.byref(st), None, None, None, 1024, C.byref(cs), None) == -1
    assert lib.kvqp_decode_attn(C.byref(st), None, C.byref(cs), None, None, 0, None) == -1
    # plausible non-null data pointers but cache buffers missing
    fake = C.c_void_p(0x1000)
    cs.tail_cap = 32
    assert lib.kvqp_compress(C.byref(st), fake, fake, fake, C.byref(cs), None, None, None, 0, None) == -1
    # complete pointers, workspace missing -> workspace error, still nothing launched
    for name in ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "tail_k", "tail_v"):
        setattr(cs, name, 0x1000)
    assert lib.kvqp_compress(C.byref(st), fake, fake, fake, C.byref(cs), None, None, None, 0, None) == -3
    cs.n_kept, cs.tail_len = 1024, 32
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, None, 0, None) == -3
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, fake, 16, None) == -3
    cs.tail_len = 64                      # beyond tail_cap
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, fake, 1 << 30, None) == -1
    cs.n_kept, cs.tail_len = 0, 0         # empty cache
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, fake, 1 << 30, None) == -1


def test_capacity_sizes_and_append_argument_checks(lib):
    """Buffers laid out for n_cap tokens are sized like a compact cache of n_cap
    tokens; kvqp_append_tail validates counts on the host before any launch."""
    cfg = kvqp.Cfg(batch=2, n_q_heads=32, n_kv_heads=8, seq_len=4096, window=32, budget=1024, bits=4, group_size=32)
    compact = kvqp.cache_sizes(cfg, 40)
    same = kvqp.cache_sizes_cap(cfg, 1024, 40)
    assert compact == same
    big = kvqp.cache_sizes_cap(cfg, 2048, 40)
    assert all(b == 2 * a for a, b in zip(compact[:6], big[:6])) and big[6:] == compact[6:]
    for bad in (1000, 1040, -64):         # not a multiple of 64 / negative
        with pytest.raises(kvqp.KvqpError):
            kvqp.cache_sizes_cap(cfg, bad, 40)
    st = cfg.struct()
    cs = kvqp.CacheStruct()
    for name in ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "tail_k", "tail_v"):
        setattr(cs, name, 0x1000)
    cs.n_kept, cs.tail_len, cs.tail_cap, cs.n_cap = 1024, 64, 96, 1088
    assert lib.kvqp_append_tail(None, C.byref(cs), 32, None) == -1
    assert lib.kvqp_append_tail(C.byref(st), None, 32, None) == -1
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 0, None) == -1       # nothing to move
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 48, None) == -1      # not whole groups
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 96, None) == -1      # more than the tail holds
    cs.tail_len = 96
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 96, None) == -1      # beyond the capacity
    cs.n_cap = 1000
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 32, None) == -1      # capacity below n_kept / misaligned
    assert (cs.n_kept, cs.tail_len) == (1024, 96)                               # untouched by rejected calls


def test_head_level_count_argument_checks(lib):
    """kvqp_compress_ragged validates every head's count on the host before anything is enqueued;
    the calls that do not take head-level counts say so."""
    cfg = kvqp.Cfg(batch=1, n_q_heads=8, n_kv_heads=2, seq_len=800, window=32, budget=256, bits=4, group_size=64)
    st = cfg.struct()
    cs = kvqp.CacheStruct()
    for name in ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "tail_k", "tail_v", "head_n_kept"):
        setattr(cs, name, 0x1000)
    cs.tail_cap = 32
    fake = C.c_void_p(0x1000)
    call = lambda counts, cache=cs: lib.kvqp_compress_ragged(C.byref(st), fake, fake, fake, (C.c_int32 * 2)(*counts),
                                                             C.byref(cache), None, None, fake, 1 << 30, None)
    assert lib.kvqp_compress_ragged(C.byref(st), fake, fake, fake, (C.c_int32 * 2)(256, 97), C.byref(cs), None, None, fake,
                                    16, None) == -3      # any count under the bound is fine: the call gets as far as the workspace check
    assert call([256, 320]) == -1         # above the bound is not
    assert call([-64, 64]) == -1
    assert lib.kvqp_compress_ragged(C.byref(st), fake, fake, fake, None, C.byref(cs), None, None, fake, 1 << 30, None) == -1
    no_counts = kvqp.CacheStruct.from_buffer_copy(cs)
    no_counts.head_n_kept = None
    assert call([256, 64], no_counts) == -1
    assert lib.kvqp_compress_ragged(C.byref(st), fake, fake, fake, (C.c_int32 * 2)(256, 64), C.byref(cs), None, None, fake,
                                    16, None) == -3      # counts fine, workspace too small: still nothing launched
    assert lib.kvqp_quantize_selected_ragged(C.byref(st), fake, fake, fake, 256, (C.c_int32 * 2)(256, 257), C.byref(cs),
                                             None) == -1      # above the bound
    assert lib.kvqp_quantize_selected_ragged(C.byref(st), fake, fake, fake, 256, None, C.byref(cs), None) == -1
    assert lib.kvqp_quantize_selected(C.byref(st), fake, fake, fake, 256, C.byref(cs), None) == -1
    # uniform calls refuse a cache that carries head-level counts
    assert lib.kvqp_compress(C.byref(st), fake, fake, fake, C.byref(cs), None, None, fake, 1 << 30, None) == -1
    cs.n_kept, cs.tail_len, cs.n_cap = 256, 32, 320
    assert lib.kvqp_append_tail(C.byref(st), C.byref(cs), 64, None) == -2
    # the head-level form checks the heads' current counts before anything is enqueued
    app = lambda counts, n=64, cache=cs: lib.kvqp_append_tail_ragged(C.byref(st), C.byref(cache), n,
                                                                      (C.c_int32 * 2)(*counts) if counts else None, None)
    cs.tail_len = 64
    assert app(None) == -1
    assert app([256, 96]) == -1           # appending wants whole key groups under the new rows
    assert app([256, 320]) == -1          # above the bound n_kept
    assert app([-64, 64]) == -1
    assert app([256, 64], 32) == -1       # n_tokens not whole groups
    assert app([256, 64], 128) == -1      # more than the tail holds (and than the capacity)
    no_counts = kvqp.CacheStruct.from_buffer_copy(cs)
    no_counts.head_n_kept = None
    assert app([256, 64], 64, no_counts) == -1
    assert (cs.n_kept, cs.tail_len) == (256, 64)
    cs.tail_len = 0
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, fake, 1 << 30, None) == -1   # a head may be empty


def test_outlier_filtering_argument_checks(lib):
    """Slot buffer sizes and the host-side rejects of the outlier-filtering mode."""
    base = dict(batch=2, n_q_heads=8, n_kv_heads=2, seq_len=800, window=32, budget=256, bits=4, group_size=32)
    on = kvqp.Cfg(**base, outlier_threshold=6.0)
    assert kvqp.outlier_sizes(on)[:2] == [2 * 2 * 256 * 4 * 4] * 2          # heads x tokens x 4 slots x 4 bytes
    assert kvqp.outlier_sizes(on, 320)[:2] == [2 * 2 * 320 * 4 * 4] * 2
    assert kvqp.outlier_sizes(on)[2:] == [2 * 2 * 12 * 4] * 2               # no list entries asked for: the prefix counts (9, padded to 12) alone
    assert kvqp.outlier_sizes(kvqp.Cfg(**{**on.__dict__, 'outlier_overflow_cap': 100}), 320)[2:] == [2 * 2 * (12 + 200) * 4] * 2
    assert kvqp.outlier_sizes(kvqp.Cfg(**base)) == [0, 0, 0, 0]
    for bad in (-1.0, float("nan"), float("inf")):
        with pytest.raises(kvqp.KvqpError):
            kvqp.outlier_sizes(kvqp.Cfg(**base, outlier_threshold=bad))
    with pytest.raises(kvqp.KvqpError):                                      # nothing is quantized at 16 bits
        kvqp.cache_sizes(kvqp.Cfg(**{**base, "bits": 16}, outlier_threshold=6.0), 32)
    st = on.struct()
    cs = kvqp.CacheStruct()
    for name in ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "tail_k", "tail_v"):
        setattr(cs, name, 0x1000)
    cs.tail_cap = 32
    fake = C.c_void_p(0x1000)
    assert lib.kvqp_compress(C.byref(st), fake, fake, fake, C.byref(cs), None, None, fake, 1 << 30, None) == -1   # no slot buffers
    cs.n_kept, cs.tail_len = 256, 32
    assert lib.kvqp_decode_attn(C.byref(st), fake, C.byref(cs), fake, fake, 1 << 30, None) == -1


def test_decode_workspace_covers_every_token_count(lib):
    """The decode workspace size does not depend on the token count, so a cache grown by appended
    tokens never outgrows it."""
    for heads, bits in ((8, 4), (8, 2), (256, 4), (2, 16)):
        sizes = set()
        for budget in (64, 1024, 8192, 32768):
            cfg = kvqp.Cfg(batch=heads // 2, n_q_heads=8, n_kv_heads=2, seq_len=40000, window=32, budget=budget, bits=bits,
                           group_size=32)
            sizes.add(kvqp.workspace_bytes(cfg)[1])
        assert len(sizes) == 1 and min(sizes) > 0, (heads, bits, sizes)
    a = kvqp.workspace_bytes(kvqp.Cfg(batch=1, n_q_heads=8, n_kv_heads=2, seq_len=4096, window=32, budget=1024, bits=4))[1]
    b = kvqp.workspace_bytes(kvqp.Cfg(batch=1, n_q_heads=8, n_kv_heads=2, seq_len=4096, window=32, budget=1024, bits=4,
                                      decode_splits=500))[1]
    assert b >= 2 * 500 * 4 * 256 * 4 and b > a      # the caller's split count is covered


def test_binding_raises_with_the_library_message(lib):
    cfg = kvqp.Cfg(batch=1, n_q_heads=32, n_kv_heads=8, seq_len=4096, window=32, budget=1024, bits=5)
    with pytest.raises(kvqp.KvqpError) as e:
        kvqp.cache_sizes(cfg, 32)
    assert "invalid argument" in str(e.value)


def test_product_package_does_not_import_the_checker():
    for root, _, files in os.walk(os.path.join(ROOT, "paper_2412_12706_amd")):
        for f in files:
            if f.endswith((".py", ".hip", ".cpp", ".h")):
                text = open(os.path.join(root, f)).read()
                assert "oracle" not in text.lower(), f"{f} mentions the checker"


def test_decode_workspace_init_and_static_entry_validate_on_the_host(lib):
    """The two decode-side additions reject bad calls before anything is enqueued (no GPU needed):
    the workspace preparation wants a workspace that holds the arrival counters, and the entry
    point on the library's own scratch array refuses launches whose partials do not fit it."""
    cfg = kvqp.Cfg(batch=4, n_q_heads=32, n_kv_heads=8, seq_len=4096, window=32, budget=1024, bits=4)
    st = cfg.struct()
    fake = C.c_void_p(0x1000)
    assert lib.kvqp_decode_workspace_init(None, fake, 1 << 20, None) == -1
    assert lib.kvqp_decode_workspace_init(C.byref(st), None, 1 << 20, None) == -3
    assert lib.kvqp_decode_workspace_init(C.byref(st), fake, 64, None) == -3            # 32 counters need 128 bytes
    assert lib.kvqp_decode_workspace_init(C.byref(st), C.c_void_p(0x1004), 1 << 20, None) == -1
    assert kvqp.workspace_bytes(cfg)[1] >= 256 + 32 * 4 * 256 * 4                         # counters, then partials
    cs = kvqp.CacheStruct()
    for name in ("k_codes", "v_codes", "k_scale", "k_zero", "v_scale", "v_zero", "tail_k", "tail_v"):
        setattr(cs, name, 0x1000)
    cs.n_kept, cs.tail_len, cs.tail_cap = 1024, 32, 32
    assert lib.kvqp_decode_attn_static(C.byref(st), None, C.byref(cs), fake, None) == -1
    assert lib.kvqp_decode_attn_static(C.byref(st), fake, None, fake, None) == -1
    # 128 heads cut into 16 splits by the caller: 16 MB of partials, beyond the library's array
    big = kvqp.Cfg(batch=16, n_q_heads=64, n_kv_heads=8, seq_len=4096, window=32, budget=1024, bits=4, decode_splits=16)
    assert kvqp.workspace_bytes(big)[1] > (8 << 20)
    assert lib.kvqp_decode_attn_static(C.byref(big.struct()), fake, C.byref(cs), fake, None) == -3


def test_structs_in_one_go_are_the_structs_field_by_field():
    """The binding packs the structs' bytes at once; numbers that do not fit are cut as ctypes cuts them."""
    import random
    import torch
    rng = random.Random(1)
    for odd in (False, True):
        for _ in range(200):
            ints = [rng.randrange(-2**(40 if odd else 31), 2**(40 if odd else 31)) for _ in range(14)]
            floats = [rng.choice([0.0, 1e-3, float("inf"), 1e39 if odd else 1.5]), rng.uniform(0, 1e4)]
            cfg = kvqp.Cfg(*ints[:12], *floats, *ints[12:])
            assert bytes(cfg.struct()) == bytes(kvqp.CfgStruct(*ints[:12], *floats, *ints[12:]))
            bufs = {n: torch.zeros(rng.choice([0, 8]), dtype=torch.uint8) for n in kvqp._NAMES + (() if rng.random() < 0.5 else ("k_out", "v_ovf"))}
            counts = None if rng.random() < 0.5 else torch.zeros(2, dtype=torch.int32)
            cache = kvqp.Cache(bufs, *ints[:4], counts)
            ptr = lambda n: bufs[n].data_ptr() if n in bufs else None
            want = kvqp.CacheStruct(*[ptr(n) for n in kvqp._NAMES], *ints[:4], None if counts is None else counts.data_ptr(),
                                    *[ptr(n) for n in ("k_out", "v_out", "k_ovf", "v_ovf")])
            assert bytes(cache.struct()) == bytes(want)
    with pytest.raises(TypeError):
        kvqp.Cfg(batch="1", n_q_heads=1, n_kv_heads=1).struct()


@pytest.mark.parametrize("missing", [None, "_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_the_undocumented_torch_names(monkeypatch, missing):
    """The binding asks torch for the current stream's handle by names that are not documented; a torch
    without one of them is asked for its current stream instead."""
    import types
    import torch
    for name, value in (("_cuda_getDevice", lambda: 3), ("_cuda_getCurrentRawStream", lambda device: 0x5000 + device)):
        monkeypatch.setattr(torch._C, name, value, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x7007))
    if missing:
        monkeypatch.delattr(torch._C, missing)
    assert kvqp._stream_ptr(None).value == (0x7007 if missing else 0x5003)
    assert kvqp._stream_ptr(types.SimpleNamespace(cuda_stream=0x9009)).value == 0x9009


def test_compress_workspace_is_no_larger_than_it_was():
    """A caller may have set aside what was stated when the statistics of up to 64 window rows came from chunks of 128 keys, two or
    four per workgroup and row, and those of more than 128 rows from workgroups of four steps or more: the size stated now is never larger."""
    import random
    cd = lambda a, b: -(-a // b)
    al = lambda v: cd(v, 256) * 256

    def former(c):
        L, W, heads = c.seq_len, c.window, c.batch * c.n_kv_heads
        P, rows = L - W, c.n_q_heads // c.n_kv_heads * W
        slabs = 0 if rows > 128 else 1 if rows <= 32 else 2 if rows <= 64 else 4
        strips, keys, share, least = (4 // slabs, 64 if slabs == 4 else 128, 16, 2) if slabs else (1, 64, 64, 4)
        n = cd(L, keys)
        wg = max(1, min(cd(min(2048, max(512, heads * n // share)), heads), cd(n, least)))
        rows_pad = 32 * slabs or 256
        tiles = max(1, cd(P, 4096))
        seg = min(15, cd(tiles, min(16, cd(512, heads), tiles)))
        kept = min(c.budget, P)
        size = al(max(heads * cd(n, cd(n, wg)) * strips * rows_pad * 8, heads * cd(tiles, seg) * 8192 if tiles > 1 else 0))
        size = al(size + heads * rows_pad * 16)
        size = al(size + heads * max(1, P) * 4)
        size = al(size + heads * max(8, cd(P, 8) * 8) * 2)
        return al(size + heads * max(1, kept) * 4) + (heads * cd(P, 8) * 8 * 4 if tiles > 1 else 0)

    rng = random.Random(5)
    for _ in range(3000):
        gq, W = rng.choice([1, 2, 4, 8]), rng.choice([1, 8, 13, 16, 32, 64])
        hkv = rng.choice([1, 2, 4, 8])
        L = int(2 ** rng.uniform(7, 17))
        if gq * W > 256 or L <= W:
            continue
        c = kvqp.Cfg(batch=rng.randint(1, 40), n_q_heads=hkv * gq, n_kv_heads=hkv, seq_len=L, window=W, budget=max(1, L // 4), bits=16)
        assert kvqp.workspace_bytes(c)[0] <= former(c), c


@pytest.mark.parametrize("P", [1, 4096, 4097, 9003, 12288, 12289, 20000])
@pytest.mark.parametrize("batch,hkv,gq,W", [(1, 8, 4, 32), (16, 8, 4, 8), (3, 2, 8, 8), (1, 8, 4, 64)])
def test_compress_workspace_holds_codes_and_pooled_scores_only_beyond_three_tiles(P, batch, hkv, gq, W):
    """Up to three pooling tiles the selection keeps the pooled scores to itself: besides row statistics, votes and survivors
    the workspace has nothing.  The parts of the statistics are whole, so what is left over shows."""
    c = kvqp.Cfg(batch=batch, n_q_heads=hkv * gq, n_kv_heads=hkv, seq_len=P + W, window=W, budget=max(1, P // 3), bits=4)
    heads, rows = batch * hkv, gq * W
    rows_pad = 32 if rows <= 32 else 64 if rows <= 64 else 128 if rows <= 128 else 256
    al = lambda v: -(-v // 256) * 256
    parts = kvqp.workspace_bytes(c)[0] - al(heads * rows_pad * 16) - al(heads * P * 4) - al(heads * c.n_kept * 4)
    if P > 12288:
        assert parts >= al(heads * -(-P // 8) * 16) + heads * -(-P // 8) * 32 + heads * 8192
    else:
        assert parts % (heads * rows_pad * 8) == 0 and 1 <= parts // (heads * rows_pad * 8) <= max(1, -(-(P + W) // 128))


def test_entry_points_are_published_with_their_argument_types(monkeypatch):
    """Threads may load the library at the same time, and one that is done calls while another still loads: an entry point must not be
    found without its argument types, which would cut addresses down to 32 bits."""
    kvqp.lib()

    class Table(dict):
        def __setitem__(self, name, function):
            assert function.argtypes is not None, name
            super().__setitem__(name, function)
    table = Table()
    monkeypatch.setattr(kvqp, "_fn", table)
    monkeypatch.setattr(kvqp, "_lib", None)
    kvqp.lib()
    assert set(table) == {"kvqp_compress", "kvqp_append_tail", "kvqp_decode_attn", "kvqp_decode_attn_static"}
