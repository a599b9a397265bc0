"""Host-side checks of libharris that need no GPU: the library loads, exports every
symbol include/harris.h declares, plans launches sensibly and rejects bad arguments
before anything is enqueued."""
import ctypes
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pkg():
    import paper_2212_12035_amd as p
    if not os.path.exists(p.library_path()):
        from paper_2212_12035_amd import build
        build.build_library()
    p.load_library()
    return p


def test_every_declared_symbol_is_exported(pkg):
    declared = set()
    for name in sorted(os.listdir(os.path.join(ROOT, "include"))):
        header = open(os.path.join(ROOT, "include", name)).read()
        header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
        declared |= set(re.findall(r"\b(harris_[a-z0-9_]+)\s*\(", header))
    assert declared == set(pkg.binding.EXPORTS)
    # the operator's own header stands alone: no launch-shape knobs in it
    public = open(os.path.join(ROOT, "include", "harris.h")).read()
    assert "HARRIS_TUNE_" not in re.sub(r"/\*.*?\*/", "", public, flags=re.S) and "harris_plan" not in public
    lib = ctypes.CDLL(pkg.library_path())
    for name in declared:
        assert getattr(lib, name) is not None


@pytest.mark.parametrize("missing", ["host compiler", "torch", "headers"])
def test_the_library_builds_without_the_bindings_module(tmp_path, monkeypatch, missing):
    # hipcc is a script that writes what it is asked for: only what build_library asks for is looked at.
    from paper_2212_12035_amd import build
    compiler = tmp_path / "hipcc"
    compiler.write_text("#!/bin/sh\nwhile [ $# -gt 1 ]; do [ \"$1\" = -o ] && : > \"$2\"; shift; done\n")
    failing = tmp_path / "c++"
    failing.write_text("#!/bin/sh\necho no headers\nexit 1\n")
    for script in (compiler, failing):
        script.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(compiler))
    monkeypatch.setenv("CXX", str(tmp_path / "none") if missing == "host compiler" else str(failing))
    if missing == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libharris.so"))
    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path / "objects"))
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / os.path.basename(build.NATIVE)))
    for stale in (build.NATIVE, str(tmp_path / "_harris_call.so")):      # of another build
        open(stale, "w").close()
    with pytest.warns(UserWarning, match="native marshalling is not built"):
        assert build.build_library() == build.LIB
    assert os.path.exists(build.LIB)
    assert [name for name in os.listdir(str(tmp_path)) if name.startswith("_harris_call")] == []


def test_the_bindings_module_is_used_with_its_own_torch_alone(pkg, monkeypatch):
    import types
    from paper_2212_12035_amd import binding
    lib, native = binding.load_library(), binding._native
    assert native is not None                            # the one built for this torch
    bound = []
    other = types.SimpleNamespace(torch_version="1.0", bind=lambda *args: bound.append(args))
    try:
        for module in (other, types.SimpleNamespace(bind=other.bind)):
            monkeypatch.setattr(pkg, "_harris_call", module)
            with pytest.warns(UserWarning, match="no native marshalling for torch"):
                binding._bind_native(lib)
            assert binding._native is None and bound == []
    finally:
        monkeypatch.undo()
        binding._bind_native(lib)
    assert binding._native is native


def test_version_and_strerror(pkg):
    assert pkg.harris_version() >= 100
    assert pkg.harris_strerror(0) == "success"
    msgs = {pkg.harris_strerror(s) for s in (-1, -2, -3, -4, -5)}
    assert len(msgs) == 5 and all(m and m != "unknown harris_status" for m in msgs)
    assert pkg.harris_strerror(-99) == "unknown harris_status"


def test_kernels_use_no_scratch_memory(pkg):
    # The library allocates nothing, and a kernel with a private segment makes the runtime back it with device
    # memory.  The code objects inside the library say what every kernel uses.  Scalar registers may go to
    # vector lanes (no memory) in the kernels that store result rows on any byte (the last template argument) alone.
    data = open(pkg.library_path(), "rb").read()
    kernels = {}
    for m in re.finditer(rb"\.name(?:\xd9(.)|\xda(..)|([\xa0-\xbf]))(_ZN?[A-Za-z0-9_]+?(?:6ParamsE|[a-z]))(?=[\x80-\xff])", data, re.S):
        end = data.find(b".wavefront_size", m.end())
        used = {}
        for key in (b".private_segment_fixed_size", b".sgpr_spill_count", b".vgpr_spill_count"):
            at = data.find(key, m.end(), end)
            if at >= 0:
                used[key] = data[at + len(key)]              # one byte: a count below 128
        if len(used) == 3:
            kernels[m.group(4)] = used
    assert len(kernels) > 150
    tiles = [name for name in kernels if b"harris_tile_kernel" in name]
    assert len(tiles) > 100 and any(b"harris_patch_kernel" in name for name in kernels)
    for name, used in kernels.items():
        assert used[b".private_segment_fixed_size"] == 0 and used[b".vgpr_spill_count"] == 0, (name, used)
        assert used[b".sgpr_spill_count"] == 0 or (b"harris_tile_kernel" in name and b"ELb1EEEv" in name), (name, used)


def test_8_bit_tiles_of_launches_resident_at_once_leave_room_for_eight_wavefronts(pkg):
    # 8-bit input, four pixels, four rows, shared rows kept: eight wavefronts per SIMD have 64 vector registers each.
    data = open(pkg.library_path(), "rb").read()
    counts = {}
    for m in re.finditer(rb"(_ZN?[A-Za-z0-9_]*harris_tile_kernelIhLi4ELi4ELin1E[A-Za-z0-9_]*?6ParamsE)(?=[\x80-\xff])", data, re.S):
        at = data.find(b".vgpr_count", m.end(), data.find(b".wavefront_size", m.end()) + 64)
        if at >= 0:
            counts[m.group(1)] = data[at + len(b".vgpr_count")]      # one byte: a count below 128
    assert len(counts) >= 8 and max(counts.values()) <= 64, counts


def test_plan_picks_widest_vector_path(pkg):
    shape, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560)
    assert shape["px"] == 4 and blocks > 128 and shape["rows"] >= 4
    # The tile kernel keeps four pixels per lane for any width and any row alignment the element
    # type allows (word-aligned vector accesses; 8-bit rows loaded as aligned words and shifted);
    # strip borders then stay where they are.
    for args, kw in (((pkg.HARRIS_F32, 1, 64, 98), {}), ((pkg.HARRIS_F32, 1, 64, 97), {}),
                     ((pkg.HARRIS_F32, 1, 64, 96), dict(rgb_align=4)), ((pkg.HARRIS_F32, 1, 64, 96), dict(out_align=8)),
                     ((pkg.HARRIS_U8, 1, 64, 96), dict(rgb_align=1)), ((pkg.HARRIS_U8, 1, 64, 99), dict(rgb_align=1, out_align=4))):
        shape = pkg.harris_plan(*args, **kw)[0]
        assert shape["px"] == 4 and shape["schedule"] == pkg.HARRIS_SCHEDULE_TILES and shape["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES, (args, kw)
        with pytest.raises(pkg.HarrisError) as e:           # moved borders need naturally aligned lanes
            pkg.harris_plan(*args, tuning=dict(flags=pkg.HARRIS_TUNE_ALIGNED_STORES), **kw)
        assert e.value.status == -3
    # shifted 8-bit rows: strips of at most 248 columns (the last lane only supplies bytes): 500 columns take 3, not 2
    plain = dict(rows=4, waves_per_block=4, flags=pkg.HARRIS_TUNE_PLAIN_STORES)
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 64, 504, tuning=plain)[1] == 2 * 5
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 64, 504, rgb_align=1, tuning=plain)[1] == 3 * 5
    # the band schedule keeps naturally aligned lanes: narrower ones for such rows
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 98, tuning=dict(schedule=1))[0]["px"] == 2
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 97, tuning=dict(schedule=1))[0]["px"] == 1
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 96, rgb_align=4, tuning=dict(schedule=1))[0]["px"] == 1
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 96, out_align=8, tuning=dict(schedule=1))[0]["px"] == 2
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 64, 96, rgb_align=1, tuning=dict(schedule=1))[0]["px"] == 1
    # 8-bit codes are one word per lane: rows of codes off 4-byte boundaries take narrower lanes
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_U8, 1, 64, 98, out_align=1)[0]["px"] == 1
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_F16, 1, 64, 98, out_align=4)[0]["px"] == 4
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_F16, 1, 64, 97, out_align=2)[0]["px"] == 1
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 8192, 8192)[0]["px"] == 4


def test_plan_tile_arithmetic(pkg):
    # 252 result columns per wavefront at px = 4; 2556 columns -> 11 strips; 1532 rows in
    # bands of 16 -> 96 bands; 4 wavefronts per workgroup.
    t = dict(schedule=pkg.HARRIS_SCHEDULE_BANDS, px=4, rows=16, prefetch=3, waves_per_block=4, flags=pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES)
    shape, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=t)
    assert shape == dict(t, lds_kb=0) and blocks == 6 * 48          # 2 strips x 2 bands per workgroup: ceil(11/2) x ceil(96/2)
    shape, blocks = pkg.harris_plan(pkg.HARRIS_F32, 3, 9, 9, tuning=dict(schedule=1, px=1, rows=2, prefetch=3, waves_per_block=1, flags=3))
    assert blocks == 3 * 3 * 1
    # tiles: 8 wavefronts x 8 rows give 60 result rows per tile -> 26 tiles down, 11 across,
    # one workgroup each
    t = dict(schedule=pkg.HARRIS_SCHEDULE_TILES, px=4, rows=8, prefetch=0, waves_per_block=8, flags=pkg.HARRIS_TUNE_CACHED_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES)
    shape, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=t)
    assert shape == dict(t, lds_kb=32) and blocks == 26 * 11      # 8 wavefronts publish 4 KB each
    # strip borders moved to 64-byte boundaries: strips of at most 240 columns; 4252 columns
    # take 18 of them instead of 17, 2556 columns still 11
    aligned = dict(t, flags=pkg.HARRIS_TUNE_CACHED_LOADS | pkg.HARRIS_TUNE_ALIGNED_STORES)
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=aligned) == (dict(aligned, lds_kb=32), 26 * 11)
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 4256, tuning=aligned)[1] == 26 * 18
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 4256, tuning=t)[1] == 26 * 17
    # empty results plan to zero workgroups
    assert pkg.harris_plan(pkg.HARRIS_F32, 0, 64, 64)[1] == 0
    assert pkg.harris_plan(pkg.HARRIS_F32, 2, 4, 64)[1] == 0
    assert pkg.harris_plan(pkg.HARRIS_F32, 2, 64, 4)[1] == 0


def test_plan_defaults_follow_the_problem_size(pkg):
    small, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560)
    # one tile per CU: 11 strips x 23 tiles of 9 wavefronts x 8 rows (68 result rows) = 253 workgroups
    assert small["schedule"] == pkg.HARRIS_SCHEDULE_TILES and (small["rows"], small["waves_per_block"]) == (8, 9) and blocks == 253
    assert small["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_ALIGNED_STORES | pkg.HARRIS_TUNE_FLAG_HANDOFF
    # few, tall tiles take ready flags instead of the barrier; tiles of fewer than 5 wavefronts keep the barrier
    assert not pkg.harris_plan(pkg.HARRIS_F32, 1, 720, 1280)[0]["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1080, 1920)[0]["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF
    assert not pkg.harris_plan(pkg.HARRIS_U8, 1, 2048, 4096)[0]["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF     # 8-bit input keeps the barrier
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=dict(flags=pkg.HARRIS_TUNE_STREAM_LOADS))[0]["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_ALIGNED_STORES
    # short tiles take few rows per wavefront, and several images with short tiles take many small tiles
    assert [pkg.harris_plan(pkg.HARRIS_F32, 1, 768, 1024)[0][key] for key in ("rows", "waves_per_block")] == [5, 4]
    assert [pkg.harris_plan(pkg.HARRIS_F32, 1, 1024, 1024)[0][key] for key in ("rows", "waves_per_block")] == [6, 4]
    assert [pkg.harris_plan(pkg.HARRIS_F32, 1, 2160, 3840)[0][key] for key in ("rows", "waves_per_block")] == [10, 14]
    # 8-bit input: fewer rows per wavefront for tall tiles
    assert [pkg.harris_plan(pkg.HARRIS_U8, 1, 1536, 2560)[0][key] for key in ("rows", "waves_per_block")] == [6, 12]
    assert [pkg.harris_plan(pkg.HARRIS_U8, 1, 2160, 3840)[0][key] for key in ("rows", "waves_per_block")] == [9, 16]
    # tiles of 26 to 32 rows (40 for 8-bit input) give way to many small tiles
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 960, 1280)[1] == 6 * 80 and pkg.harris_plan(pkg.HARRIS_F32, 1, 1080, 1920)[1] <= 256
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 1080, 1920)[1] == 8 * 90
    # ... for float32 input only while at most two small tiles come to lie on a CU (512 in all): 900x1600 would be 525
    mid, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 900, 1600)
    assert (mid["rows"], mid["waves_per_block"]) == (6, 5) and blocks == 7 * 35 and mid["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1024, 1280)[1] == 6 * 85
    two, blocks = pkg.harris_plan(pkg.HARRIS_F32, 2, 720, 1280)
    assert (two["rows"], two["waves_per_block"]) == (5, 8) and blocks == 2 * 6 * 20
    several, blocks = pkg.harris_plan(pkg.HARRIS_F32, 4, 480, 640)
    assert (several["rows"], several["waves_per_block"]) == (4, 4) and blocks == 4 * 3 * 40
    # beyond one tile per CU: many tiles, non-temporal loads except the rows two tiles share, which stay in L2,
    # and an LDS reservation that holds the tiles resident on a CU down (160 KB per CU).
    # float32 results of 128 to 400 MB: 4 wavefronts x 5 rows (16 result rows per tile), 3 tiles per CU
    mid, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 2832, 4256)
    assert (mid["schedule"], mid["rows"], mid["waves_per_block"], mid["lds_kb"]) == (2, 5, 4, 48) and blocks == 18 * 177
    assert mid["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_ALIGNED_STORES
    assert [pkg.harris_plan(pkg.HARRIS_F32, 2, 2160, 3840)[0][key] for key in ("rows", "waves_per_block", "lds_kb")] == [5, 4, 48]
    # beyond 400 MB: 8 images or more 5 wavefronts x 5 rows (21 result rows per tile), fewer images 5 x 6; 2 tiles per CU
    assert [pkg.harris_plan(pkg.HARRIS_F32, 16, 1080, 1920)[0][key] for key in ("rows", "waves_per_block", "lds_kb")] == [5, 5, 64]
    assert [pkg.harris_plan(pkg.HARRIS_F32, 1, 8192, 8192)[0][key] for key in ("rows", "waves_per_block", "lds_kb")] == [6, 5, 64]
    big, blocks = pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920)
    assert (big["rows"], big["waves_per_block"], big["lds_kb"]) == (5, 5, 64) and blocks == 64 * 52 * 8
    assert big["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_ALIGNED_STORES
    # 16-bit results above 128 MB: 4 x 6, 3 tiles per CU; one image beyond 800 MB: 5 x 6, 2 per CU
    half, _ = pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_F16, 64, 1080, 1920)
    assert (half["rows"], half["waves_per_block"], half["lds_kb"]) == (6, 4, 48)
    assert half["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_ALIGNED_STORES
    wide, _ = pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_BF16, 1, 8192, 8192)
    assert (wide["rows"], wide["waves_per_block"], wide["lds_kb"]) == (6, 5, 64)
    # an explicit shape gets no reservation beyond the tile's own rows (4 KB per wavefront); an explicit one is kept
    assert pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920, tuning=dict(rows=5, waves_per_block=5))[0]["lds_kb"] == 20
    assert pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920, tuning=dict(rows=5, waves_per_block=5, lds_kb=40))[0]["lds_kb"] == 40
    assert pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920, tuning=dict(lds_kb=28))[0]["lds_kb"] == 28
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560)[0]["lds_kb"] == 36            # one tile per CU: 9 wavefronts, no more
    # 8-bit input takes every wavefront that fits
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 8192, 8192)[0]["lds_kb"] == 16
    # many tiles below 128 MB as well (32 images of 512x512 cannot be one tile per CU): shared rows kept
    many, blocks = pkg.harris_plan(pkg.HARRIS_F32, 32, 512, 512)
    assert (many["rows"], many["waves_per_block"], many["lds_kb"]) == (4, 4, 36) and blocks > 256
    assert many["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_ALIGNED_STORES
    # lanes narrower than 16 bytes have no mixed policy: default-policy loads from 128 MB on
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 2832, 4258, tuning=dict(px=2))[0]["flags"] == pkg.HARRIS_TUNE_CACHED_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES
    # a width that is no multiple of 4 keeps the 16-byte lanes and their policy, with fixed strip borders
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 2832, 4258)[0]["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_PLAIN_STORES
    # 8-bit input: non-temporal loads; 35 strips of at most 240 columns cover 8188
    u8, blocks = pkg.harris_plan(pkg.HARRIS_U8, 1, 8192, 8192)
    assert u8["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_KEEP_SHARED_ROWS | pkg.HARRIS_TUNE_ALIGNED_STORES and blocks == 35 * 683
    assert (u8["rows"], u8["waves_per_block"]) == (4, 4)
    assert pkg.harris_plan(pkg.HARRIS_U8, 1, 64, 98, rgb_align=1)[0]["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES
    # narrower lanes and bands never move strip borders
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 98)[0]["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES
    assert pkg.harris_plan(pkg.HARRIS_F32, 1, 64, 96, tuning=dict(schedule=1))[0]["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES
    # an explicit policy is kept
    kept, _ = pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920, tuning=dict(flags=pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES))
    assert kept["flags"] == pkg.HARRIS_TUNE_STREAM_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES
    # asking for bands gives bands: one wavefront per SIMD for small problems, four-wavefront groups for large
    bands, blocks = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=dict(schedule=1))
    assert (bands["rows"], bands["prefetch"], bands["waves_per_block"]) == (17, 3, 1) and blocks == 1001
    bands, blocks = pkg.harris_plan(pkg.HARRIS_F32, 64, 1080, 1920, tuning=dict(schedule=1))
    assert (bands["rows"], bands["prefetch"], bands["waves_per_block"]) == (32, 3, 4) and blocks == 64 * 17 * 4


def test_a_planned_shape_gives_the_same_launch(pkg):
    # What a plan reports can be passed back: same shape, same workgroups.  Over the calls of the
    # performance cases, and over sizes, types and row boundaries drawn at random.
    import random
    F32, U8 = pkg.HARRIS_F32, pkg.HARRIS_U8
    O32, O16, OB16, O8 = pkg.HARRIS_OUT_F32, pkg.HARRIS_OUT_F16, pkg.HARRIS_OUT_BF16, pkg.HARRIS_OUT_U8
    calls = [(F32, O32, 1, 64, 96, 16, 16), (U8, O32, 1, 480, 640, 16, 16), (F32, O32, 1, 1536, 2560, 16, 16), (F32, O32, 1, 2832, 4256, 16, 16),
             (F32, O32, 64, 1080, 1920, 16, 16), (U8, O32, 1, 8192, 8192, 16, 16), (U8, O32, 8, 1079, 1919, 1, 4), (F32, O32, 1, 1501, 2203, 4, 4),
             (F32, O16, 1, 2831, 4255, 4, 2), (U8, O8, 16, 768, 1366, 2, 2), (U8, O8, 16, 768, 1366, 1, 1), (F32, O32, 2048, 64, 64, 16, 16),
             (F32, O32, 1000, 65, 65, 4, 4), (U8, O32, 3000, 61, 31, 1, 4), (F32, O32, 1, 2160, 3840, 16, 16), (U8, O8, 1, 8192, 8192, 16, 16)]
    rng = random.Random(7)
    for _ in range(3000):
        dtype, out = rng.choice((F32, U8)), rng.choice((O32, O16, OB16, O8))
        px, W = 10 ** rng.uniform(3, 8), int(10 ** rng.uniform(0.8, 3.9))
        H = max(5, int(10 ** rng.uniform(0.8, 3.9)))
        calls.append((dtype, out, max(1, int(px / (H * W))), H, W, rng.choice((1, 2, 4, 16) if dtype == U8 else (4, 8, 16)),
                      rng.choice({O32: (4, 8, 16), O8: (1, 2, 4, 16)}.get(out, (2, 4, 16)))))
    words = packed = 0
    for dtype, out, B, H, W, rgb_align, out_align in calls:
        shape, blocks = pkg.harris_plan_typed(dtype, out, B, H, W, rgb_align, out_align)
        assert pkg.harris_plan_typed(dtype, out, B, H, W, rgb_align, out_align, tuning=shape) == (shape, blocks), (dtype, out, B, H, W, rgb_align, out_align)
        words += bool(shape["flags"] & pkg.HARRIS_TUNE_WORD_STORES)
        packed += bool(shape["flags"] & pkg.HARRIS_TUNE_PACKED_IMAGES)
    assert words > 20 and packed > 20
    # the two bits by themselves: where the kernels can take the problem, and nowhere else
    W_, P_ = pkg.HARRIS_TUNE_WORD_STORES, pkg.HARRIS_TUNE_PACKED_IMAGES
    assert pkg.harris_plan_typed(F32, O16, 1, 64, 97, 4, 2, tuning=dict(flags=W_))[0]["px"] == 4
    assert pkg.harris_plan_typed(U8, O8, 1, 64, 7, 1, 1, tuning=dict(flags=W_, rows=8, waves_per_block=2))[0]["flags"] & W_
    assert not pkg.harris_plan_typed(F32, O16, 1, 64, 96, 16, 16, tuning=dict(flags=W_))[0]["flags"] & W_       # stored directly
    assert pkg.harris_plan(F32, 2, 5, 5, 4, 4, tuning=dict(flags=P_)) == (dict(schedule=2, px=4, rows=4, prefetch=0, waves_per_block=2, flags=P_ | 36, lds_kb=8), 1)
    assert pkg.harris_plan(F32, 7, 64, 101, 4, 4, tuning=dict(flags=P_, waves_per_block=3))[1] == 4 * 8
    for out, shape, bad in ((O32, (2, 64, 96), dict(flags=W_)), (O16, (2, 64, 97), dict(flags=W_, px=2)), (O16, (2, 64, 97), dict(flags=W_, schedule=1)),
                            (O16, (2, 64, 97), dict(flags=W_ | 16)), (O16, (2, 64, 96), dict(flags=P_)), (O32, (1, 64, 96), dict(flags=P_)),
                            (O32, (2, 64, 129), dict(flags=P_)), (O32, (2, 64, 96), dict(flags=P_ | 8)), (O32, (2, 64, 96), dict(flags=P_ | 16)),
                            (O32, (2, 64, 96), dict(flags=P_, rows=5)), (O32, (2, 64, 96), dict(flags=P_, waves_per_block=9)),
                            (O32, (2, 64, 96), dict(flags=P_, px=2)), (O32, (2, 64, 96), dict(flags=P_, schedule=1)), (O32, (2, 64, 96), dict(flags=P_ | W_))):
        with pytest.raises(pkg.HarrisError) as e:
            pkg.harris_plan_typed(F32, out, *shape, 4, 4 if out == O32 else 2, tuning=bad)
        assert e.value.status == -3, bad
    # empty results are planned, not refused
    assert pkg.harris_plan(F32, 0, 64, 64, tuning=dict(flags=P_))[1] == 0 and pkg.harris_plan(F32, 2, 4, 64, tuning=dict(flags=P_))[1] == 0


def test_plan_rejects_bad_arguments(pkg):
    E = pkg.HarrisError
    for args, status in [
        ((7, 1, 64, 64), -3),                       # unknown dtype
        ((0, -1, 64, 64), -2), ((0, 1, 3, 64), -2), ((0, 1, 64, 3), -2),
        ((0, 2 ** 31 - 1, 4096, 4096), -2),         # more tiles than a grid can hold
        ((0, 1, 8, 2 ** 28 + 4), -2),               # row offsets would not fit 32 bits
        ((0, 1, 2 ** 30 + 1, 8), -2),               # row indices would not fit int
        ((0, 2 ** 31 - 1, 2 ** 30, 2 ** 28), -2),   # byte counts would not fit 64 bits
        ((1, 2 ** 20, 2 ** 30, 2 ** 28), -2),
    ]:
        with pytest.raises(E) as e:
            pkg.harris_plan(*args)
        assert e.value.status == status
    for bad in (dict(px=3), dict(px=4, prefetch=5), dict(schedule=1, px=4, waves_per_block=3), dict(waves_per_block=1), dict(flags=256), dict(flags=12), dict(flags=48), dict(flags=64), dict(flags=64 | 4), dict(schedule=1, flags=64 | 8), dict(px=2, flags=64 | 8),
                dict(flags=128 | 4), dict(flags=128 | 64 | 8), dict(schedule=1, flags=128), dict(px=2, flags=128), dict(schedule=1, flags=16), dict(px=2, flags=16), dict(rows=-1),
                dict(schedule=3), dict(schedule=2, rows=7), dict(schedule=2, px=2, rows=5), dict(schedule=2, waves_per_block=1), dict(schedule=2, waves_per_block=17),
                dict(schedule=2, prefetch=3), dict(schedule=2, px=8), dict(px=8), dict(prefetch=2), dict(schedule=1, prefetch=6), dict(schedule=2, px=2, rows=8),
                dict(lds_kb=65), dict(lds_kb=-1), dict(schedule=1, lds_kb=16)):
        with pytest.raises(E) as e:
            pkg.harris_plan(0, 1, 64, 64, tuning=bad)
        assert e.value.status == -3
    with pytest.raises(E):                          # px = 4 in the band schedule needs W % 4 == 0
        pkg.harris_plan(0, 1, 64, 98, tuning=dict(schedule=1, px=4))
    with pytest.raises(E) as e:                     # ready flags: float32 input only
        pkg.harris_plan(pkg.HARRIS_U8, 1, 64, 64, tuning=dict(flags=pkg.HARRIS_TUNE_FLAG_HANDOFF))
    assert e.value.status == -3


def test_plan_for_16_bit_results(pkg):
    # 16-bit results: tile kernel only; moved strip borders reach up to 28 columns (64 bytes),
    # so strips are at most 224 columns; the widest lanes need 8-byte aligned result rows.
    F16, BF16 = pkg.HARRIS_OUT_F16, pkg.HARRIS_OUT_BF16
    shape, blocks = pkg.harris_plan_typed(pkg.HARRIS_F32, F16, 64, 1080, 1920)
    assert shape["schedule"] == pkg.HARRIS_SCHEDULE_TILES and shape["px"] == 4 and shape["flags"] & pkg.HARRIS_TUNE_ALIGNED_STORES
    assert blocks == 64 * 54 * 9                                # ceil(1916 / 224) = 9 strips (8 for float32 results); tiles of 20 result rows
    # small problems and 8-bit input keep the wider strips with fixed borders
    small, blocks = pkg.harris_plan_typed(pkg.HARRIS_F32, F16, 1, 1536, 2560)
    assert small["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES and (small["rows"], small["waves_per_block"]) == (8, 9) and blocks == 253
    assert pkg.harris_plan_typed(pkg.HARRIS_U8, BF16, 1, 8192, 8192)[0]["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, F16, 1, 1536, 2560, tuning=dict(flags=pkg.HARRIS_TUNE_ALIGNED_STORES))[1] % 12 == 0
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, BF16, 1, 64, 96, out_align=4)[0]["px"] == 4      # word-aligned 8-byte stores
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, BF16, 1, 64, 96, out_align=2)[0]["px"] == 1
    # rows with an odd number of 16-bit results: the last column would share a 32-bit word with what lies behind the row
    for odd in (97, 131, 1001):
        assert pkg.harris_plan_typed(pkg.HARRIS_F32, F16, 2, 64, odd, out_align=4)[0]["px"] == 1
        assert pkg.harris_plan_typed(pkg.HARRIS_U8, BF16, 2, 64, odd, rgb_align=1, out_align=4)[0]["px"] == 1
        assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_F32, 2, 64, odd, out_align=4)[0]["px"] == 4
        with pytest.raises(pkg.HarrisError):
            pkg.harris_plan_typed(pkg.HARRIS_F32, F16, 2, 64, odd, out_align=4, tuning=dict(px=4))
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_F32, 1, 1536, 2560) == pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560)
    for bad in (dict(out_dtype=4), dict(out_dtype=F16, tuning=dict(schedule=1)), dict(out_dtype=F16, tuning=dict(prefetch=3)),
                dict(out_dtype=F16, out_align=1), dict(out_dtype=F16, tuning=dict(px=8))):
        with pytest.raises(pkg.HarrisError) as e:
            pkg.harris_plan_typed(pkg.HARRIS_F32, bad["out_dtype"], 1, 64, 96, out_align=bad.get("out_align", 16), tuning=bad.get("tuning"))
        assert e.value.status == -3
    # 8-bit results: plain strips by default, at most 192 columns with moved borders, byte-aligned rows allowed
    u8out, blocks = pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_U8, 64, 1080, 1920)
    assert u8out["flags"] & pkg.HARRIS_TUNE_PLAIN_STORES and blocks == 64 * 54 * 8
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_U8, 64, 1080, 1920, tuning=dict(flags=pkg.HARRIS_TUNE_ALIGNED_STORES))[1] == 64 * 54 * 10
    assert pkg.harris_plan_typed(pkg.HARRIS_F32, pkg.HARRIS_OUT_U8, 1, 64, 96, out_align=1)[0]["px"] == 1
    lib = pkg.load_library()
    one = ctypes.c_void_p(4096)
    assert lib.harris_coarsity_typed(one, 0, 1, 64, 64, None, 0.04, 1.0, 0, one, 7, None, None) == -3
    assert lib.harris_coarsity_typed(one, 0, 1, 64, 64, None, 0.04, 1.0, 0, one, pkg.HARRIS_OUT_U8, None, None) == -3   # 8-bit codes need a scale
    assert lib.harris_coarsity_quantized(one, 0, 1, 64, 64, None, 0.04, 1.0, 0, float("nan"), 0.0, one, None, None) == -3
    assert lib.harris_coarsity_quantized(one, 0, 1, 64, 64, None, 0.04, 1.0, 0, 1.0, float("inf"), one, None, None) == -3
    assert lib.harris_coarsity_quantized(None, 0, 1, 64, 64, None, 0.04, 1.0, 0, 1.0, 0.0, one, None, None) == -1
    assert lib.harris_coarsity_quantized(None, 0, 0, 64, 64, None, 0.04, 1.0, 0, 1.0, 0.0, None, None, None) == 0
    assert lib.harris_coarsity_typed(one, 0, 1, 64, 64, None, 0.04, 1.0, 0, ctypes.c_void_p(4097), 1, None, None) == -3
    assert lib.harris_coarsity_typed(None, 0, 0, 64, 64, None, 0.04, 1.0, 0, None, 2, None, None) == 0


def test_plan_of_codes_from_8_bit_images_weighs_the_last_tile(pkg):
    # Codes of 8-bit images above 128 MB: tiles of 36 result rows where they compute at most 0.9 of the
    # rows that tiles of 12 do, as images of a few rows more than a multiple of 36 do not.
    for H, rows in ((16, 4), (24, 4), (40, 10), (44, 4), (60, 4), (80, 4), (96, 4), (112, 10), (240, 10), (720, 10)):
        B = 250000000 // (4 * H * 512)
        shape = pkg.harris_plan_typed(pkg.HARRIS_U8, pkg.HARRIS_OUT_U8, B, H, 512)[0]
        assert (shape["px"], shape["rows"], shape["waves_per_block"]) == (4, rows, 4), H
    assert pkg.harris_plan_typed(pkg.HARRIS_U8, pkg.HARRIS_OUT_U8, 1, 8192, 8192)[0]["rows"] == 10
    assert pkg.harris_plan_typed(pkg.HARRIS_U8, pkg.HARRIS_OUT_U8, 8, 1080, 1920)[0]["rows"] == 4


def test_plan_takes_wide_lanes_for_odd_rows_where_they_replace_enough_strips(pkg):
    # 16-bit results and codes on rows off 4-byte boundaries: four pixels per lane only where a strip of
    # them replaces more strips of the narrower lanes than it costs, and from a size on (see the planner).
    F32, U8, O16, O8 = pkg.HARRIS_F32, pkg.HARRIS_U8, pkg.HARRIS_OUT_F16, pkg.HARRIS_OUT_U8
    for dtype, out, B, H, W, px in (
            (F32, O16, 13889, 64, 9, 1), (U8, O8, 2049, 64, 61, 1), (F32, O16, 1289, 64, 97, 1), (U8, O16, 1289, 64, 97, 4), (U8, O8, 248, 64, 101, 1),
            (F32, O16, 776, 64, 161, 4), (F32, O16, 33, 200, 301, 1), (F32, O16, 415, 64, 301, 4), (F32, O16, 130, 64, 241, 1), (F32, O16, 1, 1079, 1919, 4),
            (F32, O16, 1, 2831, 4255, 4), (U8, O16, 8, 1079, 1919, 4), (F32, O16, 1, 401, 700 + 1, 1),
            # an even number of codes: the narrower lanes hold two pixels
            (U8, O8, 248, 64, 102, 2), (F32, O8, 8000, 64, 122, 2), (U8, O8, 1000, 64, 242, 4), (F32, O8, 1000, 64, 254, 4), (U8, O8, 1000, 64, 254, 2),
            (U8, O8, 16, 768, 1366, 4), (U8, O8, 1, 768, 1366, 2)):
        two = out == O8 and W % 2 == 0
        shape = pkg.harris_plan_typed(dtype, out, B, H, W, rgb_align=(8 if two else 4) if dtype == F32 else 2 if two else 1, out_align=2 if two or out == O16 else 1)[0]
        assert shape["px"] == px and bool(shape["flags"] & pkg.HARRIS_TUNE_WORD_STORES) == (px == 4), (dtype, out, B, H, W, shape)


def test_copy_probe_validates_its_arguments(pkg):
    lib = pkg.load_library()
    one = ctypes.c_void_p(4096)
    assert lib.harris_probe_copy(None, 0, 1, 64, 64, one, None) == -1
    assert lib.harris_probe_copy(one, 2, 1, 64, 64, one, None) == -3
    assert lib.harris_probe_copy(one, 0, 1, 3, 64, one, None) == -2
    assert lib.harris_probe_copy(ctypes.c_void_p(4100), 0, 1, 64, 64, one, None) == -3      # rgb not 16-byte aligned
    assert lib.harris_probe_copy(one, 1, 1, 5, 7, one, None) == -3                           # planes of 35 bytes
    assert lib.harris_probe_copy(one, 0, 1, 9, 11, one, None) == -3                          # 35 results: rows of images not 16-byte multiples
    assert lib.harris_probe_copy(None, 0, 0, 64, 64, None, None) == 0


def test_stream_probe_validates_its_arguments(pkg):
    lib = pkg.load_library()
    one = ctypes.c_void_p(4096)
    assert lib.harris_probe_stream(0, one, one, 1024, None) == -3                      # unknown kind
    assert lib.harris_probe_stream(4, one, one, 1024, None) == -3
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_NONE, None, None, -1, None) == -2     # the idle launch ignores all but the sign
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_READ, None, one, 1024, None) == -1
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_READ, one, None, 1024, None) == -1
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_WRITE, None, None, 1024, None) == -1
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_WRITE, None, one, 1000, None) == -3     # not a multiple of 16
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_WRITE, None, ctypes.c_void_p(4100), 1024, None) == -3
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_READ, ctypes.c_void_p(4104), one, 1024, None) == -3
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_WRITE, None, one, -16, None) == -2
    assert lib.harris_probe_stream(pkg.HARRIS_PROBE_READ, None, None, 0, None) == 0          # nothing to move


def test_index_division_by_multiplication_is_exact(tmp_path):
    # The tile kernel splits its workgroup index with a multiply-high division whose constants
    # the host computes; the same header functions are checked here against the hardware division.
    import subprocess
    exe = str(tmp_path / "fastdiv_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2212_12035_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fastdiv_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout


def test_compact_kernel_arguments(tmp_path):
    # The tile kernels and those for narrow images take their arguments in 96 bytes: what they unpack is what the planner
    # decided, over random calls, and calls that do not fit go to the kernels with whole arguments.
    import subprocess
    csrc = os.path.join(ROOT, "paper_2212_12035_amd", "csrc")
    exe = str(tmp_path / "arguments_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                    os.path.join(ROOT, "tests", "arguments_check.cpp"), os.path.join(csrc, "harris_api.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout


def test_planned_launches(tmp_path):
    # Batches of narrow images in every combination of gaps between rows, planes and images: whatever
    # kernel the planner takes, no lane loads a byte that belongs to no row of the call (harris.h excepts
    # only 8-bit rows off 4-byte boundaries, by whole words, in the other kernels).  And the groupings take
    # four pixels of two rows per thread, and stores are written through, only where that is measured faster.
    import subprocess
    csrc = os.path.join(ROOT, "paper_2212_12035_amd", "csrc")
    exe = str(tmp_path / "plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                    os.path.join(ROOT, "tests", "plan_check.cpp"), os.path.join(csrc, "harris_api.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout


def test_entry_points_validate_before_touching_the_device(pkg):
    # None of these reaches a kernel launch, so they are safe without a GPU.
    lib = pkg.load_library()
    nan = float("nan")
    one = ctypes.c_void_p(4096)
    assert lib.harris_coarsity(None, 1, 64, 64, 0.04, one, None) == -1
    assert lib.harris_coarsity(one, 1, 64, 64, 0.04, None, None) == -1
    assert lib.harris_coarsity(one, 1, 3, 64, 0.04, one, None) == -2
    assert lib.harris_coarsity(one, -1, 64, 64, 0.04, one, None) == -2
    assert lib.harris_coarsity(one, 1, 64, 64, nan, one, None) == -3
    assert lib.harris_coarsity_u8(one, 1, 64, 64, float("inf"), one, None) == -3
    assert lib.harris_coarsity_ex(one, 0, 1, 64, 64, 0.04, nan, 0, one, None, None) == -3
    assert lib.harris_coarsity_ex(one, 0, 1, 64, 64, 0.04, 1.0, 2, one, None, None) == -3
    assert lib.harris_coarsity_ex(one, 5, 1, 64, 64, 0.04, 1.0, 0, one, None, None) == -3
    assert lib.harris_coarsity_ex(one, 0, 1, 64, 64, 0.04, 1.0, 0, ctypes.c_void_p(4098), None, None) == -3  # out not 4-byte aligned
    # empty results succeed without looking at the pointers
    assert lib.harris_coarsity(None, 0, 64, 64, 0.04, None, None) == 0
    assert lib.harris_coarsity(None, 3, 4, 64, 0.04, None, None) == 0
    assert lib.harris_coarsity_u8(None, 3, 64, 4, 0.04, None, None) == 0


def test_grouped_workspace_sizes_and_validation(pkg):
    lib = pkg.load_library()
    H, W = 10, 12
    n0, n2, n4 = H * W, (H - 2) * (W - 2), (H - 4) * (W - 4)
    assert pkg.harris_grouped_workspace_bytes(1, 2, H, W) == 4 * 2 * (n0 + 5 * n2 + 3 * n4)
    assert pkg.harris_grouped_workspace_bytes(2, 2, H, W) == 4 * 2 * (n0 + 3 * n2)
    assert pkg.harris_grouped_workspace_bytes(3, 2, H, W) == 4 * 2 * (n0 + 2 * n2)
    assert pkg.harris_grouped_workspace_bytes(4, 2, H, W) == 0
    assert pkg.harris_grouped_workspace_bytes(5, 2, H, W) == -1 and pkg.harris_grouped_workspace_bytes(1, 2, 3, W) == -1
    one = ctypes.c_void_p(4096)
    need = pkg.harris_grouped_workspace_bytes(1, 1, H, W)
    assert lib.harris_coarsity_grouped(one, 0, 1, H, W, 0.04, 1.0, 0, 0, one, need, one, None) == -3      # grouping 0
    assert lib.harris_coarsity_grouped(one, 0, 1, H, W, 0.04, 1.0, 0, 1, one, need - 4, one, None) == -3  # workspace too small
    assert lib.harris_coarsity_grouped(one, 0, 1, H, W, 0.04, 1.0, 0, 1, None, need, one, None) == -1
    assert lib.harris_coarsity_grouped(one, 0, 1, 3, W, 0.04, 1.0, 0, 2, one, need, one, None) == -2
    assert lib.harris_coarsity_grouped(None, 0, 0, H, W, 0.04, 1.0, 0, 3, None, 0, None, None) == 0


def test_static_scratch_entry_rejects_what_does_not_fit(pkg):
    # Checked on the host before anything touches a device.
    lib = pkg.load_library()
    one = ctypes.c_void_p(4096)
    cap = pkg.HARRIS_GROUPED_SCRATCH_BYTES
    assert cap == 64 << 20
    assert pkg.harris_grouped_workspace_bytes(2, 1, 1536, 2560) <= cap < pkg.harris_grouped_workspace_bytes(1, 1, 1536, 2560)
    assert lib.harris_coarsity_grouped_static(one, 0, 1, 1536, 2560, 0.04, 1.0, 0, 1, one, None) == -5
    assert lib.harris_coarsity_grouped_static(one, 0, 64, 1080, 1920, 0.04, 1.0, 0, 3, one, None) == -5
    assert lib.harris_coarsity_grouped_static(one, 0, 2 ** 31 - 1, 2 ** 30, 2 ** 28, 0.04, 1.0, 0, 2, one, None) == -5
    assert lib.harris_coarsity_grouped_static(one, 0, 1, 64, 64, 0.04, 1.0, 0, 0, one, None) == -3      # grouping 0
    assert lib.harris_coarsity_grouped_static(one, 0, 1, 64, 64, 0.04, 1.0, 0, 5, one, None) == -3
    assert lib.harris_coarsity_grouped_static(one, 0, 1, 3, 64, 0.04, 1.0, 0, 1, one, None) == -2
    assert lib.harris_coarsity_grouped_static(None, 0, 1, 64, 64, 0.04, 1.0, 0, 1, one, None) == -1
    assert lib.harris_coarsity_grouped_static(None, 0, 0, 64, 64, 0.04, 1.0, 0, 2, None, None) == 0       # empty: no work, no scratch
    assert lib.harris_coarsity_grouped_static(None, 0, 3, 4, 64, 0.04, 1.0, 0, 3, None, None) == 0
    assert "scratch" in pkg.harris_strerror(-5)


def test_pitched_entry_validates_the_layout(pkg):
    lib = pkg.load_library()
    one = ctypes.c_void_p(4096)
    H, W = 10, 12

    def call(**kw):
        lay = dict(rgb_row_pitch=W, rgb_plane_pitch=H * W, rgb_image_pitch=3 * H * W, out_row_pitch=W - 4, out_image_pitch=(H - 4) * (W - 4))
        lay.update(kw)
        return lib.harris_coarsity_pitched(one, 0, 2, H, W, ctypes.byref(pkg.HarrisLayout(**lay)), 0.04, 1.0, 0, one, None, None)

    assert call(rgb_row_pitch=W - 1) == -2
    assert call(rgb_plane_pitch=H * W - 1) == -2
    assert call(rgb_image_pitch=3 * H * W - 1) == -2
    assert call(out_row_pitch=W - 5) == -2
    assert call(out_image_pitch=(H - 4) * (W - 4) - 1) == -2
    # padded rows need matching plane pitch
    assert call(rgb_row_pitch=W + 4) == -2
    # NULL layout means dense: same checks as harris_coarsity_ex
    assert lib.harris_coarsity_pitched(None, 0, 1, H, W, None, 0.04, 1.0, 0, one, None, None) == -1
    assert lib.harris_coarsity_pitched(None, 0, 0, H, W, None, 0.04, 1.0, 0, None, None, None) == 0


def test_product_sources_never_reach_for_the_oracle():
    # The oracle is test infrastructure: nothing under the package (or the headers) may name it.
    pkg_dir = os.path.join(ROOT, "paper_2212_12035_amd")
    for base, _, files in os.walk(pkg_dir):
        for name in files:
            if name.endswith((".py", ".hip", ".cpp", ".h")):
                text = open(os.path.join(base, name)).read()
                assert "oracle" not in text.lower(), os.path.join(base, name)
    for name in os.listdir(os.path.join(ROOT, "include")):
        assert "oracle" not in open(os.path.join(ROOT, "include", name)).read().lower()
    bench = open(os.path.join(ROOT, "bench.py")).read()
    assert "__graft_entry__" not in bench              # the benchmark builds the library by the package's own build step
    assert "paper_2212_12035_amd" not in open(os.path.join(ROOT, "oracle", "harris_oracle.py")).read()
    assert "harris.h" not in open(os.path.join(ROOT, "oracle", "harris_ref.cpp")).read()


def test_binding_refuses_host_tensors(pkg):
    import torch
    with pytest.raises(TypeError):
        pkg.harris_coarsity(torch.zeros(1, 3, 8, 8))


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_with_and_without_torchs_internal_function(pkg, monkeypatch, raw):
    # Without a GPU: torch's answers are stand-ins, the library function is caught.
    import types
    import torch
    if raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 100 + index, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=100 + device.index))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    calls = []

    def function(*args):
        calls.append([getattr(a, "value", a) for a in args])
        return 0

    device = torch.device("cuda", 3)
    pkg.binding._enqueue(function, device, None, 1, 2)
    pkg.binding._enqueue(function, device, 55, 1, 2)
    pkg.binding._enqueue(function, device, types.SimpleNamespace(cuda_stream=66), 1, 2)
    assert calls == [[1, 2, 103], [1, 2, 55], [1, 2, 66]]


@pytest.mark.parametrize("kind", ["none", "torch", "handle", "object", "null"])
def test_internal_workspace_is_allocated_in_the_order_of_the_launch_stream(pkg, monkeypatch, kind):
    # harris_coarsity_grouped gives its own workspace back to torch on return, with its kernels still
    # queued: only a block of the stream they run on is safe from being handed out before they end.
    # (Without a GPU: torch's streams are stand-ins, and the library call is caught.)
    import contextlib
    import types
    import torch

    class Stream:
        def __init__(self, handle, device=None):
            self.cuda_stream = handle

    current = [Stream(11)]
    used = []

    @contextlib.contextmanager
    def on(stream):
        before = current[0]
        if stream is not None:
            current[0] = stream
        yield
        current[0] = before

    def empty(*args, **kw):
        used.append(current[0].cuda_stream)
        return torch.zeros(args[0])

    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", Stream)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: Stream(0))
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch, "empty", empty)
    launched = []
    monkeypatch.setattr(pkg.binding, "_prepare", lambda rgb, out, dtype: (1, rgb.shape[2], rgb.shape[3], out))
    monkeypatch.setattr(pkg.binding, "_enqueue", lambda function, device, stream, *args: launched.append(stream))
    stream, handle = {"none": (None, 11), "torch": (Stream(22), 22), "handle": (33, 33),
                      "object": (types.SimpleNamespace(cuda_stream=44), 44), "null": (0, 0)}[kind]
    rgb = torch.zeros(1, 3, 8, 8)
    pkg.harris_coarsity_grouped(rgb, grouping=2, out=torch.zeros(1, 4, 4), stream=stream)
    assert used == [handle] and launched == [stream] and current[0].cuda_stream == 11
    pkg.harris_coarsity_grouped(rgb, grouping=2, workspace=torch.zeros(4096), out=torch.zeros(1, 4, 4), stream=stream)
    assert used == [handle] and launched == [stream, stream]     # the caller's workspace is the caller's


def test_sweep_candidates_are_launch_shapes_the_library_knows(pkg):
    # The launch-shape sweep times the planner's choice against candidates; every candidate must be a
    # shape harris_plan accepts or cleanly refuses (never one that would only fail at launch), the
    # default must come first, and for a one-tile-per-CU size the planner's own choice must be among them.
    from paper_2212_12035_amd import sweep
    for dtype in (pkg.HARRIS_F32, pkg.HARRIS_U8):
        for B, H, W in ((1, 1536, 2560), (1, 900, 1600), (4, 480, 640), (64, 1080, 1920), (1, 8192, 8192)):
            cands = sweep.candidates(pkg, dtype, B, H, W)
            assert cands[0][0] == "default" and len({name for name, _ in cands}) == len(cands)
            accepted = []
            for name, t in cands:
                try:
                    shape, blocks = pkg.harris_plan(dtype, B, H, W, tuning=t)
                    assert blocks > 0 and shape["schedule"] == pkg.HARRIS_SCHEDULE_TILES and shape["px"] == 4
                    accepted.append((shape["rows"], shape["waves_per_block"]))
                except pkg.HarrisError as e:
                    assert e.status == -3, name
            assert len(accepted) >= 8
    chosen = pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560)[0]
    shapes = [pkg.harris_plan(pkg.HARRIS_F32, 1, 1536, 2560, tuning=t)[0] for _, t in sweep.candidates(pkg, pkg.HARRIS_F32, 1, 1536, 2560)[1:]]
    assert any((s["rows"], s["waves_per_block"], s["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF) == (chosen["rows"], chosen["waves_per_block"], chosen["flags"] & pkg.HARRIS_TUNE_FLAG_HANDOFF) for s in shapes)


def test_plan_for_batches_of_narrow_images(pkg):
    # Images side by side in a wavefront: the launch must hold every image and every result row, whatever
    # the width, and the lanes' division by the lanes of an image (a multiplication) must be exact.
    for W in range(5, 140):
        lanes = (W + 3) // 4
        images = 64 // lanes
        inverse = (65535 + lanes) // lanes
        assert all((lane * inverse) >> 16 == lane // lanes for lane in range(64))
        for dtype in (pkg.HARRIS_F32, pkg.HARRIS_U8):
            for H in (5, 31, 32, 33, 60, 61, 64, 200):
                B = max((1 << 18) // (H * W), 768 // -(-(H - 4) // 12)) + 2
                shape, blocks = pkg.harris_plan(dtype, B, H, W)
                packed = images >= 2 and not (images == 2 and dtype == pkg.HARRIS_F32 and W % 4)
                assert shape["schedule"] == pkg.HARRIS_SCHEDULE_TILES and bool(shape["flags"] & pkg.HARRIS_TUNE_PACKED_IMAGES) == packed
                if not packed:
                    assert shape["flags"] & pkg.HARRIS_TUNE_STREAM_LOADS
                    continue
                assert shape["flags"] == pkg.HARRIS_TUNE_PACKED_IMAGES | pkg.HARRIS_TUNE_CACHED_LOADS | pkg.HARRIS_TUNE_PLAIN_STORES
                n, groups = H - 4, -(-B // images)
                assert shape["px"] == 4 and shape["rows"] == 4 and 2 <= shape["waves_per_block"] <= 8 and blocks % groups == 0
                bands = blocks // groups
                assert bands * 4 * (shape["waves_per_block"] - 1) >= n > (bands - 1) * -(-n // bands)
                # a caller's own shape, other result types and single images are not affected
                assert pkg.harris_plan(dtype, B, H, W, tuning=dict(rows=4, waves_per_block=4))[1] == B * -(-n // 12) * -(-(W - 4) // 252)
        assert pkg.harris_plan(pkg.HARRIS_F32, 1, 1 << 14, W)[1] != 0


def test_small_batches_of_narrow_images_keep_a_wavefront_each(pkg):
    # As long as one image per wavefront takes at most one tile of 12 result rows per CU (256), and for
    # two wide float32 images also where it takes three and the packed launch would have at most 128
    # workgroups: measured faster so (see the planner).
    def packed(dtype, B, H, W):
        return bool(pkg.harris_plan(dtype, B, H, W)[0]["flags"] & pkg.HARRIS_TUNE_PACKED_IMAGES)
    F32, U8 = pkg.HARRIS_F32, pkg.HARRIS_U8
    for dtype in (F32, U8):
        for B, H, W in ((20, 120, 128), (64, 32, 128), (5, 500, 128), (32, 100, 88), (85, 32, 96), (25, 120, 84)):
            assert not packed(dtype, B, H, W), (dtype, B, H, W)
        for B, H, W in ((26, 120, 88), (86, 32, 100), (64, 64, 64), (2048, 64, 64), (341, 24, 128), (8192, 32, 32)):
            assert packed(dtype, B, H, W), (dtype, B, H, W)
    assert not packed(F32, 256, 32, 128) and packed(U8, 256, 32, 128) and packed(F32, 258, 32, 128) and packed(F32, 228, 32, 96)


def test_benchmark_refuses_more_than_one_gpu():
    # The benchmark measures one GPU; asked for more it says so and exits before touching a device.
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one GPU" in (r.stdout + r.stderr) and "{" not in r.stdout


def test_traffic_figures_belong_to_the_kernels_in_the_tree():
    # roofline.traffic is reported only while the kernel sources hash to the value recorded with
    # the counters; after a change to the kernels the figure must be re-measured, not carried over.
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    sys.path.insert(0, root)
    import bench
    assert set(bench.TRAFFIC_BYTES) == {"noise_f32_1536x2560", "rects_f32_64x1080x1920", "blobs_f32_2832x4256", "noise_u8_8192x8192"}
    assert len(bench.TRAFFIC_SOURCES_SHA256) == 64 and len(bench.kernel_sources_sha256()) == 64
    for name, traffic in bench.TRAFFIC_BYTES.items():
        # measured HBM bytes lie between the algorithmic bytes and 1.15 times them
        import harris_inputs
        gen, seed, B, H, W, dt = harris_inputs.WORKLOADS[name]
        algo = B * (3 * H * W * (1 if dt == "u8" else 4) + 4 * (H - 4) * (W - 4))
        assert algo <= traffic <= 1.15 * algo, name
