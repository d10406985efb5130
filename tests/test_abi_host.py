"""Host-side checks of the C ABI (no GPU needed): the library loads, exports every
function include/knnlm.h declares, and rejects bad arguments before enqueuing
anything."""
import ctypes
import os
import random

import pytest

from paper_2405_19325_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "knnlm.h")

OK, INVALID, R_EXCEEDS_N, UNSUPPORTED, WORKSPACE, HIP = range(6)


@pytest.fixture(scope="module")
def lib():
    return _lib.load()


def test_exports_every_declared_function(lib):
    names = _lib.header_functions(HEADER)
    assert len(names) >= 9
    for n in names:
        assert hasattr(lib, n), n
        assert n in _lib.SIGNATURES, f"{n} declared in the header but not bound"
    assert set(_lib.SIGNATURES) == set(names)


def test_abi_version_and_status_strings(lib):
    assert lib.knn_abi_version() == 2
    for s in range(6):
        assert lib.knn_status_string(s).decode()
    assert lib.knn_status_string(99).decode() == "unknown status"


# A valid decode-shaped call: B=1, d=4096, V=32000, one set of 65536 keys, r=1024.
BASE = dict(B=1, d=4096, V=32000, S=1, total_keys=65536, min_keys=65536, max_keys=65536, max_queries=1,
            dtype=1, r=1024, mu=1 / 64, lam=0.3)
FAKE = 1 << 20  # a non-null pointer value; validation never dereferences it


def _ws_size(lib, a):
    return lib.knn_lm_mixture_workspace_size(a["B"], a["d"], a["V"], a["S"], a["total_keys"], a["min_keys"],
                                             a["max_keys"], a["max_queries"], a["dtype"], a["r"])


def _validate(lib, ws=FAKE, ws_bytes=None, nulls=(), **over):
    a = dict(BASE, **over)
    if ws_bytes is None:
        ws_bytes = _ws_size(lib, dict(BASE)) + 0
    ptr = {n: (None if n in nulls else FAKE) for n in
           ("queries", "keys", "values", "key_offsets", "query_offsets", "p_lm", "p_m", "ids", "dists")}
    return lib.knn_lm_mixture_validate(ptr["queries"], ptr["keys"], ptr["values"], ptr["key_offsets"],
                                       ptr["query_offsets"], ptr["p_lm"], a["B"], a["d"], a["V"], a["S"],
                                       a["total_keys"], a["min_keys"], a["max_keys"], a["max_queries"], a["dtype"],
                                       a["r"], a["mu"], a["lam"], ptr["p_m"], ptr["ids"], ptr["dists"], ws, ws_bytes)


def test_valid_call_validates(lib):
    assert _ws_size(lib, BASE) > 65536 * 4
    assert _validate(lib) == OK


@pytest.mark.parametrize("over,expect", [
    (dict(r=0), INVALID), (dict(r=-3), INVALID), (dict(B=0), INVALID), (dict(d=0), INVALID),
    (dict(V=0), INVALID), (dict(S=0), INVALID), (dict(dtype=7), INVALID), (dict(mu=0.0), INVALID),
    (dict(mu=-1.0), INVALID), (dict(mu=float("nan")), INVALID), (dict(mu=float("inf")), INVALID),
    (dict(lam=-0.01), INVALID), (dict(lam=1.01), INVALID), (dict(lam=float("nan")), INVALID),
    (dict(min_keys=70000), INVALID), (dict(max_keys=70000), INVALID), (dict(max_queries=2), INVALID),
    (dict(max_queries=0), INVALID), (dict(r=65537), UNSUPPORTED), (dict(r=4097), UNSUPPORTED),
    (dict(min_keys=1000, r=1001), R_EXCEEDS_N), (dict(min_keys=0), R_EXCEEDS_N),
])
def test_rejects_bad_scalars(lib, over, expect):
    assert _validate(lib, **over) == expect


def test_lambda_and_r_edges_accepted(lib):
    assert _validate(lib, lam=0.0) == OK
    assert _validate(lib, lam=1.0) == OK
    assert _validate(lib, r=1) == OK
    assert _validate(lib, r=4096) == OK


@pytest.mark.parametrize("null", ["queries", "keys", "values", "key_offsets", "query_offsets", "p_lm", "p_m", "ids",
                                  "dists"])
def test_rejects_null_pointers(lib, null):
    assert _validate(lib, nulls=(null,)) == INVALID


def test_workspace_checks(lib):
    need = _ws_size(lib, BASE)
    assert _validate(lib, ws=None) == WORKSPACE
    assert _validate(lib, ws_bytes=need - 1) == WORKSPACE
    assert _validate(lib, ws=FAKE + 8) == WORKSPACE  # not 256-byte aligned
    assert _validate(lib, ws_bytes=need) == OK


def test_workspace_size_zero_for_invalid_sizes(lib):
    assert _ws_size(lib, dict(BASE, r=0)) == 0
    assert _ws_size(lib, dict(BASE, min_keys=10)) == 0


def test_entry_points_reject_before_touching_the_device(lib):
    # Invalid arguments return an error code without any HIP call, so these run without a GPU.
    a = BASE
    st = lib.knn_lm_mixture(FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, a["B"], a["d"], a["V"], a["S"],
                            a["total_keys"], a["min_keys"], a["max_keys"], a["max_queries"], a["dtype"], 0, a["mu"],
                            a["lam"], FAKE, FAKE, FAKE, FAKE, 1 << 30, None)
    assert st == INVALID
    st = lib.knn_lm_mixture_part(9, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, a["B"], a["d"], a["V"], a["S"],
                                 a["total_keys"], a["min_keys"], a["max_keys"], a["max_queries"], a["dtype"], 16,
                                 a["mu"], a["lam"], FAKE, FAKE, FAKE, FAKE, 1 << 30, None)
    assert st == INVALID
    assert lib.knn_key_sqnorms(None, 10, 8, 1, FAKE, None) == INVALID
    assert lib.knn_key_sqnorms(FAKE, 10, 0, 1, FAKE, None) == INVALID
    assert lib.knn_mix(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 100, 1, 8, 0.1, 2.0, FAKE, None) == INVALID
    assert lib.knn_mix(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 100, 1, 5000, 0.1, 0.5, FAKE, None) == UNSUPPORTED
    assert lib.knn_distances(FAKE, FAKE, None, FAKE, FAKE, 1, 64, 1, 100, 1, 1, FAKE, 99, None) == INVALID


def test_mixture_part_stage_pointer_rules(lib):
    # The mix stage needs no workspace and no queries/keys; distances needs no outputs.
    a = BASE
    args = lambda part, q, k, ws, pm, ids: lib.knn_lm_mixture_part(
        part, q, k, None, FAKE, FAKE, FAKE, FAKE, a["B"], a["d"], a["V"], a["S"], a["total_keys"], a["min_keys"],
        a["max_keys"], a["max_queries"], a["dtype"], a["r"], float("nan"), a["lam"], pm, ids, ids, ws, 0, None)
    # distances stage with a null workspace: rejected
    assert args(1, FAKE, FAKE, None, None, None) == WORKSPACE
    # select stage with null outputs: rejected
    assert args(2, None, None, FAKE, None, None) == INVALID
    # mix stage: mu = NaN is rejected
    assert args(3, None, None, None, FAKE, FAKE) == INVALID


BF16_PACKED, F16_PACKED, KEYS_PACKED = 0x101, 0x102, 0x100


def test_packed_keys_bytes(lib):
    # blocks of 16 rows, each 32 d bytes of fragments then 16 fp32 norms
    assert lib.knn_packed_keys_bytes(16, 128, 1) == 32 * 128 + 64
    assert lib.knn_packed_keys_bytes(17, 128, 2) == 2 * (32 * 128 + 64)
    assert lib.knn_packed_keys_bytes(8388608, 1024, 2) == 8388608 // 16 * (32 * 1024 + 64)
    assert lib.knn_packed_keys_bytes(1000, 256, BF16_PACKED) == 63 * (32 * 256 + 64)  # the flag is ignored here
    for n, d, t in ((0, 128, 1), (16, 0, 1), (16, 128, 0), (16, 192, 1), (16, 65536 + 128, 1), (16, 128, 7)):
        assert lib.knn_packed_keys_bytes(n, d, t) == 0, (n, d, t)


def test_pack_keys_rejects_before_touching_the_device(lib):
    assert lib.knn_pack_keys(None, 16, 128, 1, FAKE, None) == INVALID
    assert lib.knn_pack_keys(FAKE, 16, 128, 1, None, None) == INVALID
    assert lib.knn_pack_keys(FAKE, 0, 128, 1, FAKE, None) == INVALID
    assert lib.knn_pack_keys(FAKE + 8, 16, 128, 1, FAKE, None) == INVALID  # not 16-byte aligned
    assert lib.knn_pack_keys(FAKE, 16, 128, 0, FAKE, None) == UNSUPPORTED  # fp32
    assert lib.knn_pack_keys(FAKE, 16, 192, 1, FAKE, None) == UNSUPPORTED  # d % 128 != 0


def test_packed_dtype_validation(lib):
    # a batch the matrix cores serve: 128 queries on one set of 65536 keys at d = 1024
    mc = dict(B=128, d=1024, max_queries=128, min_keys=65536, max_keys=65536)
    ws = _ws_size(lib, dict(BASE, **mc))
    assert _validate(lib, ws_bytes=ws, dtype=2, **mc) == OK
    assert _validate(lib, ws_bytes=ws, dtype=F16_PACKED, **mc) == OK
    assert _validate(lib, ws_bytes=ws, dtype=BF16_PACKED, **mc) == OK
    assert _ws_size(lib, dict(BASE, dtype=F16_PACKED, **mc)) == ws
    # fp32 keys cannot be packed; the flag on its own is no element type
    assert _validate(lib, ws_bytes=ws, dtype=KEYS_PACKED, **mc) == INVALID
    # fewer than 16 queries per set (the streaming kernel), or d % 128 != 0: not served packed
    assert _validate(lib, dtype=BF16_PACKED) == UNSUPPORTED
    mc_odd = dict(mc, d=1000)
    assert _validate(lib, ws_bytes=_ws_size(lib, dict(BASE, **mc_odd)), dtype=BF16_PACKED, **mc_odd) == UNSUPPORTED
    # the select and mix stages read no keys: the flag changes nothing there
    a = dict(BASE, **mc)
    st = lib.knn_lm_mixture_part(3, None, None, None, FAKE, FAKE, FAKE, FAKE, a["B"], a["d"], a["V"], a["S"],
                                 a["total_keys"], a["min_keys"], a["max_keys"], a["max_queries"], BF16_PACKED,
                                 a["r"], a["mu"], a["lam"], FAKE, FAKE, FAKE, None, 0, None)
    assert st == OK or st == HIP  # validated; the launch itself needs a GPU
    # knn_distances: packed keys with a streaming-path batch are refused
    assert lib.knn_distances(FAKE, FAKE, None, FAKE, FAKE, 1, 1024, 1, 100, 1, BF16_PACKED, FAKE, 100, None) == \
        UNSUPPORTED
    assert lib.knn_distances(FAKE, FAKE, None, FAKE, FAKE, 16, 1024, 1, 100, 16, KEYS_PACKED, FAKE, 100, None) == \
        INVALID


def test_routes_at_the_edges_of_their_rules():
    """The distance kernel, its tiles and the select path at the sizes where the host code changes them."""
    from select_paths import route

    # decode shape: 32-row tiles, 8192 groups of 8 rows: on for every r <= 1024
    assert route(1, 4096, 1, 1, 65536, 1, 1024)[:2] == ("streaming", 32)
    assert route(1, 4096, 1, 1, 65536, 1, 1024, 32000)[3:] == ("groups", 16, 8)
    # 4096 keys in 16-row tiles: 1024 groups of 4 rows, so r <= 819 (5/4 r); of the shortest row
    assert route(1, 4096, 1, 1, 4096, 1, 819, 32000)[3:] == ("groups", 1, 4)
    assert route(1, 4096, 1, 1, 4096, 1, 820, 32000)[3:] == ("parts", 1, 0)
    assert route(2, 4096, 1, 2, 4096, 1, 513, 32000, min_keys=2564)[3:] == ("parts", 1, 0)
    assert route(2, 4096, 1, 2, 4096, 1, 513, 32000, min_keys=2568)[3:] == ("groups", 1, 4)
    # a vocabulary of more slices than the chip takes at once: no group minima
    assert route(2, 16, 0, 1, 40000, 2, 1024, 600001).select == "parts"
    assert route(2, 16, 0, 1, 40000, 2, 1024).select == "groups"
    # 16 bf16 queries on a set take the matrix cores: no group minima
    assert route(16, 4096, 1, 1, 4096, 16, 512)[3:] == ("parts", 1, 0)
    # 64-row tiles (many sets): the parts kernel samples the rows
    assert route(32, 256, 1, 32, 4096, 1, 256, 32000)[1:] == (64, 1, "parts", 1, 0)
    # 1024 parts over all rows, then one workgroup a row of the sampled select; r = 1024 is the split select's most
    assert route(64, 16, 0, 1, 65536, 64, 1024, 32000)[3:5] == ("parts", 16)
    assert route(65, 16, 0, 1, 65536, 65, 1024, 32000).select == "one-workgroup"
    assert route(65, 16, 0, 1, 65537, 65, 1024, 32000)[3:5] == ("wide", 4)
    assert route(600, 16, 0, 1, 32768, 600, 1024, 32000)[3:5] == ("sampled", 1)
    assert route(600, 16, 0, 1, 32769, 600, 1024, 32000).select == "one-workgroup"
    # more than two parts a CU, no more rows than CUs, of at most 32768 keys: one workgroup a row
    assert route(64, 16, 0, 1, 32768, 64, 1024, 64001).select == "parts"
    assert route(65, 16, 0, 1, 32768, 65, 1024, 64001).select == "one-workgroup"
    assert route(65, 16, 0, 1, 32768, 65, 1024, 1000).select == "groups"
    assert route(256, 16, 0, 1, 12288, 256, 1024, 64001).select == "one-workgroup"
    assert route(257, 16, 0, 1, 12288, 257, 1024, 64001).select == "parts"
    # rows of one part and a large vocabulary: fixed lambda from 257 rows on, the rest past 1024
    for rows, mode, V, want in ((256, "fixed", 32000, "parts"), (257, "fixed", 32000, "one-workgroup"),
                                (257, "fixed", 16384, "parts"), (257, "nest", 32000, "parts"),
                                (1025, "nest", 32000, "one-workgroup"), (1025, "fixed", 16384, "sampled")):
        assert route(rows, 16, 0, 1, 4096, rows, 1000, V, mode=mode).select == want, (rows, mode, V)
    assert route(1025, 16, 0, 1, 4097, 1025, 1000, 32000).select == "sampled"
    assert route(3, 16, 0, 1, 40000, 3, 1025).select == "sampled"
    assert route(3, 16, 0, 1, 40000, 3, 2049).select == "general"
    # 128-query batches on long rows: fused where the rows hold 2 r coarse tiles (1024 rows at d = 1024, 256 at
    # d = 4096), which the finer tiles of shorter rows don't count for
    assert route(128, 1024, 2, 1, 131072, 128, 64)[1::2] == (1024, "fused", 0)
    assert route(128, 1024, 2, 1, 130048, 128, 64)[1::2] == (128, "wide", 0)
    assert route(128, 4096, 1, 1, 65800, 128, 64)[1::2] == (256, "fused", 0)
    assert route(128, 128, 1, 1, 65800, 128, 64).select != "fused"
    # several queries a set: enough rows to read in all, and in each set where the sets outnumber the shares
    def kernel(sets, keys, queries, d, dtype=1):
        return route(sets * queries, d, dtype, sets, keys, queries, min(keys, 16)).kernel

    assert [kernel(1, n, 8, 256) for n in (9999, 10000)] == ["streaming", "several-queries"]
    assert [kernel(1, n, 8, 4096) for n in (2499, 2500)] == ["streaming", "several-queries"]  # four passes of two
    assert [kernel(s, 100, 8, 256) for s in (256, 257)] == ["several-queries", "streaming"]
    assert [kernel(4096, n, 8, 256) for n in (16, 171, 172)] == ["streaming", "streaming", "several-queries"]
    assert [kernel(4096, n, 6, 256, 0) for n in (149, 150)] == ["streaming", "several-queries"]
    assert [kernel(s, 64, 40, 1000) for s in (80, 81)] == ["several-queries", "streaming"]  # three query groups
    assert kernel(4096, 128, 40, 1000) == "several-queries"
    assert kernel(4096, 1000, 4, 256) == "streaming"  # one pass of four
    # a workspace that holds no lists: one workgroup a row
    assert route(65, 16, 0, 1, 65536, 65, 1024, workspace_bytes=0).select == "one-workgroup"
    assert route(3, 16, 0, 1, 40000, 3, 1025, 100, workspace_bytes=0).select == "general"
    assert route(17, 16, 0, 1, 65536, 17, 1024, workspace_bytes=0).select == "one-workgroup"
    assert route(16, 16, 0, 1, 65536, 16, 1024, workspace_bytes=0).select == "groups"
    assert route(3, 16, 0, 1, 40000, 3, 2048, workspace_bytes=0).select == "general"


def _preferred(lib, a):
    return lib.knn_lm_mixture_workspace_preferred(a["B"], a["d"], a["V"], a["S"], a["total_keys"], a["min_keys"],
                                                  a["max_keys"], a["max_queries"], a["dtype"], a["r"])


def test_workspace_size_is_the_least_accepted(lib):
    """A workspace of knn_lm_mixture_workspace_size() is accepted and a byte less refused, of query batches on small
    row-major stores (whose finer tiles need less) and of rows whose larger selects want more, too."""
    rng = random.Random(5)
    for _ in range(2000):
        S = rng.choice([1, 2, 8, 60, 1000])
        keys = int(2 ** rng.uniform(3, 18))
        q = int(2 ** rng.uniform(0, 8))
        d = rng.choice([8, 128, 384, 1000, 1024, 4096, 8192])
        few = max(1, int(keys * rng.uniform(0.3, 1)))
        a = dict(BASE, B=S * q, d=d, S=S, total_keys=S * keys, min_keys=few, max_keys=keys, max_queries=q,
                 dtype=rng.choice([0, 1, 2]), r=rng.choice([1, 64, 1000, 1024, 2048, 4096]))
        a["r"] = min(a["r"], few)
        size, most = _ws_size(lib, a), _preferred(lib, a)
        assert 0 < size <= most, a
        kw = {k: a[k] for k in a if k not in ("mu", "lam")}
        assert _validate(lib, ws_bytes=size, **kw) == OK and _validate(lib, ws_bytes=most, **kw) == OK, a
        assert _validate(lib, ws_bytes=size - 1, **kw) == WORKSPACE, a
        if a["dtype"] != 0:
            assert _preferred(lib, dict(a, dtype=a["dtype"] | KEYS_PACKED)) == most, a


def test_workspace_sizes_of_the_header_examples(lib):
    """The static scratch array serves what the header says, by the size that it gates on."""
    scratch = 32 << 20
    long_rows = dict(BASE, B=64, S=64, total_keys=64 * 65536)
    assert 16 << 20 < _ws_size(lib, long_rows) < 17 << 20
    assert 48 << 20 < _preferred(lib, long_rows) < 49 << 20
    wide = dict(BASE, B=16, d=8192, S=16, total_keys=16 * 131072, min_keys=131072, max_keys=131072)
    assert _ws_size(lib, wide) <= scratch
    many = dict(BASE, B=20000, d=256, S=2000, total_keys=2000 * 10000, min_keys=10000, max_keys=10000, max_queries=10)
    assert 760 << 20 < _ws_size(lib, many) < 790 << 20 and 1400 << 20 < _preferred(lib, many) < 1415 << 20
    assert _preferred(lib, dict(BASE, r=0)) == 0


def test_stages_agree_on_what_lies_between_them():
    """What one stage leaves for another does not depend on the workspace's size, on the key layout or on the
    shortest row."""
    from select_paths import route

    rng = random.Random(6)
    seen = set()
    for _ in range(3000):
        S, q, d = rng.choice([1, 2, 8, 60, 1000]), int(2 ** rng.uniform(0, 8)), rng.choice([16, 128, 1000, 1024, 4096])
        keys, dtype = int(2 ** rng.uniform(5, 18)), rng.choice([0, 1, 2])
        r = min(rng.choice([16, 64, 1000, 1024, 2048]), keys)
        args = (S * q, d, dtype, S, keys, q, r, rng.choice([None, 1000, 32000]))
        one = route(*args, stage=True)
        others = [route(*args, stage=True, workspace_bytes=0), route(*args, min_keys=r, stage=True)]
        if one.kernel == "matrix-core":
            others.append(route(*args[:2], dtype | KEYS_PACKED, *args[3:], stage=True))
        for o in others:
            assert (o.tile_rows, o.group_rows, o.select == "fused") == (one.tile_rows, one.group_rows,
                                                                       one.select == "fused"), args
        seen.add((one.tile_rows == route(*args).tile_rows, one.group_rows == route(*args).group_rows))
    assert seen >= {(True, True), (False, True), (True, False)}  # whole calls differ in either


@pytest.mark.parametrize("rows,keys,r", [(100_000, 1000, 64), (100_000, 4096, 1024), (10_000, 1000, 1000), (4096, 1000, 64)])
def test_lists_of_many_short_rows_are_bounded(lib, rows, keys, r):
    """A select's candidate lists take at most 128 MiB, or no more than the distances, the group minima and
    extrema a tenth of those."""
    S = rows // 10
    size = _preferred(lib, dict(BASE, B=rows, d=256, S=S, total_keys=keys * S, min_keys=keys, max_keys=keys,
                              max_queries=10, r=r))
    dist = 4 * rows * (keys + 256)  # the row rounded up to its tiles of at most 256
    assert dist * keys // (keys + 256) < size < 1.2 * dist + max(dist, 129 << 20)
