"""The matrix-core distance kernel over its tile sizes (32, 64 and 128 rows and more), group sizes and step
counts: the packed kernel, whose tiles stay large, gives the same bits on every one."""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import select_paths

pytestmark = pytest.mark.gpu

knn = pytest.importorskip("paper_2405_19325_amd")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    knn.load()
    yield
    torch.cuda.synchronize()


# queries per set, keys per set, d.  One set: up to 8,192 keys take 32-row tiles, up to 16,384 (32,768 for up to
# 32 queries) 64-row ones, more 128-row ones; steps per row 1 to 9 (of 128 elements) and 2 to 18 (of 64), so
# that the padding of the step count is 0 to 3; rows that end inside a pass, a block, a tile; several groups.
CASES = [(q, n, d) for q in (16, 20, 40, 100, 130) for n, d in (
    ((1, 31), 128), ((3001,), 384), ((8192,), 256), ((8193,), 640), ((16385,), 128), ((33000,), 384),
    ((300, 0, 5007, 17), 1152))]


@pytest.mark.parametrize("norms", [False, True], ids=["own-norms", "given-norms"])
@pytest.mark.parametrize("q,sizes,d", CASES)
def test_bits_of_the_packed_kernel(q, sizes, d, norms):
    dtype = torch.bfloat16 if d % 256 else torch.float16
    print(f"[gpu] batch tiles q={q} {sizes} d={d} norms={norms}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(q + d)
    S, n, V, r = len(sizes), sum(sizes), 500, min(min(s for s in sizes if s), 64)
    ko = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rows = [q if s else 0 for s in sizes]
    if S > 1:
        rows[-1] = q - 3
    qo = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    k = (torch.randn((n, d), generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype)
    x = (torch.randn((int(qo[-1]), d), generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype)
    tko, tqo = torch.from_numpy(ko).cuda(), torch.from_numpy(qo).cuda()
    packed = knn.pack_keys(k)
    kn = knn.key_sqnorms(k) if norms else None
    args = dict(key_sqnorms=kn, key_offsets_host=ko, query_offsets_host=qo)
    one, two = knn.distances(x, k, tko, tqo, **args), knn.distances(x, k, tko, tqo, packed_keys=packed, **args)
    assert torch.equal(one.view(torch.int32), two.view(torch.int32))  # NaN past every set included
    values = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    p_lm = torch.softmax(torch.randn(x.shape[0], V, generator=g, device="cuda"), 1)
    mask = knn.mask_words(np.arange(0, n, 5), n, "cuda")
    outs = []
    for pk in (None, packed):
        prob = knn.MixtureProblem(x, k, values, tko, tqo, p_lm, r, packed_keys=pk, **args)
        outs.append(prob.run_nest(0.3, 0.1, 0.5, key_mask=mask))
    for name in ("ids", "dists", "lambdas"):
        assert torch.equal(outs[0][name], outs[1][name]), name
    torch.testing.assert_close(outs[0]["p_m"], outs[1]["p_m"], rtol=1e-5, atol=1e-8)


# Stores large enough for tiles of whole 256-row passes, which groups of more than 64 queries take: 4 to 20 steps a
# tile (the step count padded to a multiple of three by 0, 1 and 2), one pass a tile and several, two query groups.
@pytest.mark.parametrize("norms", [False, True], ids=["own-norms", "given-norms"])
@pytest.mark.parametrize("q,S,n,d", [(100, 4, 66001, 256), (128, 3, 66057, 384), (70, 20, 20001, 128),
                                     (130, 3, 40003, 640), (66, 1, 300100, 512)])
def test_bits_of_the_packed_kernel_in_256_row_passes(q, S, n, d, norms):
    print(f"[gpu] 256-row passes q={q} S={S} n={n} d={d} norms={norms}", flush=True)
    assert select_paths.route(q * S, d, 2, S, n, q, 64).tile_rows % 256 == 0
    g = torch.Generator(device="cuda").manual_seed(q + d)
    ko, qo = np.arange(S + 1, dtype=np.int64) * n, np.arange(S + 1, dtype=np.int64) * q
    k, x = ((torch.randn((m, d), generator=g, device="cuda") * (8 / math.sqrt(d))).half() for m in (S * n, S * q))
    args = dict(key_sqnorms=knn.key_sqnorms(k) if norms else None, key_offsets_host=ko, query_offsets_host=qo)
    tko, tqo = torch.from_numpy(ko).cuda(), torch.from_numpy(qo).cuda()
    one, two = (knn.distances(x, k, tko, tqo, packed_keys=p, **args) for p in (None, knn.pack_keys(k)))
    assert torch.equal(one.view(torch.int32), two.view(torch.int32))


def test_workspace_of_both_key_layouts():
    """One workspace size serves a batch on row-major and on packed keys, finer tiles or not."""
    lib = knn.load()
    for q, n in ((16, 3001), (40, 8193), (130, 33000), (16, 262144)):
        for size in (lib.knn_lm_mixture_workspace_size, lib.knn_lm_mixture_workspace_preferred):
            a, b = (size(q, 1024, 500, 1, n, n, n, q, dt, 64)
                    for dt in (knn.DTYPES["bf16"], knn.DTYPES["bf16"] | knn.KEYS_PACKED))
            assert a == b > 0
