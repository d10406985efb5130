"""The streaming distance kernel for a few queries per key set: every distance carries the bits of the
one-query kernel's, over its group sizes, remainders, element types, given norms, masks and ragged sets."""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import select_paths

pytestmark = pytest.mark.gpu

knn = pytest.importorskip("paper_2405_19325_amd")

DTYPES = {torch.float32: 0, torch.bfloat16: 1, torch.float16: 2}


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    knn.load()
    yield
    torch.cuda.synchronize()


def _batch(rows, sizes, d, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    ko = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    qo = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    k = (torch.randn((int(ko[-1]), d), generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype).contiguous()
    q = (torch.randn((int(qo[-1]), d), generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype).contiguous()
    q[0] = k[min(5, k.shape[0] - 1)]  # a query equal to a key
    return q, k, ko, qo


def _dev(x):
    return torch.from_numpy(np.asarray(x, np.int64)).cuda()


# queries per set, keys per set, d -- each with keys enough for the multi-query kernel (key rows times the
# streaming kernel's passes >= 10,000): group sizes 2, 4, 8 and 16 and several groups; one step a row and many;
# a row's last step whole and partly past it; sets that end inside a tile and a wave's four rows, one key, no
# key, no query; more sets than lanes; more tiles than a workgroup keeps extrema of.
CASES = [
    ("2q-wide", (2,), (5003,), 8192), ("4q", (4, 3), (2513, 2050), 4096), ("8q-ragged", (5, 0, 8, 1), (3000, 64, 1, 1601), 1000),
    ("8q-wide", (8, 6), (701, 660), 8192), ("9q", (9,), (3501,), 2048), ("15q", (15, 2), (4099, 31), 256),
    ("12q-two-groups", (12,), (910,), 8192),
    ("70 sets", tuple(1 + i % 6 for i in range(70)), tuple(1 + 7 * (i % 31) for i in range(70)), 768),
    ("300 sets", tuple(i % 6 for i in range(300)), tuple(1 + 8 * (i % 51) for i in range(300)), 256),
    ("empty set", (2, 0, 2), (1700, 0, 1709), 5120), ("64q-segments", (64,), (40000,), 8),
]


@pytest.mark.parametrize("norms", [False, True], ids=["own-norms", "given-norms"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("name,rows,sizes,d", CASES, ids=[c[0] for c in CASES])
def test_bits_of_one_query(name, rows, sizes, d, dtype, norms):
    if dtype == torch.float32:
        d = min(d, 4096)
    print(f"[gpu] multi {name} {dtype} norms={norms} d={d}", flush=True)
    assert select_paths.route(sum(rows), d, DTYPES[dtype], len(sizes), max(sizes), max(rows), 1).kernel == \
        "several-queries"
    q, k, ko, qo = _batch(rows, sizes, d, dtype, 7 + d)
    kn = knn.key_sqnorms(k) if norms else None
    got = knn.distances(q, k, _dev(ko), _dev(qo), key_sqnorms=kn, key_offsets_host=ko, query_offsets_host=qo)
    for s in range(len(sizes)):
        k0, k1 = int(ko[s]), int(ko[s + 1])
        for b in range(int(qo[s]), int(qo[s + 1])):
            if k1 == k0:
                continue
            one = knn.distances(q[b:b + 1], k[k0:k1], _dev([0, k1 - k0]), _dev([0, 1]),
                                key_sqnorms=kn[k0:k1] if norms else None)
            assert torch.equal(got[b, :k1 - k0].view(torch.int32), one[0].view(torch.int32)), (s, b)
            assert torch.isnan(got[b, k1 - k0:]).all()  # past the set: untouched
    if k.shape[0] > 5 and sizes[0] > 5:
        assert got[0, 5] == 0.0


@pytest.mark.parametrize("name,rows,sizes,d,dtype,r", [
    ("groups", (5, 6), (5100, 4200), 512, torch.bfloat16, 64), ("tiles", (7, 5), (2500, 3000), 4096, torch.float16, 1000),
    ("fp32", (20,), (3601,), 256, torch.float32, 300), ("long", (10,), (70000,), 128 + 8, torch.bfloat16, 256),
], ids=["groups", "tiles", "fp32", "long"])
def test_step_of_one_query(name, rows, sizes, d, dtype, r):
    """The masked decoding step over several queries a set selects what one-query steps select."""
    print(f"[gpu] multi step {name} {dtype}", flush=True)
    q, k, ko, qo = _batch(rows, sizes, d, dtype, 11 + d)
    n, V = k.shape[0], 1000
    g = torch.Generator(device="cuda").manual_seed(3)
    values = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    p_lm = torch.softmax(torch.randn(q.shape[0], V, generator=g, device="cuda"), 1)
    masked = np.arange(0, n, 3)
    mask = knn.mask_words(masked, n, "cuda")
    prob = knn.MixtureProblem(q, k, values, _dev(ko), _dev(qo), p_lm, r)
    out = {a: b.clone() for a, b in prob.run_nest(0.3, 0.1, 0.5, key_mask=mask).items()}
    for s in range(len(sizes)):
        k0, k1 = int(ko[s]), int(ko[s + 1])
        m1 = knn.mask_words(masked[(masked >= k0) & (masked < k1)] - k0, k1 - k0, "cuda")
        for b in range(int(qo[s]), int(qo[s + 1])):
            one = knn.MixtureProblem(q[b:b + 1], k[k0:k1], values[k0:k1], _dev([0, k1 - k0]), _dev([0, 1]),
                                     p_lm[b:b + 1].contiguous(), r).run_nest(0.3, 0.1, 0.5, key_mask=m1)
            assert torch.equal(out["ids"][b], one["ids"][0]) and torch.equal(out["dists"][b], one["dists"][0])
            assert torch.equal(out["lambdas"][b], one["lambdas"][0])
            torch.testing.assert_close(out["p_m"][b], one["p_m"][0], rtol=1e-5, atol=1e-8)
            assert not (out["ids"][b] % 3 == (-k0) % 3).any()
