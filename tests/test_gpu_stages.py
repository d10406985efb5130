"""The stages run one at a time, each told another workspace size and key layout, a select several times after one
distance stage: the neighbours and distances of the whole call, bit for bit."""
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


# queries and keys per set, d, dtype, r, V, packed keys, the select of the whole call
CASES = {
    "finer tiles": (20, (3001, 2000), 384, torch.bfloat16, 64, 500, False, "parts"),
    "packed": (20, (3001, 2000), 384, torch.bfloat16, 64, 500, True, "parts"),
    "finer tiles, long rows": (100, (70001,), 128, torch.float16, 64, 500, False, "wide"),
    "groups, 2 r of them": (2, (9000, 7437), 16, torch.float32, 1000, 5001, False, "groups"),
    "groups, 5/4 r of them": (2, (5200, 7437), 16, torch.float32, 1024, 5001, False, "groups"),
    "groups, 5/4 r of them, whole rows": (2, (5200, 7437), 16, torch.float32, 1024, 270001, False, "parts"),
    "groups, 320 parts": (40, (8000, 5000, 4097, 7999), 64, torch.float32, 1000, 1000, False, "groups"),
    "sampled": (20, (262144,), 128, torch.bfloat16, 1024, 1003, False, "sampled"),
    "fused": (66, (600000,), 128, torch.bfloat16, 64, 500, False, "fused"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_stages_of_unlike_workspaces(name):
    q, sizes, d, dtype, r, V, packs, want = CASES[name]
    print(f"[gpu] stages: {name}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(q + d + r)
    S, n = len(sizes), sum(sizes)
    ko = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    qo = np.arange(S + 1, dtype=np.int64) * q
    k, x = ((torch.randn(m, d, generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype) for m in (n, S * q))
    values = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    p_lm = torch.softmax(torch.randn(S * q, V, generator=g, device="cuda"), 1)
    prob = knn.MixtureProblem(x, k, values, torch.from_numpy(ko).cuda(), torch.from_numpy(qo).cuda(), p_lm, r,
                              key_offsets_host=ko, query_offsets_host=qo, packed_keys=knn.pack_keys(k) if packs else None)
    assert select_paths.of_problem(prob).select == want
    p_m, ids, dists = (t.clone() for t in prob.run())
    whole, own = prob.workspace, prob.dtype
    least = knn.load().knn_lm_mixture_workspace_size(prob.B, d, V, S, n, prob.min_keys, prob.max_keys, q, own, r)
    other = own ^ knn.KEYS_PACKED if dtype != torch.float32 else own
    for first, rest in ((whole.numel(), least), (least, whole.numel())):
        prob.dtype, prob.workspace = own, whole[:first]
        whole.random_()
        prob.run_part("distances")
        for size in (rest, first):
            prob.dtype, prob.workspace = other, whole[:size]  # (a select reads no keys)
            for part in ("select_mix", "select", "select_mix"):
                for t in (prob.ids, prob.dists, prob.p_m):
                    t.fill_(-7)
                prob.run_part(part)
                assert torch.equal(prob.ids, ids) and torch.equal(prob.dists, dists), (first, size, part)
                if part == "select_mix":
                    torch.testing.assert_close(prob.p_m, p_m, rtol=1e-5, atol=1e-8)


@pytest.mark.parametrize("public", [False, True], ids=["handle", "public name"])
def test_current_stream(public, monkeypatch):
    if public:
        monkeypatch.setattr(knn, "_raw_stream", None)
    side = torch.cuda.Stream()
    assert knn._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert knn._stream() == side.cuda_stream
    assert knn._stream(side) == side.cuda_stream
