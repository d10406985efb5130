"""Every select path, on workspaces that hold its lists and on the smallest accepted one, against a stable sort
of the distance matrix; the mixture of rows that 16-byte accesses fit and don't."""
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


def _smallest_workspace(prob):
    """The fewest bytes that knn_lm_mixture accepts for the problem."""
    size = knn.load().knn_lm_mixture_workspace_size(prob.B, prob.d, prob.V, prob.S, prob.total_keys, prob.min_keys,
                                                    prob.max_keys, prob.max_queries, prob.dtype, prob.r)
    assert prob._validate(256, size) == 0 and prob._validate(256, size - 1) != 0
    return size


def _reference(dist, ko, qo, r, masked):
    ids, ds = [], []
    for s in range(len(ko) - 1):
        n = int(ko[s + 1] - ko[s])
        m = torch.from_numpy(masked[int(ko[s]):int(ko[s + 1])]).cuda()
        for b in range(int(qo[s]), int(qo[s + 1])):
            d, i = torch.where(m, math.inf, dist[b, :n]).sort(stable=True)
            ds.append(d[:r])
            ids.append(torch.where(torch.isinf(d[:r]), -1, i[:r]).int())
    return torch.stack(ids), torch.stack(ds)


# queries and keys per set, d, dtype, r, V, largest entry of integer keys (0: normal keys), the selects of the
# fixed-lambda step, of the masked step, and of both on the smallest workspace
CASES = {
    "groups, 320 parts": (40, (8000, 5000, 4097, 7999), 64, torch.float32, 1000, 1000, 0, "groups", "groups", "one-workgroup"),
    "split, 600 parts": (150, (8000, 5000), 64, torch.float32, 1000, 5001, 0, "parts", "parts", "one-workgroup"),
    "split, rows of one part": (45, (4096, 4000, 1024, 4500, 3001), 64, torch.float32, 1024, 1003, 0, "parts", "parts",
                                "one-workgroup"),
    "split, every distance alike": (300, (4096,), 8, torch.float32, 64, 500, 1, "parts", "parts", "one-workgroup"),
    "groups, 5/4 r of them": (2, (5200, 7437), 16, torch.float32, 1024, 5001, 0, "groups", "groups", "groups"),
    "one workgroup a row, 900 parts": (90, (20000, 9000), 64, torch.float32, 1024, 5001, 0, "one-workgroup",
                                       "one-workgroup", "one-workgroup"),
    "one workgroup a row of one part": (300, (3000,), 8, torch.float32, 64, 17001, 0, "one-workgroup", "parts",
                                        "one-workgroup"),
    "one workgroup a short row": (1100, (3000,), 8, torch.float32, 64, 17001, 0, "one-workgroup", "one-workgroup",
                                  "one-workgroup"),
    "one workgroup a long row": (100, (48000, 33001), 16, torch.float32, 1000, 1000, 0, "one-workgroup", "one-workgroup",
                                 "one-workgroup"),
    "rows over 1024 parts": (1100, (3000, 4097), 8, torch.float32, 100, 37, 0, "sampled", "sampled", "one-workgroup"),
    "sampled, r over 1024": (3, (5000, 2100, 40000), 16, torch.float32, 2048, 40001, 0, "sampled", "sampled", "general"),
    "sampled, long rows": (20, (262144,), 128, torch.bfloat16, 1024, 1003, 0, "sampled", "sampled", "general"),
    "sampled from 16384": (18, (300000, 4099), 128, torch.float16, 1024, 1000, 0, "sampled-16384", "sampled-16384", "general"),
    "sampled, few values": (18, (100000,), 128, torch.bfloat16, 900, 1001, 1, "sampled", "sampled", "general"),
    "streamed, r over 2048": (2, (9000,), 32, torch.float32, 3000, 1000, 0, "general", "general", "general"),
}


@pytest.mark.parametrize("share", [0.0, 0.02, 0.5], ids=["all-keys", "masked", "half-masked"])
@pytest.mark.parametrize("name", list(CASES))
def test_select_and_mixture(name, share):
    q, sizes, d, dtype, r, V, top, fixed, nest, small = CASES[name]
    masks = share > 0
    print(f"[gpu] select route: {name} masked={share}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(q + d + r)
    S, n = len(sizes), sum(sizes)
    ko = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    qo = np.arange(S + 1, dtype=np.int64) * q

    def draw(rows):
        if top:
            x = torch.zeros(rows, d, device="cuda")
            x[:, :4] = torch.randint(-top, top + 1, (rows, 4), generator=g, device="cuda").float()
            return x.to(dtype)
        return (torch.randn(rows, d, generator=g, device="cuda") * (8 / math.sqrt(d))).to(dtype)

    k, x = draw(n), draw(S * q)
    values = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    p_lm = torch.softmax(torch.randn(S * q, V, generator=g, device="cuda"), 1)
    masked = np.zeros(n, bool)
    if masks:
        masked[np.random.default_rng(5).choice(n, int(n * share), replace=False)] = True
    tko, tqo = torch.from_numpy(ko).cuda(), torch.from_numpy(qo).cuda()
    prob = knn.MixtureProblem(x, k, values, tko, tqo, p_lm, r, lam=0.3, key_offsets_host=ko, query_offsets_host=qo)
    dist = knn.distances(x, k, tko, tqo, key_offsets_host=ko, query_offsets_host=qo)
    ids, ds = _reference(dist, ko, qo, r, masked)
    mask = knn.mask_words(np.flatnonzero(masked), n, "cuda") if masks else None
    base = torch.from_numpy(np.repeat(ko[:-1], q)).cuda()[:, None]
    w = torch.where(ids < 0, 0.0, torch.exp(-prob.mu * (ds.double() - ds[:, :1].double())))
    p_knn = torch.zeros(S * q, V, dtype=torch.float64, device="cuda")
    p_knn.scatter_add_(1, values[(base + ids.clamp(min=0)).flatten()].view_as(ids).long(), w / w.sum(1, keepdim=True))
    whole = prob.workspace
    for size in (whole.numel(), _smallest_workspace(prob)):
        prob.workspace = whole[:size]
        want = small if size < whole.numel() else nest if masks else fixed
        assert select_paths.of_problem(prob, "nest" if masks else "fixed").select == want
        if masks:  # lambda_t and the decoding outputs too
            out = prob.run_nest(0.3, 0.1, 0.5, key_mask=mask)
            lam = out["lambdas"].double()[:, None]
            assert torch.equal(out["next_token"].long(), out["p_m"].argmax(1)) or \
                torch.equal(out["p_max"], out["p_m"].max(1).values)
        else:
            prob.run()
            lam = 0.3
        assert torch.equal(prob.ids, ids), size
        assert torch.equal(prob.dists, ds), size
        # a weight's fp32 argument is off by at most an ulp of mu d (2^-18 at d = 128): 1e-5 of p_kNN
        torch.testing.assert_close(prob.p_m.double(), lam * p_lm.double() + (1 - lam) * p_knn, rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("case", ["sample-far", "sample-near"])
def test_one_workgroup_row_misjudged(case):
    """20 rows of 65,536 keys in the smallest workspace, where one workgroup selects each row: with the keys at
    its sample's positions all far or all nearest, its threshold misjudges the count and the row is streamed."""
    print(f"[gpu] one-workgroup row, {case}", flush=True)
    n, B, d, r, V = 65536, 20, 16, 1024, 50
    t = np.arange(1024)
    sample = (t & 15) * 4096 + 4 * t + ((t >> 4) & 3)
    rng = np.random.default_rng(11)
    k = rng.integers(-30, 31, (n, d)).astype(np.float32)
    if case == "sample-far":
        k[sample] = 100
    else:
        k[:, 0] += 100
        k[sample, 0] -= 100
    dev = "cuda"
    tk = torch.as_tensor(k, device=dev)
    tq = torch.as_tensor(rng.integers(-3, 4, (B, d)).astype(np.float32), device=dev)
    ko, qo = np.array([0, n]), np.array([0, B])
    tko, tqo = torch.as_tensor(ko, device=dev), torch.as_tensor(qo, device=dev)
    values = torch.as_tensor(rng.integers(0, V, n).astype(np.int32), device=dev)
    p_lm = torch.full((B, V), 1.0 / V, device=dev)
    prob = knn.MixtureProblem(tq, tk, values, tko, tqo, p_lm, r, key_offsets_host=ko, query_offsets_host=qo)
    prob.workspace = prob.workspace[:_smallest_workspace(prob)]
    assert select_paths.of_problem(prob).select == "one-workgroup"
    prob.run()
    ids, ds = _reference(knn.distances(tq, tk, tko, tqo), ko, qo, r, np.zeros(n, bool))
    assert torch.equal(prob.ids, ids) and torch.equal(prob.dists, ds)


@pytest.mark.parametrize("offset", [0, 1], ids=["rows alike", "rows off by four bytes"])
@pytest.mark.parametrize("V", [5, 1003, 4099, 33001])
@pytest.mark.parametrize("B,r", [(3, 64), (3, 300), (40, 64)])
def test_rows_off_a_16_byte_boundary(B, r, V, offset):
    """p_M and the decoding outputs of rows whose length is no multiple of four, by slices and whole, with p_LM
    lying as p_M does or not; r = 64 sorts its candidates by rank."""
    print(f"[gpu] odd rows B={B} r={r} V={V} offset={offset}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(V + B)
    n, d = 6000, 8
    k, x = (torch.randn(m, d, generator=g, device="cuda") for m in (n, B))
    values = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    flat = torch.empty(B * V + 1, device="cuda")
    p_lm = flat[offset:offset + B * V].view(B, V)
    p_lm.copy_(torch.softmax(torch.randn(B, V, generator=g, device="cuda"), 1))
    drafts = torch.randint(0, V, (B,), generator=g, device="cuda", dtype=torch.int32)
    drafts[:3] = torch.tensor([0, V - 1, min(V - 1, 4097)], device="cuda")
    off, qo = torch.tensor([0, n], device="cuda"), torch.tensor([0, B], device="cuda")
    prob = knn.MixtureProblem(x, k, values, off, qo, p_lm, r)
    out = prob.run_nest(0.3, 0.1, 0.5, draft_tokens=drafts)
    d64 = torch.cdist(x.double(), k.double()).square()
    ds, ids = d64.topk(r, largest=False)
    assert torch.equal(out["ids"].sort(1).values, ids.int().sort(1).values)
    w = torch.exp(-prob.mu * (ds - ds[:, :1]))
    p_knn = torch.zeros(B, V, dtype=torch.float64, device="cuda").scatter_add_(1, values[ids].long(), w / w.sum(1, True))
    lam = out["lambdas"].double()[:, None]
    torch.testing.assert_close(out["p_m"].double(), lam * p_lm.double() + (1 - lam) * p_knn, rtol=2e-5, atol=1e-7)
    assert torch.equal(out["p_draft"], out["p_m"].gather(1, drafts.long()[:, None])[:, 0])
    assert torch.equal(out["p_max"], out["p_m"].max(1).values)
    first = (out["p_m"] == out["p_max"][:, None]).int().argmax(1)
    assert torch.equal(out["next_token"].long(), first)
