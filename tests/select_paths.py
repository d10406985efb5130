"""How a call runs -- the distance kernel and the select path -- as the library's own host code decides it
(knnlm_route: no part of the ABI, exported for the tests), under the names that the tests use."""
import ctypes
from typing import NamedTuple, Optional

from paper_2405_19325_amd import _lib

ANY_BYTES = (1 << 64) - 1  # a workspace that holds every list

KERNELS = ("elements", "streaming", "several-queries", "matrix-core", "packed")
SELECTS = ("groups", "parts", "wide", "sampled", "sampled-16384", "one-workgroup", "general")
MODES = {"none": 0, "fixed": 1, "rrc": 2, "nest": 3}


class Route(NamedTuple):
    kernel: str       # of the distance stage, rows aligned to 16 bytes
    tile_rows: int
    queries: int      # per distance workgroup
    select: str       # see route
    parts: int        # per row (split, wide and sampled selects)
    group_rows: int   # keys per group where the distance stage writes group minima, else 0


def route(B: int, d: int, dtype: int, S: int, max_keys: int, max_queries: int, r: int, V: Optional[int] = None,
          min_keys: Optional[int] = None, mode: str = "fixed", workspace_bytes: int = ANY_BYTES,
          stage: bool = False) -> Route:
    """Of a whole call (stage: of knn_lm_mixture_part's stages) with a mixture of `mode` over V tokens (V None: no mixture).  select is "fused", "groups" or
    "parts" (the split select, from group minima or from the parts kernel's sample), "wide", "sampled" or
    "sampled-16384", "one-workgroup" (the row in registers) or "general" (streamed)."""
    f = _lib.load()["knnlm_route"]
    f.restype = None
    f.argtypes = [ctypes.c_int64] * 7 + [ctypes.c_int, ctypes.c_int32, ctypes.c_int, ctypes.c_size_t, ctypes.c_int,
                                        ctypes.c_void_p]
    out = (ctypes.c_int32 * 7)()
    f(B, d, V or 0, S, max_keys if min_keys is None else min_keys, max_keys, max_queries, dtype, r,
      MODES[mode] if V else 0, workspace_bytes, int(stage), out)
    kernel, tile, queries, select, parts, group, fused = out
    return Route(KERNELS[kernel], tile, queries, "fused" if fused else SELECTS[select], parts, group)


def of_problem(prob, mode: str = "fixed", workspace_bytes: Optional[int] = None, stage: bool = False) -> Route:
    """Of a MixtureProblem's calls (mode "none": the select alone)."""
    return route(prob.B, prob.d, prob.dtype, prob.S, prob.max_keys, prob.max_queries, prob.r,
                 None if mode == "none" else prob.V, prob.min_keys, mode,
                 prob.workspace.numel() if workspace_bytes is None else workspace_bytes, stage)


def take(prob, select: str, *modes: str):
    """Has prob's calls (steps of these modes, by default of a fixed lambda) take the select `select`: on its own
    workspace or, where they take another there, on the smallest accepted one."""
    modes = modes or ("fixed",)
    if any(of_problem(prob, m).select != select for m in modes):
        prob.workspace = prob.workspace[:_lib.load().knn_lm_mixture_workspace_size(
            prob.B, prob.d, prob.V, prob.S, prob.total_keys, prob.min_keys, prob.max_keys, prob.max_queries, prob.dtype,
            prob.r)]
    assert {of_problem(prob, m).select for m in modes} == {select}, [of_problem(prob, m) for m in modes]
