"""How a call runs -- the distance kernel and the select path -- as the library's own host code decides it
(knnlm_route: no part of the ABI, exported for the tests), under the names that the tests use."""
import ctypes
from typing import NamedTuple, Optional

from paper_2405_19325_amd import _lib

ANY_BYTES = (1 << 64) - 1  # a workspace that holds every list

KERNELS = ("elements", "streaming", "several-queries", "matrix-core", "packed")
SLICE, SLICED_BLOCKS = 4096, 256  # the sliced finish: vocabulary entries a workgroup, workgroups at most


class Route(NamedTuple):
    kernel: str       # of the distance stage, rows aligned to 16 bytes
    tile_rows: int
    queries: int      # per distance workgroup
    select: str       # see select_path
    parts: int        # per row (split, wide and sampled selects)
    group_rows: int   # keys per group where the distance stage writes group minima, else 0


def sliced(B: int, V: Optional[int]) -> bool:
    """Whether a split select's finish with a mixture over V tokens (None: no mixture) may read group minima."""
    return V is None or B * ((V + SLICE - 1) // SLICE) <= SLICED_BLOCKS


def route(B: int, d: int, dtype: int, S: int, max_keys: int, max_queries: int, r: int, V: Optional[int] = None,
          min_keys: Optional[int] = None, workspace_bytes: int = ANY_BYTES) -> Route:
    """Of a whole call (V None: no mixture).  select is "fused", "groups" or "parts" (the split select, from group
    minima or from the parts kernel's sample), "wide", "sampled" or "sampled-16384", "one-workgroup" (the row in
    registers) or "general" (streamed)."""
    f = _lib.load()["knnlm_route"]
    f.restype = None
    f.argtypes = [ctypes.c_int64] * 6 + [ctypes.c_int, ctypes.c_int32, ctypes.c_size_t, ctypes.c_void_p]
    out = (ctypes.c_int32 * 8)()
    f(B, d, S, max_keys if min_keys is None else min_keys, max_keys, max_queries, dtype, r, workspace_bytes, out)
    kernel, tile, queries, path, parts, group, fused, registers = out
    select = ("one-workgroup" if registers else "general", "groups" if group and sliced(B, V) else "parts", "wide",
              "sampled", "sampled-16384")[path]
    return Route(KERNELS[kernel], tile, queries, "fused" if fused else select, parts, group)


def of_problem(prob, mixture: bool = True, workspace_bytes: Optional[int] = None) -> Route:
    """Of a MixtureProblem's calls."""
    return route(prob.B, prob.d, prob.dtype, prob.S, prob.max_keys, prob.max_queries, prob.r,
                 prob.V if mixture else None, prob.min_keys,
                 prob.workspace.numel() if workspace_bytes is None else workspace_bytes)
