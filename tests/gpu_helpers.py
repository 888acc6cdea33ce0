"""Helpers for the GPU tests: move synth inputs to the device, build problem
descriptions, compare against the oracle."""
from __future__ import annotations

import numpy as np
import torch

import oracle as O
from paper_2609_10549_amd import compass as C

TOL = 5e-3   # normwise relative error bound for bf16 outputs

# Rows and columns of kernel_params.h's tile configurations.
TILE_SHAPES = [(256, 256), (128, 128), (256, 192), (256, 128), (128, 128), (128, 64), (128, 64), (64, 64), (192, 192), (128, 192)]

# (M, N, K, partial, tile configuration, K slices): plain GEMMs that reach
# every tile of kernel_params.h's TileCfg whole, with and without a partial,
# and every tile that splits K in an even and an odd count, with edges inside
# tiles and stages. tests/test_decode_host.py holds the plan to these.
PLAN_SIZES = [
    (4095, 3080, 328, False, 0, 1), (300, 3000, 72, False, 1, 1), (3000, 4992, 200, True, 1, 1),
    (4090, 3064, 520, True, 2, 1), (2040, 4088, 2048, False, 3, 1), (3969, 1992, 1000, False, 8, 1), (2049, 1000, 2048, True, 4, 1),
    (65, 72, 200, False, 5, 1), (770, 2056, 4096, True, 6, 1), (129, 1032, 4104, True, 6, 5),
    (512, 512, 12288, False, 6, 8), (513, 1024, 520, False, 7, 1), (1000, 776, 4104, True, 7, 1),
    (256, 3072, 8192, False, 4, 5), (1024, 3072, 8192, True, 9, 2),
    (2500, 4912, 264, True, 0, 1), (2500, 2512, 3080, False, 0, 2), (2500, 1792, 4104, True, 0, 3),
    (1300, 936, 3080, False, 1, 2), (1537, 656, 2056, False, 1, 3),
    (2500, 3472, 264, False, 2, 1), (3000, 1552, 4104, True, 2, 2), (2500, 1160, 5128, False, 2, 3),
    (3000, 2032, 1032, True, 3, 1), (2500, 1160, 4104, False, 3, 2), (2500, 824, 4104, True, 3, 3),
    (3000, 656, 2048, False, 4, 1), (1537, 992, 3080, True, 4, 2), (2500, 1552, 136, True, 5, 1), (1537, 656, 520, False, 6, 1),
    (2500, 3232, 136, True, 8, 1), (2500, 1552, 3080, True, 8, 2), (1537, 1440, 4104, False, 8, 3), (129, 6832, 12288, True, 8, 6),
    (2500, 1552, 520, False, 9, 1), (1300, 2992, 264, True, 9, 1), (1537, 936, 5128, True, 9, 3),
]


# (M, N, K, n, d, ring, tile configuration, K slices): InterDecom
# ReduceScatters with sends whose sub-GEMMs (M / d rows) reach every tile with
# the row map, the epilogue gate, the done counts and written-through stores,
# whole and split. The plan is held to these too.
DECOMP_RS_SIZES = [
    (4096, 6352, 264, 4, 2, "single", 0, 1), (4096, 2512, 4104, 4, 2, "double", 0, 3),
    (3072, 2752, 136, 8, 2, "double", 1, 1),
    (4096, 4432, 136, 4, 2, "single", 2, 1), (4096, 2272, 4104, 8, 2, "double", 2, 2), (2048, 3232, 5128, 4, 2, "single", 2, 3),
    (4096, 3232, 1032, 4, 2, "double", 3, 1), (3072, 1384, 4104, 4, 2, "single", 3, 3),
    (4096, 1048, 136, 4, 2, "single", 4, 1), (3072, 1104, 3080, 2, 2, "double", 4, 2),
    (5120, 3232, 136, 8, 4, "single", 5, 1), (768, 264, 3080, 4, 4, "double", 6, 5), (768, 264, 264, 4, 4, "single", 7, 1),
    (4096, 4192, 136, 8, 2, "double", 8, 1), (1152, 4192, 4104, 4, 2, "double", 8, 3),
    (3072, 2752, 264, 4, 2, "single", 9, 1), (3072, 1328, 4104, 4, 2, "double", 9, 3),
]


# Few-row GEMMs: every row-block count, K from less than one stage to several
# rounds of every wave, columns that end inside a workgroup's 16.
FEW_ROW_SIZES = [(1, 8, 8, False), (16, 264, 520, True), (17, 2048, 4096, False), (32, 72, 72, True),
                 (33, 1032, 1544, True), (48, 3072, 8192, False), (49, 776, 4104, True), (64, 264, 2056, False),
                 (8, 12288, 1032, True)]


def dev_bits(bits: np.ndarray, pinned: bool = False) -> torch.Tensor:
    """uint16 bf16 patterns -> int16 tensor on the GPU (or pinned host)."""
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16))
    if pinned:
        return t.pin_memory()
    return t.cuda()


def dev_f32(x: np.ndarray, pinned: bool = False) -> torch.Tensor:
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32))
    return t.pin_memory() if pinned else t.cuda()


def host_bits(t: torch.Tensor) -> np.ndarray:
    return t.cpu().numpy().view(np.uint16)


def host_f64(t: torch.Tensor) -> np.ndarray:
    return O.bf16_to_f64(host_bits(t))


def rel_err(got: np.ndarray, ref: np.ndarray) -> float:
    return float(np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-300))


class AGCase:
    """Device buffers of one AllGather+GEMM instance."""

    def __init__(self, inp: dict, rank: int, ring: str, pinned_remote: bool = False, local_in_place: bool = True):
        M, N, K, n = inp["M"], inp["N"], inp["K"], inp["n"]
        self.inp, self.rank, self.ring = inp, rank, ring
        self.gathered = torch.zeros((M, K), dtype=torch.int16, device="cuda")
        self.W = dev_bits(inp["W"])
        self.C = torch.zeros((M, N), dtype=torch.int16, device="cuda")
        rows = M // n
        self.shards = []
        for q, s in enumerate(inp["shards"]):
            if q == rank:
                if local_in_place:
                    self.gathered[q * rows:(q + 1) * rows] = dev_bits(s)
                    self.shards.append(self.gathered[q * rows:(q + 1) * rows])
                else:
                    self.shards.append(dev_bits(s))
            else:
                self.shards.append(dev_bits(s, pinned=pinned_remote))
        self.problem = C.ag_problem(self.shards, self.gathered, self.W, self.C, rank, ring)

    def reference(self) -> np.ndarray:
        sh = [O.bf16_to_f64(s) for s in self.inp["shards"]]
        return O.ag_gemm(sh, O.bf16_to_f64(self.inp["W"]))


class RSCase:
    """Device buffers of one GEMM+ReduceScatter instance."""

    def __init__(self, inp: dict, rank: int, ring: str, sends: bool = True, pinned_remote: bool = False):
        M, N, K, n = inp["M"], inp["N"], inp["K"], inp["n"]
        self.inp, self.rank, self.ring = inp, rank, ring
        self.A = dev_bits(inp["A"])
        self.W = dev_bits(inp["W"])
        self.C = torch.zeros((M, N), dtype=torch.int16, device="cuda")
        self.stage = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        self.partials = [dev_f32(p, pinned=pinned_remote) for p in inp["P_in"]]
        rows = M // n
        self.send = None
        if sends:
            self.send = [None if q == rank else torch.zeros((rows, N), dtype=torch.int16, device="cuda")
                         for q in range(n)]
        self.problem = C.rs_problem(self.A, self.W, self.partials, self.stage, self.C, self.send, rank, ring)

    def reference(self) -> np.ndarray:
        P = [p.astype(np.float64) for p in self.inp["P_in"]]
        return O.gemm_rs(O.bf16_to_f64(self.inp["A"]), O.bf16_to_f64(self.inp["W"]), P, self.inp["n"])
