"""Helpers shared by the GPU parity tests: upload of generated tensors, the error
metric, and construction of (raw / packed) factor pairs."""
import numpy as np

import synth_inputs as si

from paper_2604_17709_amd import TOKEN_TILE_BOTH  # noqa: F401  (importing the binding loads nothing)

# bf16 and fp32: the stated bars; fp16: the bf16 bar scaled by the ratio of the unit roundoffs (2^-11 / 2^-8), rounded up
TOL = {"bf16": 1e-2, "f16": 2e-3, "f32": 1e-5}

# (T, d_in, r, d_out) of the test of the RAW kernel's tiles; tests/test_plans.py checks that on 256 compute units they
# take every tile that the choice has, in both stages, for 32- and 16-bit pairs
RAW_ROWS = [
    (5, 700, 21, 66),          # 16 x 16; k = 21 in the second stage
    (5, 4200, 21, 66),         # 16 x 16, k shared by 16 wavefronts
    (4, 30, 4200, 66),         # ... in the second stage
    (101, 301, 1001, 37),      # 16 x 16, in 16 bits 16 x 32
    (63, 131, 4090, 15),       # 32 x 32
    (201, 47, 1638, 1643),     # 64 x 32; second stage in 16 bits 16 x 32
    (205, 19, 4092, 4076),     # rows aligned to four elements: 32 x 64 and 64 x 64 (in 16 bits the other way round)
    (1025, 17, 2044, 51),      # 32 x 64 (64 x 64) likewise, then 16 x 32
    (169, 33, 41, 1115),       # two products: 32 x 32
    (325, 33, 17, 773),        # two products in 16 bits: 64 x 32
]


def workspace_of_eight_ranges(dn, T, pair) -> int:
    """Bytes that a packed pair's first stage with a long k and few features runs in as eight k-ranges instead of sixteen."""
    t = -(-(32 if T <= 32 else 64 if T <= 64 else 128) * -(-pair.desc.r // 32) * 32 * 2 // 256) * 256
    part = dn.deinfer_workspace_bytes(T, [pair]) - 256 - t
    assert part % 16 == 0
    return 256 + t + part // 2


def to_dev(t: si.Tensor):
    import torch
    if t.dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(t.bits)).cuda()
    return torch.from_numpy(np.ascontiguousarray(t.bits).view(np.int16)).cuda().view(torch.float16 if t.dtype == "f16" else torch.bfloat16)


def to_host(y) -> np.ndarray:
    """Device result -> float64 numpy (exact for f32 and bf16)."""
    import torch
    return y.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def max_err(y: np.ndarray, ref: np.ndarray) -> float:
    """max |y - ref| / max |ref| over one output tensor (the parity gate)."""
    denom = float(np.max(np.abs(ref))) if ref.size else 1.0
    if denom == 0.0:
        return float(np.max(np.abs(y))) if y.size else 0.0
    return float(np.max(np.abs(y - ref))) / denom


def pair(dn, U: si.Tensor, V: si.Tensor, packed: bool):
    """Returns (Pair, keepalive)."""
    Ud, Vd = to_dev(U), to_dev(V)
    p = dn.raw_pair(Ud, Vd)
    if packed:
        return dn.deinfer_pack_factors(p), (Ud, Vd)
    return p, (Ud, Vd)
