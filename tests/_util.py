"""Helpers shared by the GPU parity tests."""
import numpy as np
import torch

MAX_REL = 2e-2   # max|O_gpu - O_ref| / max|O_ref|, per head   (acceptance bar of the target)
MEAN_REL = 5e-3  # mean|O_gpu - O_ref| / mean|O_ref|, per head


def to_f64(x: torch.Tensor) -> np.ndarray:
    """[B,H,n,d] (or [BH,...]) tensor -> float64 numpy with batch and head flattened"""
    a = x.detach().float().cpu().numpy().astype(np.float64)
    if a.ndim == 4:
        a = a.reshape(a.shape[0] * a.shape[1], a.shape[2], a.shape[3])
    return a


def rel_errors(got: np.ndarray, ref: np.ndarray, rows=None):
    """per-head (max_rel, mean_rel); got/ref are [BH, n, d]; rows optionally restricts the tokens"""
    if rows is not None:
        got, ref = got[:, rows], ref[:, rows]
    out = []
    for h in range(ref.shape[0]):
        d = np.abs(got[h] - ref[h])
        out.append((d.max() / np.abs(ref[h]).max(), d.mean() / np.abs(ref[h]).mean()))
    return out


def assert_close(got, ref, rows=None, what=""):
    assert np.isfinite(got if rows is None else got[:, rows]).all(), f"{what}: non-finite output"
    for h, (mx, mean) in enumerate(rel_errors(got, ref, rows)):
        assert mx <= MAX_REL and mean <= MEAN_REL, f"{what}: head {h}: max_rel={mx:.3e} mean_rel={mean:.3e}"



def align256(x):
    return (x + 255) // 256 * 256


def attn_layout(s):
    """(bytes, offset of the slots for unit sums, slots per head) of the attention workspace that every entry point takes for a
    shape: the slices' results, a bitmap, the statistics tiles, the group matrices, the sums of units of at most 32 blocks
    (halved, down to 8, while that leaves fewer than 1024 of them), key means"""
    bh, nb = s.B * s.H, -(-s.n // s.block)
    chunks, total, partial, slots = -(-nb // 32), 0, 0, 0
    if s.kv_slices > 1:
        total += align256(bh * s.kv_slices * s.n * s.d * 4)
        total = align256(total + bh * s.kv_slices * s.n * 8) + 256
    total += align256(bh * nb * chunks * 4)
    if s.group > 0:
        group = min(s.group, nb)
        unit = min(group, 32)
        while unit > 8 and bh * -(-nb // unit) < 1024:
            unit //= 2
        slots = -(-nb // unit)
        partial = total + align256(bh * chunks * 64 * s.d * 2) + align256(bh * -(-nb // group) * s.d * s.d * 2)
        total = partial + align256(bh * slots * s.d * s.d * 4) + align256(bh * nb * s.d * 4)
    return total, partial, slots
