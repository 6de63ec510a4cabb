"""The rotation of q and k and the append to the cache (rope_append of csrc/elementwise.hip) against the same arithmetic in numpy: the same
bits.  The slices are added in their order in float32; the first value of a turned pair is fma(x1, cos, -(x2 sin)), the second
fma(x2, cos, x1 sin), each rounded to the model type.  A product of two float32 is exact in float64, so each fma is one float64 sum
rounded to float32 (the sum's own rounding matters in 1 of some 2^29 values)."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu

TYPES = {"fp32": (0, torch.float32), "bf16": (1, torch.bfloat16), "f16": (2, torch.float16)}


class KvGeom(ctypes.Structure):
    _fields_ = [("pool", ctypes.c_void_p), ("layer_stride", ctypes.c_int64), ("block_size", ctypes.c_int32), ("n_kv_heads", ctypes.c_int32),
                ("head_dim", ctypes.c_int32), ("max_blocks_per_slot", ctypes.c_int32), ("block_table", ctypes.c_void_p)]


def _k_index(tin, d, hd):
    if hd % 32:
        return tin * hd + d
    tt = tin % 32
    lane = (tt // 8) * 4 + tt % 4
    frag = ((tin // 32) * 2 + (tt // 4) % 2) * (hd // 32) + d // 32
    return frag * 512 + (((d % 32) // 8) * 16 + lane) * 8 + d % 8


# heads of 24: a pair to a thread; of 48 and 128 (also in the packed order): four pairs
@pytest.mark.parametrize("act", ["fp32", "bf16", "f16"])
@pytest.mark.parametrize("hd,perm", [(24, 0), (48, 0), (128, 0), (128, 1)])
def test_rotation_rounds_the_same_products_for_any_number_of_slices(hd, perm, act):
    from paper_2605_26606_amd import binding
    f = binding.library().pc_internal_rope_append
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int] + [ctypes.c_void_p] * 4 + [ctypes.c_int] * 2 + [ctypes.c_void_p, ctypes.c_int] + \
        [ctypes.c_void_p] * 2
    code, dtype = TYPES[act]
    rng = np.random.default_rng(hd)
    rows, hq, hkv, bs, half = 90, 10, 3, 32, hd // 2
    width = (hq + 2 * hkv) * hd
    pos = np.arange(rows) * 3 % 128
    slot = np.arange(rows, dtype=np.int32) % 2
    slot_of = {}   # (no two rows on one place of the cache)
    for r in range(rows):
        while (slot[r], pos[r]) in slot_of:
            pos[r] = (pos[r] + 1) % 128
        slot_of[slot[r], pos[r]] = r
    table = np.array([[3, 0, 6, 5], [1, 7, 2, 4]], np.int32)
    angle = np.arange(128)[:, None] * 1e4 ** (-np.arange(half) / half)[None]
    cos, sin = np.cos(angle).astype(np.float32), np.sin(angle).astype(np.float32)
    up = lambda a, t=None: torch.from_numpy(np.ascontiguousarray(a if t is None else a.astype(t))).cuda()  # noqa: E731
    d_pos, d_slot, d_table, d_cos, d_sin = up(pos, np.int32), up(slot), up(table), up(cos), up(sin)
    j = np.arange(hd)
    col = j if not perm else np.where(j < half, 32 * (j // 16) + j % 16, 32 * ((j - half) // 16) + 16 + (j - half) % 16)
    for slices in range(1, 9):
        say("rotation, %s, heads of %d%s, %d slices" % (act, hd, ", packed" if perm else "", slices))
        parts = rng.standard_normal((slices, rows, width)).astype(np.float32)
        x = parts[0].copy()
        for z in range(1, slices):
            x = x + parts[z]
        heads = x.reshape(rows, hq + 2 * hkv, hd)
        qk = heads[:, :hq + hkv][:, :, col]
        x1, x2 = qk[:, :, :half], qk[:, :, half:]
        c, s = cos[pos][:, None], sin[pos][:, None]
        wide = lambda a: a.astype(np.float64)  # noqa: E731
        first = (wide(x1) * wide(c) - wide(x2 * s)).astype(np.float32)
        second = (wide(x2) * wide(c) + wide(x1 * s)).astype(np.float32)
        want = torch.from_numpy(np.concatenate([first, second], 2)).to(dtype)
        want_v = torch.from_numpy(heads[:, hq + hkv:].copy()).to(dtype)
        pool = torch.zeros(8 * hkv * 2 * bs * hd, dtype=dtype, device="cuda")
        q = torch.zeros((rows, hq, hd), dtype=dtype, device="cuda")
        d_parts = up(parts)
        geom = KvGeom(pool.data_ptr(), pool.numel(), bs, hkv, hd, 4, d_table.data_ptr())
        assert f(code, d_parts.data_ptr(), slices, d_slot.data_ptr(), d_pos.data_ptr(), d_cos.data_ptr(), d_sin.data_ptr(), rows, hq,
                 ctypes.addressof(geom), perm, q.data_ptr(), torch.cuda.current_stream().cuda_stream) == 1
        torch.cuda.synchronize()
        assert torch.equal(q.cpu(), want[:, :hq])
        cache = pool.cpu().reshape(8, hkv, 2 * bs * hd)
        r, h, d = np.meshgrid(np.arange(rows), np.arange(hkv), np.arange(hd), indexing="ij")
        block, tin = table[slot[r], pos[r] // bs], pos[r] % bs
        assert torch.equal(cache[block, h, _k_index(tin, d, hd)], want[:, hq:])
        if hd % 32:
            assert torch.equal(cache[block, h, bs * hd + d * bs + tin], want_v)
