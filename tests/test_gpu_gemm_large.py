"""Every tile of the large projection kernel by name, in every epilogue it is built for and both 16-bit types, against 64-bit
sums: row and column remainders, two, three and five steps of K to a tile, several output tiles per block, an uneven last K slice.
(The library chooses a tile by an estimate of its time, so the sizes of a model test say little about which one runs.)  The
q/k/v tiles on eight waves that share such batches are run alongside; all give the same bits.

Tolerances.  The operands are exact in 16 bits; a product is summed in float32, K of them with at most K roundings of 2^-24 each:
|sum - exact| <= K 2^-24 sum |a w|, called d below.  Results in the model type add their own rounding, 2^-11 of the value in half
and 2^-8 in bfloat16."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu

STORE, RESID, SWIGLU, SWIGLU_RS, LOGPROB, QKV = 0, 1, 2, 4, 5, 6
TILES = {
    STORE: [(256, 256), (256, 192), (192, 256), (256, 128), (192, 128), (128, 128)],
    RESID: [(256, 256), (256, 192), (192, 256), (256, 128), (192, 128), (128, 128)],
    SWIGLU: [(256, 256), (192, 256), (192, 128)],
    SWIGLU_RS: [(256, 256), (192, 256)],
    LOGPROB: [(256, 256), (192, 256)],
    QKV: [(256, 256), (192, 256), (192, 128)],
}
EIGHT = {(64, 128): 1, (128, 128): 2, (256, 128): 3, "256x256 on eight waves": 4, "128x128 two to a CU": 5}   # their routes
CASES = [(e, t) for e, ts in TILES.items() for t in ts]
TYPES = {"f16": (2, torch.float16, 2.0 ** -11, 2.0 ** -24), "bf16": (1, torch.bfloat16, 2.0 ** -8, 0.0)}
GUARD = -77.0


class RowScale(ctypes.Structure):
    _fields_ = [("ssq", ctypes.c_void_p), ("tiles", ctypes.c_int), ("d", ctypes.c_int), ("eps", ctypes.c_float)]


class Logprob(ctypes.Structure):
    _fields_ = [("inv_t", ctypes.c_float), ("tokens", ctypes.c_void_p), ("token_index", ctypes.c_void_p), ("part_max", ctypes.c_void_p),
                ("target", ctypes.c_void_p), ("part_sum", ctypes.c_void_p)]


class KvGeom(ctypes.Structure):
    _fields_ = [("pool", ctypes.c_void_p), ("layer_stride", ctypes.c_int64), ("block_size", ctypes.c_int32), ("n_kv_heads", ctypes.c_int32),
                ("head_dim", ctypes.c_int32), ("max_blocks_per_slot", ctypes.c_int32), ("block_table", ctypes.c_void_p)]


class Qkv(ctypes.Structure):
    _fields_ = [("row_slot", ctypes.c_void_p), ("row_pos", ctypes.c_void_p), ("slot_len", ctypes.c_void_p), ("rope_cos", ctypes.c_void_p),
                ("rope_sin", ctypes.c_void_p), ("kv", KvGeom), ("layer", ctypes.c_int), ("hq", ctypes.c_int), ("q_out", ctypes.c_void_p)]


def _launch(act, tile, epi, a, w, c, extra=None, slices=1, sat=None):
    from paper_2605_26606_amd import binding
    f = binding.library().pc_internal_gemm_large
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_void_p] * 3 + [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3
    assert a.is_contiguous() and w.is_contiguous() and a.shape[1] == w.shape[1]
    got = f(TYPES[act][0], tile[0], tile[1], epi, slices, a.data_ptr(), w.data_ptr(), None if c is None else c.data_ptr(), a.shape[0],
            w.shape[0], a.shape[1], None if extra is None else ctypes.addressof(extra), None if sat is None else sat.data_ptr(),
            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return got


def _launch_eight(act, route, a, w, extra):
    from paper_2605_26606_amd import binding
    f = binding.library().pc_internal_gemm_qkv
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 2 + [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3
    got = f(TYPES[act][0], route, a.data_ptr(), w.data_ptr(), a.shape[0], w.shape[0], a.shape[1], ctypes.addressof(extra), None,
            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return got


def _operands(act, m, n, k, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn((m, k), generator=g, device="cuda").to(TYPES[act][1])
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.25).to(TYPES[act][1])
    a64, w64 = a.double(), w.double()
    exact = a64 @ w64.t()
    return a, w, exact, (a64.abs() @ w64.abs().t()) * (k * 2.0 ** -24)


def _guarded(shape, dtype, fill):
    # the array with 64 rows of guard values behind it, which must not change
    whole = torch.full((shape[0] + 64, shape[1]), GUARD, dtype=dtype, device="cuda")
    whole[:shape[0]] = fill
    return whole, whole[:shape[0]]


def _sizes(epi, tile):
    """(rows, columns, K): less than a tile and a bit more than one, the reductions of odd and even step counts; then more than
    256 tiles, so that blocks compute several"""
    bm, bn = tile
    unit = 64 if epi in (SWIGLU, SWIGLU_RS) else (128 if epi == QKV else 16)
    few = (bn * 2 + bn // 3 + unit) // unit * unit
    many = (90 * bn - 7 * bn // 16) // unit * unit
    return [(bm - 19, max(unit, few // 4 // unit * unit), 128), (bm + 37, few, 320), (2 * bm + 37, many, 192), (2 * bm + 1, many, 128)]


def _pairs(n):
    # where gate (first half) and up (second half) rows go: chunks of 16 gate rows and their 16 up rows
    j = torch.arange(n // 2)
    gate = 32 * (j // 16) + j % 16
    return torch.cat([gate, gate + 16])


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("epi,tile", [c for c in CASES if c[0] in (STORE, RESID)])
def test_plain_tiles(epi, tile, act):
    for m, n, k in _sizes(epi, tile):
        say("large tile %dx%d, epilogue %d, %s: %d x %d x %d" % (*tile, epi, act, m, n, k))
        a, w, exact, d = _operands(act, m, n, k, m + k)
        old = torch.randn((m, n), device="cuda") if epi == RESID else torch.zeros((m, n), device="cuda")
        whole, c = _guarded((m, n), torch.float32, old)
        assert _launch(act, tile, epi, a, w, c)
        want = exact + old.double()
        assert bool(((c.double() - want).abs() <= d + 2.0 ** -23 * want.abs()).all())
        assert bool((whole[m:] == GUARD).all())
    if epi == STORE:   # results that start at any float
        m, n, k = tile[0] + 3, tile[1] + 48, 128
        a, w, exact, d = _operands(act, m, n, k, 6)
        flat = torch.full((m * n + 8,), GUARD, device="cuda")
        assert _launch(act, tile, epi, a, w, flat[1:])
        assert bool(((flat[1:1 + m * n].double().reshape(m, n) - exact).abs() <= d).all())
        assert bool((flat[1 + m * n:] == GUARD).all()) and float(flat[0]) == GUARD
    if epi == STORE:   # K slices: 4 + 4 + 3 steps; the sum of the slices is the product
        m, n, k, s = tile[0] + 5, tile[1] + 16, 704, 3
        a, w, exact, d = _operands(act, m, n, k, 5)
        out = torch.full((s + 1, m, n), GUARD, device="cuda")
        assert _launch(act, tile, epi, a, w, out, slices=s)
        assert bool(((out[:s].double().sum(0) - exact).abs() <= d).all())
        assert bool((out[s] == GUARD).all())


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("epi,tile", [c for c in CASES if c[0] in (SWIGLU, SWIGLU_RS)])
def test_gate_up_tiles(epi, tile, act):
    _, dtype, u, tiny = TYPES[act]
    for m, n, k in _sizes(epi, tile):
        say("large tile %dx%d, epilogue %d, %s: %d x %d x %d" % (*tile, epi, act, m, n, k))
        a, w, exact, d = _operands(act, m, n, k, m + k)
        extra = None
        if epi == SWIGLU_RS:   # partial sums of squares of 32 columns each; one row is tiny, so that its scale is large
            tiles = k // 32
            ssq = torch.rand((tiles, m), device="cuda") * 64 + 1
            ssq[:, m // 2] *= 1e-4
            extra = RowScale(ssq.data_ptr(), tiles, k, 1e-6)
            scale = (1.0 / torch.sqrt(ssq.double().sum(0) / k + float(np.float32(1e-6))))[:, None]
            exact, d = exact * scale, d * scale + (exact * scale).abs() * (tiles + 8) * 2.0 ** -24
        at = _pairs(n).cuda()
        g, up, dg, du = exact[:, at[:n // 2]], exact[:, at[n // 2:]], d[:, at[:n // 2]], d[:, at[n // 2:]]
        sig = torch.sigmoid(g)
        want = g * sig * up
        # derivative of g sigmoid(g): at most 1.1; exp2 and reciprocal of the hardware: a few 2^-24 of the value times 1 + |g|
        bound = 1.1 * up.abs() * dg + (g * sig).abs() * du + 1.1 * dg * du + want.abs() * (u + (2 + g.abs()) * 2.0 ** -21) + tiny
        whole, c = _guarded((m, n // 2), dtype, 0)
        sat = torch.zeros(1, dtype=torch.int32, device="cuda")
        assert _launch(act, tile, epi, a, w, c, extra, sat=sat)
        if act == "f16":   # beyond the half range: clamped, and counted once each
            over = want.abs() > 65504 * (1 + 2.0 ** -10)
            near = (want.abs() > 65504 * (1 - 2.0 ** -10)) & ~over
            assert int(over.sum()) <= int(sat) <= int(over.sum() + near.sum())
            want = want.clamp(-65504, 65504)
        assert bool(((c.double() - want).abs() <= bound).all())
        assert bool((whole[m:] == GUARD).all())
    if act == "f16":
        # values beyond the range in the first and last row and column, and none elsewhere
        m, n, k = tile[0] + 3, tile[1] + 64, 192
        a, w = torch.zeros((m, k), device="cuda").half(), torch.zeros((n, k), device="cuda").half()
        a[0, 0] = a[m - 1, 0] = 512.0
        at = _pairs(n).cuda()
        cols = torch.tensor([0, n // 2 - 1], device="cuda")
        w[at[:n // 2][cols], 0] = 2.0
        w[at[n // 2:][cols], 0] = -2.0
        extra = None
        if epi == SWIGLU_RS:
            ssq = torch.full((k // 32, m), 32.0, device="cuda")
            extra = RowScale(ssq.data_ptr(), k // 32, k, 0.0)
        whole, c = _guarded((m, n // 2), dtype, 0)
        sat = torch.zeros(1, dtype=torch.int32, device="cuda")
        assert _launch(act, tile, epi, a, w, c, extra, sat=sat)
        want = torch.zeros((m, n // 2), device="cuda")
        for r in (0, m - 1):
            want[r, cols] = -65504.0
        assert torch.equal(c.float(), want) and int(sat) == 4


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("tile", TILES[LOGPROB])
def test_log_softmax_tiles(tile, act):
    for m, n, k in _sizes(LOGPROB, tile):
        say("large tile %dx%d, log-softmax, %s: %d x %d x %d" % (*tile, act, m, n, k))
        a, w, exact, d = _operands(act, m, n, k, m + k)
        strips = (n + 255) // 256 * 2
        rng = np.random.default_rng(m)
        tokens = torch.from_numpy(rng.integers(0, n, m + 1).astype(np.int32)).cuda()
        tokens[1], tokens[2], tokens[3], tokens[m] = 0, n - 1, n + 5, n - 1      # first, last and no column
        index = torch.arange(m, dtype=torch.int32, device="cuda")
        inv_t = float(np.float32(1.0 / 0.7))
        mx_all, mx = _guarded((strips, m), torch.float32, 3.0)
        sm_all, sm = _guarded((strips, m), torch.float64, 3.0)
        target = torch.full((m,), GUARD, device="cuda")
        extra = Logprob(inv_t, tokens.data_ptr(), index.data_ptr(), mx.data_ptr(), target.data_ptr(), sm.data_ptr())
        assert _launch(act, tile, LOGPROB, a, w, None, extra)
        col = tokens[1:].long()
        inside = col < n
        assert bool((target[~inside] == GUARD).all())
        r = torch.arange(m, device="cuda")[inside]
        assert bool(((target[inside].double() - exact[r, col[inside]]).abs() <= d[r, col[inside]]).all())
        pad = strips * 128 - n
        x = torch.nn.functional.pad(exact * inv_t, (0, pad), value=-float("inf")).reshape(m, strips, 128)
        e = torch.nn.functional.pad((d + exact.abs() * 2.0 ** -24) * inv_t, (0, pad)).reshape(m, strips, 128).amax(2)
        empty = torch.isinf(x).all(2)
        assert bool((torch.isinf(mx.t()) == empty).all()) and bool((sm.t()[empty] == 0).all())
        full = ~empty
        assert bool(((mx.t().double() - x.amax(2))[full].abs() <= e[full]).all())
        # the strip's log-sum: every exponential is off by e (and by its own rounding and the subtraction's, 2^-22 of 1 + |x|)
        want = torch.logsumexp(x, 2)
        got = mx.t().double() + torch.log(sm.t())
        assert bool(((got - want)[full].abs() <= (2 * e + 2.0 ** -21 * (1 + x.abs().nan_to_num(0, 0, 0).amax(2)))[full]).all())
        assert bool((mx_all[strips:] == GUARD).all()) and bool((sm_all[strips:] == GUARD).all())


def _packed(j):
    # the column of dim j of a q or k head: blocks of 16 dims and their 16 rotary partners
    return torch.where(j < 64, 32 * (j // 16) + j % 16, 32 * ((j - 64) // 16) + 16 + j % 16)


def _k_index(tin, d):
    tt = tin % 32
    lane = (tt // 8) * 4 + tt % 4
    frag = ((tin // 32) * 2 + (tt // 4) % 2) * 4 + d // 32
    return frag * 512 + (((d % 32) // 8) * 16 + lane) * 8 + d % 8


def _v_index(tin, d, bs):
    frag = (tin // 32) * 8 + d // 16
    return bs * 128 + frag * 512 + (((tin % 32) // 8) * 16 + d % 16) * 8 + tin % 8


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("tile", TILES[QKV])
@pytest.mark.parametrize("decode", [False, True])
def test_rotating_tiles(tile, act, decode):
    _, dtype, u, tiny = TYPES[act]
    # enough heads for more than 256 tiles at two row blocks and a remainder in the last size
    many = -(-260 * tile[1] // (3 * 128))
    for m, hq, hkv, k, bs in [(tile[0] - 19, 2, 1, 128, 32), (tile[0] + 37, 3, 3, 320, 64), (2 * tile[0] + 37, many - 6, 3, 192, 128)]:
        n = (hq + 2 * hkv) * 128
        say("large tile %dx%d, q/k/v, %s, %s: %d x %d x %d" % (*tile, act, "decode" if decode else "prefill", m, n, k))
        a, w, exact, d = _operands(act, m, n, k, m + k)
        # weight rows in the order of the packed heads (the values are those of the natural order)
        order = torch.arange(n)
        for h in range(hq + hkv):
            order[128 * h + _packed(torch.arange(128))] = 128 * h + torch.arange(128)
        w = w[order.cuda()].contiguous()
        rng = np.random.default_rng(m)
        max_ctx, per_slot = 4 * bs, 4
        if decode:      # every row a sequence of its own, anywhere in its context
            slots = m
            row_slot = rng.permutation(slots)
            slot_len = rng.integers(0, max_ctx, slots)
            pos = slot_len[row_slot]
        else:           # prompts one behind the other, ragged
            lens, left = [], m
            while left:
                lens.append(min(left, int(rng.integers(1, max_ctx + 1))))
                left -= lens[-1]
            slots = len(lens)
            ids = rng.permutation(slots)
            row_slot = np.repeat(ids, lens)
            pos = np.concatenate([np.arange(x) for x in lens])
            slot_len = np.full(slots, 10 ** 6)
        table = rng.permutation(slots * per_slot).astype(np.int32).reshape(slots, per_slot)
        inv = 1.0e4 ** (-2.0 * np.arange(64) / 128)
        ang = np.arange(max_ctx)[:, None] * inv[None]
        cos, sin = (torch.from_numpy(f(ang).astype(np.float32)).cuda() for f in (np.cos, np.sin))
        d_slot, d_pos, d_len, d_table = (torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()
                                         for x in (row_slot, pos, slot_len, table))
        head_elems, layer = 2 * bs * 128, 1
        block_elems = hkv * head_elems
        pool = torch.full((2, slots * per_slot, hkv, head_elems), 9.0, dtype=dtype, device="cuda")
        whole, q = _guarded((m, hq * 128), dtype, 0)
        extra = Qkv(d_slot.data_ptr(), None if decode else d_pos.data_ptr(), d_len.data_ptr(), cos.data_ptr(), sin.data_ptr(),
                    KvGeom(pool.data_ptr(), slots * per_slot * block_elems, bs, hkv, 128, per_slot, d_table.data_ptr()), layer, hq, q.data_ptr())
        assert _launch(act, tile, QKV, a, w, None, extra)
        c, s = cos[d_pos.long()].double()[:, None], sin[d_pos.long()].double()[:, None]

        def rotated(x, e):
            x, e = x.reshape(m, -1, 128), e.reshape(m, -1, 128)
            x1, x2, e1, e2 = x[..., :64], x[..., 64:], e[..., :64], e[..., 64:]
            y = torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], 2)
            # two products and a sum in float32 on top of what the products were off by
            b = torch.cat([e1 * c.abs() + e2 * s.abs(), e2 * c.abs() + e1 * s.abs()], 2) + 2.0 ** -22 * (x1.abs() + x2.abs()).repeat(1, 1, 2)
            return y, b + y.abs() * u + tiny

        want, bound = rotated(exact[:, :hq * 128], d[:, :hq * 128])
        assert bool(((q.double().reshape(m, hq, 128) - want).abs() <= bound).all())
        assert bool((whole[m:] == GUARD).all())
        kw, kb = rotated(exact[:, hq * 128:(hq + hkv) * 128], d[:, hq * 128:(hq + hkv) * 128])
        vw, vb = exact[:, (hq + hkv) * 128:].reshape(m, hkv, 128), d[:, (hq + hkv) * 128:].reshape(m, hkv, 128)
        tin = (d_pos.long() % bs)[:, None, None]
        block = d_table.long()[d_slot.long(), d_pos.long() // bs][:, None, None]
        head, dim = torch.arange(hkv, device="cuda")[None, :, None], torch.arange(128, device="cuda")[None, None, :]
        base = layer * slots * per_slot * block_elems + block * block_elems + head * head_elems
        flat = pool.reshape(-1)
        k_at, v_at = base + _k_index(tin, dim), base + _v_index(tin, dim, bs)
        assert bool(((flat[k_at].double() - kw).abs() <= kb).all())
        assert bool(((flat[v_at].double() - vw).abs() <= vb + vw.abs() * u + tiny).all())
        q_bits, kv_bits = q.clone(), flat.clone()
        flat[k_at] = 9.0
        flat[v_at] = 9.0
        assert bool((flat == 9.0).all())   # nothing else was touched
        for route in EIGHT.values():
            flat.fill_(9.0)
            q.zero_()
            assert _launch_eight(act, route, a, w, extra)
            assert torch.equal(q, q_bits) and torch.equal(flat, kv_bits), route
            assert bool((whole[m:] == GUARD).all())
