"""The projections with their weights in slabs, the order of the library's 16-bit copies: the by-name tests of test_gpu_gemm_large run again
with the weights laid out so (columns that are no whole slabs stay in plain rows, as in a copy), then the tiles that the library chooses,
up to 512 rows and the eight-wave ones above, on slabs and on plain rows: the same bits.  Tolerances: see there."""
import ctypes

import pytest
import torch

import test_gpu_gemm_large as plain
from gpu_util import say
from test_gpu_gemm_large import CASES, GUARD, LOGPROB, QKV, RESID, STORE, SWIGLU, SWIGLU_RS, TILES, TYPES, _guarded, _operands, _pairs

pytestmark = pytest.mark.gpu


def _slabs(w):
    # slabs of 32 rows x 64 columns, a row's 64 values behind the previous row's, slabs one after another along a row
    n, k = w.shape
    return w.reshape(n // 32, 32, k // 64, 64).permute(0, 2, 1, 3).contiguous().reshape(n, k)


_plain_launch, _plain_sizes = plain._launch, plain._sizes


def _launch(act, tile, epi, a, w, c, extra=None, slices=1, sat=None):
    from paper_2605_26606_amd import binding
    if w.shape[0] % 32:
        return _plain_launch(act, tile, epi, a, w, c, extra, slices, sat)
    f = binding.library().pc_internal_gemm_large_slabs
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_void_p] * 3 + [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3
    assert a.is_contiguous() and w.is_contiguous() and a.shape[1] == w.shape[1]
    w = _slabs(w)
    got = f(TYPES[act][0], tile[0], tile[1], epi, slices, a.data_ptr(), w.data_ptr(), None if c is None else c.data_ptr(), a.shape[0],
            w.shape[0], a.shape[1], None if extra is None else ctypes.addressof(extra), None if sat is None else sat.data_ptr(),
            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return got


def _launch_eight(act, route, a, w, extra):
    from paper_2605_26606_amd import binding
    f = binding.library().pc_internal_gemm_qkv_slabs
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 2 + [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3
    w = _slabs(w)
    got = f(TYPES[act][0], route, a.data_ptr(), w.data_ptr(), a.shape[0], w.shape[0], a.shape[1], ctypes.addressof(extra), None,
            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return got


@pytest.fixture
def on_slabs(monkeypatch):
    # whole slabs of columns: the next multiple of 32
    monkeypatch.setattr(plain, "_sizes", lambda epi, tile: [(m, (n + 31) // 32 * 32, k) for m, n, k in _plain_sizes(epi, tile)])
    monkeypatch.setattr(plain, "_launch", _launch)
    monkeypatch.setattr(plain, "_launch_eight", _launch_eight)


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("epi,tile", [c for c in CASES if c[0] in (STORE, RESID)])
def test_plain_tiles(on_slabs, epi, tile, act):
    plain.test_plain_tiles(epi, tile, act)
    if epi == STORE:   # K slices of whole slabs, a ragged last column: 4 + 4 + 3 steps
        m, n, k, s = tile[0] + 5, tile[1] + 32, 704, 3
        a, w, exact, d = _operands(act, m, n, k, 5)
        out = torch.full((s + 1, m, n), GUARD, device="cuda")
        assert _launch(act, tile, epi, a, w, out, slices=s)
        assert bool(((out[:s].double().sum(0) - exact).abs() <= d).all())
        assert bool((out[s] == GUARD).all())


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("epi,tile", [c for c in CASES if c[0] in (SWIGLU, SWIGLU_RS)])
def test_gate_up_tiles(on_slabs, epi, tile, act):
    plain.test_gate_up_tiles(epi, tile, act)


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("tile", TILES[LOGPROB])
def test_log_softmax_tiles(on_slabs, tile, act):
    plain.test_log_softmax_tiles(tile, act)


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("tile", TILES[QKV])
@pytest.mark.parametrize("decode", [False, True])
def test_rotating_tiles(on_slabs, tile, act, decode):
    plain.test_rotating_tiles(tile, act, decode)


# (columns, K, epilogue, rows): the tiles of up to 512 rows for wide, very wide, mid-width, long and small projections, the eight-wave ones
# above; last tiles of 32 or 64 columns
CHOSEN = [
    (12352, 192, STORE, [3, 50, 100, 170, 250, 300, 400]),
    (33088, 128, STORE, [3, 50, 100, 170, 250]),
    (12352, 192, SWIGLU, [3, 50, 100, 170, 250, 300, 400]),
    (33088, 128, SWIGLU, [50, 100, 170, 250]),
    (4160, 2112, RESID, [3, 50, 100, 170, 250, 300, 400]),
    (1600, 5504, RESID, [3, 50, 200, 300, 400]),
    (1600, 576, STORE, [3, 50, 250]),
    (1600, 1536, RESID, [577, 1000]),
    (512, 128, RESID, [600]),
    (12352, 128, STORE, [600, 6000]),
]


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("n,k,epi,rows", CHOSEN)
def test_chosen_tiles_give_the_same_bits_on_slabs_and_rows(n, k, epi, rows, act):
    from paper_2605_26606_amd import binding
    f = binding.library().pc_internal_gemm
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 2 + [ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_size_t] + \
        [ctypes.c_void_p] * 2
    _, dtype, u, tiny = TYPES[act]
    cap = 8 << 20
    buffer = torch.empty(cap, device="cuda")
    for m in rows:
        say("chosen tile, epilogue %d, %s: %d x %d x %d" % (epi, act, m, n, k))
        a, w, exact, d = _operands(act, m, n, k, m + k)
        old = torch.randn((m, n), device="cuda")
        results = []
        for order in (w, _slabs(w)):
            whole, c = _guarded((m, n // 2) if epi == SWIGLU else (m, n), dtype if epi == SWIGLU else torch.float32, old if epi == RESID else 0)
            sat = torch.zeros(1, dtype=torch.int32, device="cuda")
            s = f(TYPES[act][0], epi, a.data_ptr(), order.data_ptr(), int(order is not w), c.data_ptr(), m, n, k,
                  buffer.data_ptr() if epi == RESID else None, cap if epi == RESID else 0, sat.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert s >= 1 and bool((whole[m:] == GUARD).all())
            results.append(buffer[:s * m * n].reshape(s, m, n).clone() if s > 1 else c.clone())
        assert torch.equal(results[0], results[1])
        got = results[1].double()
        if epi == SWIGLU:
            at = _pairs(n).cuda()
            g, up, dg, du = exact[:, at[:n // 2]], exact[:, at[n // 2:]], d[:, at[:n // 2]], d[:, at[n // 2:]]
            sig = torch.sigmoid(g)
            want = g * sig * up
            bound = 1.1 * up.abs() * dg + (g * sig).abs() * du + 1.1 * dg * du + want.abs() * (u + (2 + g.abs()) * 2.0 ** -21) + tiny
            if act == "f16":
                want = want.clamp(-65504, 65504)
            assert bool(((got - want).abs() <= bound).all())
        elif got.dim() == 3:
            assert bool(((got.sum(0) - exact).abs() <= d).all())
        else:
            want = exact + old.double() if epi == RESID else exact
            assert bool(((got - want).abs() <= d + 2.0 ** -23 * want.abs()).all())


@pytest.mark.parametrize("act", ["f16", "bf16"])
@pytest.mark.parametrize("m,n,k", [
    (1024, 1536, 1536),     # 128 x 64 blocks
    (577, 1600, 1536), (2000, 512, 2048), (513, 2048, 1472),       # 64 x 64 (23 steps of K: an uneven last slice)
    (600, 512, 256),        # short: one sum
])
def test_residual_blocks_give_the_bits_of_the_slices_they_stand_for(m, n, k, act):
    # The blocks of 64 rows that residual projections of some hundred rows run in, against the large tile and the K slices that they replace,
    # added up as the norm behind does: the slices in order, their sum to the residual.  With and without room for slices.
    from paper_2605_26606_amd import binding
    lib = binding.library()
    assert lib.pc_internal_resid_tile(m, n, k) > 0
    f = lib.pc_internal_gemm
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 2 + [ctypes.c_int, ctypes.c_void_p] + [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_size_t] + \
        [ctypes.c_void_p] * 2
    a, w, exact, d = _operands(act, m, n, k, m + k)
    old = torch.randn((m, n), device="cuda")
    order, cut = _slabs(w), 0
    for cap in (8 << 20, 0):
        s = ctypes.c_int()
        tile = lib.pc_internal_gemm_large_pick(RESID, 0, min(8, cap // (m * n)), m, n, k, ctypes.byref(s))
        cut += s.value > 1
        say("residual blocks, %s: %d x %d x %d, %d slices" % (act, m, n, k, s.value))
        parts = torch.empty((s.value, m, n), device="cuda")
        assert _launch(act, TILES[RESID][tile], STORE, a, w, parts, slices=s.value)
        want = torch.zeros((m, n), device="cuda")
        for part in parts:
            want += part
        want = old + want
        whole, c = _guarded((m, n), torch.float32, old)
        buffer = torch.empty(max(cap, 4), device="cuda")
        assert f(TYPES[act][0], RESID, a.data_ptr(), order.data_ptr(), 1, c.data_ptr(), m, n, k, buffer.data_ptr() if cap else None, cap, None,
                 torch.cuda.current_stream().cuda_stream) == 1
        torch.cuda.synchronize()
        assert torch.equal(c, want) and bool((whole[m:] == GUARD).all())
        assert bool(((c.double() - exact - old.double()).abs() <= d + 2.0 ** -23 * want.abs()).all())
    assert cut == (0 if k == 256 else 1)
