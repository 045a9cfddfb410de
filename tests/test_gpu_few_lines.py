"""Few lines: the tracer with four lanes to a half line against the one with one lane
(which a call with many lines takes), and the prep pass at the edges of its rows.

Both tracers form every sum in one order, so the same half line comes out bit for bit
the same. Every case prints what it runs before touching the GPU.
"""

import sys

import numpy as np
import pytest

import oracle
import synth
from synth import Plane, cubic_grid

from gpu_util import compare_maps, to_np

pytestmark = pytest.mark.gpu

F32X, F64 = 0, 1
LINE_KEYS = ("end_b", "end_f", "face_b", "face_f", "bn_b", "bn_f", "bn0", "tw", "length", "status")


def _say(msg):
    print(f"[gpu case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def fq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2208_12569_amd as m

    m._lib.load()
    return m


def _dev(B):
    import torch

    return torch.from_numpy(np.ascontiguousarray(B)).cuda()


def _grid(stretched):
    if not stretched:
        return cubic_grid(24, 21, 19)
    rng = np.random.default_rng(5)
    ax = []
    for n in (24, 21, 19):
        x = np.concatenate([[0.0], np.cumsum(rng.uniform(0.4, 1.6, n - 1))])
        ax.append(x / x[-1])
    return synth.stretched_grid(*ax)


def _field(g, seed, dtype):
    pos, q = synth.draw_charges(np.random.default_rng(seed), 5)
    return _dev(synth.charges_field(g, pos, q, dtype=dtype))


def _equal(a, b, label, rows=slice(None)):
    for k in a:
        if k.startswith("_"):
            continue
        if isinstance(a[k], dict):
            _equal(a[k], b[k], label, rows)
        elif a[k] is not None:
            x, y = to_np(a[k]), to_np(b[k])[rows]
            assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f"), (label, k)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 65, 257])
@pytest.mark.parametrize("prec", [F32X, F64], ids=["f32x", "f64"])
def test_short_lists_equal_long_ones(fq, n, prec):
    """The first n seeds of a list of 40000, alone: fewer and more than the 16 half lines
    of a wave, on uniform and stretched grids, with seeds on the faces, outside and on a
    null point's zero field."""
    import torch

    rng = np.random.default_rng(n)
    for stretched in (False, True):
        g = _grid(stretched)
        B = _field(g, 3, np.float32 if n % 2 else np.float64)
        s = rng.uniform(0.0, 1.0, (40000, 3)) * np.array(g.upper)
        s[1::5, 2] = 0.0
        s[2::5, 0] = g.upper[0]
        s[3::61, 1] = -0.25
        S = torch.from_numpy(s).cuda()
        _say(f"{n} of 40000 seeds, precision {prec}, stretched {stretched}")
        for tw in (True, False):
            p = dict(precision=prec, want_tw=tw)
            few = fq.trace(B, g, S[:n], params=fq.Params(**p))
            many = fq.trace(B, g, S, params=fq.Params(**p))
            torch.cuda.synchronize()
            _equal(few, many, (n, prec, stretched, tw), slice(0, n))


@pytest.mark.parametrize("nu,nv", [(2, 2), (3, 5), (8, 8), (17, 9), (70, 33)])
@pytest.mark.parametrize("method", ["I", "II"])
def test_small_maps_equal_batched_ones(fq, nu, nv, method):
    """A map by itself and the same map next to one of 420 x 420 points, at the bottom face
    and above it (rotated S0). graze = 2 sends every line through the FP64 pass, whose
    list is then longer than four lanes to a line are taken for."""
    import torch

    for stretched in (False, True) if method == "I" else (False,):
        g = _grid(stretched)
        B = _field(g, 7, np.float64)
        for z in (0.0, 0.21):
            small = Plane((0.23, 0.31, z), (1, 0, 0), (0, 1, 0), nu, nv, 0.4 / nu, 0.3 / nv)
            big = Plane((0.02, 0.03, 0.0), (1, 0, 0), (0, 1, 0), 420, 420, 0.0023, 0.0022)
            for kw in (dict(precision=F64), dict(precision=F32X), dict(precision=F32X, graze=2.0)):
                _say(f"{nu}x{nv} z {z}, method {method}, stretched {stretched}, {kw}")
                kw = dict(kw, method=fq.FQ_METHOD_II if method == "II" else fq.FQ_METHOD_I)
                st = torch.zeros(5, dtype=torch.int64, device="cuda")
                few = fq.q2d(B, g, small, fq.Params(**kw), want_lines=True)
                many = fq.q2d_batch([(B, g, small), (B, g, big)], fq.Params(stats=st, **kw), want_lines=True)
                torch.cuda.synchronize()
                if "graze" in kw:
                    assert int(st[4]) > 131072
                _equal(few, many[0], (nu, nv, z, method, stretched))


@pytest.mark.parametrize("n", [(5, 9, 6), (63, 7, 5), (64, 5, 9), (65, 6, 7), (129, 11, 5)])
@pytest.mark.parametrize("prec", [F32X, F64], ids=["f32x", "f64"])
def test_prep_at_row_and_wave_edges(fq, n, prec):
    """Node records of grids whose rows are shorter than, as long as and longer than a wave
    or two, and whose rows in y do not divide by the rows a thread keeps in flight: maps
    with twist against the oracle, from FP32 and FP64 fields."""
    import torch

    g = cubic_grid(*n)
    rng = np.random.default_rng(n[0])
    up = np.array(g.upper)
    M = rng.normal(size=(3, 3))
    M -= np.eye(3) * np.trace(M) / 3
    for dt in (np.float32, np.float64):
        B = synth.linear_field(g, 0.2 * M, [0.1, -0.1, 1.0], dtype=dt)
        k, j, i = np.meshgrid(*(np.arange(m) for m in reversed(n)), indexing="ij")
        B[0] += (0.02 * np.sin(0.7 * j + 0.4 * k)).astype(dt)
        B[1] += (0.02 * np.cos(0.6 * i - 0.3 * k)).astype(dt)
        pl = Plane((0.1 * up[0], 0.1 * up[1], 0.0), (1, 0, 0), (0, 1, 0), 23, 11, 0.8 * up[0] / 22, 0.8 * up[1] / 10)
        _say(f"prep {n}, precision {prec}, {np.dtype(dt)}")
        r = fq.q2d(_dev(B), g, pl, fq.Params(precision=prec), want_lines=True)
        torch.cuda.synchronize()
        compare_maps(r, oracle.q2d(B, g, pl, {"tol": 1e-10}), f"prep {n}")


@pytest.mark.parametrize("nu,nv", [(2, 2), (4, 4), (17, 3), (40, 21)])
@pytest.mark.parametrize("prec", [F32X, F64], ids=["f32x", "f64"])
def test_reverse_of_few_lines(fq, nu, nv, prec):
    """The reverse pass with four lanes to a half line, segments of 1, 5 and 32 steps: every
    replay finds its next checkpoint, and in FP64 the gradient does not depend on the
    segments (sums in another order, so 1e-12 of the largest value)."""
    import torch

    rng = np.random.default_rng(nu)
    for stretched in (False, True):
        g = _grid(stretched)
        B = _field(g, 11, np.float64)
        for z in (0.0, 0.21):
            pl = Plane((0.23, 0.31, z), (1, 0, 0), (0, 1, 0), nu, nv, 0.4 / nu, 0.3 / nv)
            dq = torch.from_numpy(rng.normal(size=(nv, nu))).cuda()
            dtw = torch.from_numpy(rng.normal(size=(nv, nu))).cuda()
            ref = None
            for seg in (32, 5, 1):
                _say(f"reverse {nu}x{nv} z {z}, precision {prec}, stretched {stretched}, segments of {seg}")
                st = torch.zeros(5, dtype=torch.int64, device="cuda")
                r = fq.backward(B, g, pl, fq.Params(precision=prec, stats=st, tape_steps=1000),
                                segment=seg, dq=dq, dtw=dtw)
                torch.cuda.synchronize()
                gb = to_np(r)
                assert int(st[0]) > 0 and int(st[2]) == 0 and int(st[3]) == 0, st
                assert np.all(np.isfinite(gb))
                if ref is None:
                    ref = gb
                if prec == F64:
                    lim = 1e-12 * np.abs(ref).max()
                    assert np.abs(gb - ref).max() <= lim, (seg, np.abs(gb - ref).max(), lim)


@pytest.mark.parametrize("n", [(2, 2, 2), (5, 9, 6), (16, 8, 8), (41, 5, 5), (33, 31, 2), (64, 16, 16), (201, 150, 150)])
@pytest.mark.parametrize("prec", [F32X, F64], ids=["f32x", "f64"])
def test_records_without_twist_at_block_edges(fq, n, prec):
    """Node records without twist (Bx, By, Bz, 0 of every node, in the type the trace
    computes in) of grids of fewer, exactly and more nodes than a block takes at once, and
    of more than all blocks do, from FP32 and FP64 fields: exact, read from the workspace."""
    import torch

    rng = np.random.default_rng(sum(n))
    for dt in (np.float32, np.float64):
        B = rng.normal(size=(3, n[2], n[1], n[0])).astype(dt)
        B[0].flat[3], B[2].flat[-1] = -0.0, np.nan
        _say(f"records without twist {n}, precision {prec}, {np.dtype(dt)}")
        r = fq.trace(_dev(B), cubic_grid(*n), torch.zeros((1, 3), dtype=torch.float64).cuda(),
                     params=fq.Params(precision=prec, want_tw=False, max_steps=50))
        torch.cuda.synchronize()
        want = np.zeros((n[0] * n[1] * n[2], 4), dtype=np.float32 if prec == F32X else np.float64)
        want[:, :3] = B.reshape(3, -1).T
        ws, bits = to_np(r["_ws"]), want.view(np.uint8).ravel()
        # (workspace arrays begin at multiples of 256 bytes)
        at = [o for o in range(0, len(ws) - len(bits) + 1, 256) if ws[o] == bits[0]
              and np.array_equal(ws[o:o + 64], bits[:64])]
        assert any(np.array_equal(ws[o:o + len(bits)], bits) for o in at)
