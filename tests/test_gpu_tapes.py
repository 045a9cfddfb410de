"""The adjoint of calls with more lines than take four lanes to a half line: their forward
pass records its checkpoints in the one-lane kernel, and the reverse pass replays them, in
FP64 with four lanes to a half line.

A small plane's forward pass takes four lanes. The same seeds inside a large plane, with
loss only there, give the same half lines, the same steps and, up to the order of the
sums, the same gradient.
"""

import sys

import numpy as np
import pytest

import synth
from synth import Plane, cubic_grid

from gpu_util import to_np

pytestmark = pytest.mark.gpu

F32X, F64 = 0, 1
# the node sums of both calls have the same terms (each half line's replay and reverse
# sweep is the same arithmetic), at most some 1e4 of them in any order: 1e4 x 1.1e-16 of the
# largest partial sum, which cancellation may leave ten times the largest result
SAME = 1e-11


@pytest.fixture(scope="module")
def fq():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2208_12569_amd as m

    m._lib.load()
    return m


def _grid(stretched):
    if not stretched:
        return cubic_grid(24, 21, 19)
    rng = np.random.default_rng(5)
    ax = []
    for n in (24, 21, 19):
        x = np.concatenate([[0.0], np.cumsum(rng.uniform(0.4, 1.6, n - 1))])
        ax.append(x / x[-1])
    return synth.stretched_grid(*ax)


@pytest.mark.parametrize("stretched", [False, True], ids=["uniform", "stretched"])
@pytest.mark.parametrize("prec", [F32X, F64], ids=["f32x", "f64"])
@pytest.mark.parametrize("z,side", [(0.0, 270), (0.25, 192)], ids=["face", "interior"])
@pytest.mark.parametrize("tw", [True, False], ids=["twist", "no twist"])
def test_adjoint_above_the_four_lane_limit(fq, stretched, prec, z, side, tw):
    import torch

    g = _grid(stretched)
    pos, q = synth.draw_charges(np.random.default_rng(11), 5)
    B = torch.from_numpy(np.ascontiguousarray(synth.charges_field(g, pos, q, dtype=np.float64))).cuda()
    # seeds at multiples of 1/512: the same numbers in both planes
    d, (i0, j0), (nu, nv) = 1.0 / 512, (83, 71), (27, 23)
    big = Plane((0.25, 0.125, z), (1, 0, 0), (0, 1, 0), side, side, d, d)
    small = Plane((0.25 + i0 * d, 0.125 + j0 * d, z), (1, 0, 0), (0, 1, 0), nu, nv, d, d)
    rng = np.random.default_rng(side)
    loss = np.zeros((2, nv, nu))
    loss[:, 1:-1, 1:-1] = rng.normal(size=(2, nv - 2, nu - 2))  # stencils inside the small plane
    out = {}
    for name, pl in (("large", big), ("small", small)):
        w = np.zeros((2, pl.nv, pl.nu))
        if name == "large":
            w[:, j0:j0 + nv, i0:i0 + nu] = loss
        else:
            w[:] = loss
        w = torch.from_numpy(w).cuda()
        print(f"[gpu case] {name} {pl.nu}x{pl.nv} z {z}, precision {prec}, stretched {stretched}, twist {tw}", flush=True)
        sys.stdout.flush()
        st = torch.zeros(5, dtype=torch.int64, device="cuda")
        p = fq.Params(precision=prec, stats=st, tape_steps=512, want_tw=tw)
        gb = fq.backward(B, g, pl, p, segment=7, dq=w[0].contiguous(), dtw=w[1].contiguous() if tw else None)
        torch.cuda.synchronize()
        out[name] = to_np(gb), [int(x) for x in st]
    (a, sa), (b, sb) = out["large"], out["small"]
    assert sb[0] > 0 and sb[2] == 0 and sb[3] == 0, sb  # half lines; replay mismatches; dropped
    assert sa == sb
    assert np.all(np.isfinite(b)) and np.abs(b).max() > 0
    assert np.abs(a - b).max() <= SAME * np.abs(b).max(), np.abs(a - b).max() / np.abs(b).max()
