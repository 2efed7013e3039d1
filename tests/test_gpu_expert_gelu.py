"""GELU and its derivative in the expert's MLP at pre-activations far outside the
usual ones: a gain that leaves one feature and up weights of +-1 .. +-1e18 on it
give pre-activations of both signs and that size; the down weights undo the
scale.  There the derivative is exactly one or nothing, so the up gradient's rows
follow the fp64 oracle as at ordinary sizes: relative L2 per size 1.2e-2, three
bf16 factors (output gradient, its product, feature) of which each may round to
the other side, 3 x 2^-8."""
import numpy as np
import pytest

import workloads as W
from test_gpu_expert import _oracle_refs, expert_spec, run_experts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = (1.0, 8.0, 1e3, 1e6, 1e9, 1e12, 1e13, 1e15, 1e18)


def bits(x):
    u = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def test_gradients_at_large_preactivations():
    L, d, H, f = 1, 256, 4, 512
    wl = W.make_workload(expert_spec((L, d, H, f), 8, [(5, 7)]))
    w, rng = wl.experts[0]["layers"][0], np.random.default_rng(3)
    size = np.array([SIZES[u % len(SIZES)] for u in range(f)])
    up, down = rng.normal(0, 0.02, (f, d)), rng.normal(0, 0.02, (d, f)) / size
    up[:, 0] = size * np.where(np.arange(f) // len(SIZES) % 2, 1, -1)
    w["w_up"], w["w_down"] = bits(up), bits(down)
    w["g3"] = bits(np.eye(1, d)[0])
    st, targets, noisy = run_experts(wl)
    ref = _oracle_refs(wl, st, targets, noisy, [(0, True)])[(0, True)]["grads"]
    got = {k: t.cpu().numpy().astype(np.float64) for k, t in st.ios[0].layers[0].items()}
    for k, x in got.items():
        assert np.isfinite(x).all(), k
    for s in SIZES:
        rows = size == s
        a, b = got["w_up"][rows, 0], ref["0.w_up"][rows, 0]
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(f"size {s:g}: up gradient {err:.2e}", flush=True)
        assert err < 1.2e-2, s
