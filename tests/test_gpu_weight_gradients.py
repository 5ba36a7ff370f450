"""The size-generic weight-product kernel and the chunk reduction at their edges: one chunk, a
ragged last chunk, many chunks, one output tile a layer (a workgroup with two idle waves) and 64
of them, for both storage types, against the float64 backward oracle.  Biases of magnitude 1 to 1.5 keep
every decision away from its kink (|v|, |o| deviate from their bias by far less), so the
gradients have one correct value.  Bars: 6e-6 (fp32, gpu_util.TIGHT), 2e-2 (bf16)."""
import numpy as np
import pytest

import paper_2208_05419_amd as afno
from oracle import backward as ob
from paper_2208_05419_amd import synth
from gpu_util import TIGHT, dev_weights, say, to_dev, to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # B, H, W, nb, bs
    (1, 4, 2, 1, 16),      # 64 modes: two steps, one chunk
    (1, 20, 12, 1, 16),    # 224 modes, one chunk of seven steps
    (2, 45, 40, 1, 16),    # 2,688 modes, 21 chunks
    (3, 32, 60, 2, 48),  # 2,976 modes: 23 chunks, the last one shorter
    (1, 50, 54, 3, 80),
    (1, 36, 40, 1, 128),   # 64 tiles a layer
]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "B{}_H{}_W{}_nb{}_bs{}".format(*c))
def test_weight_gradients(case, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, H, W, nb, bs = case
    wl = synth.Workload("wgrad", B, H, W, nb * bs, nb, dtype, 0.01, 1.0)
    say(f"[wgrad] {case} {dtype}")
    rng = np.random.default_rng(H * W + bs)
    x_st, w_st = synth.make_x(wl, seed=1), synth.make_weights(wl, seed=1)
    for k in ("b1", "b2"):
        b = rng.choice([-1.0, 1.0], w_st[k].shape) * rng.uniform(1.0, 1.5, w_st[k].shape)
        w_st[k] = synth.quantize(b, dtype)
    g_st = synth.quantize(rng.standard_normal(x_st.shape), dtype)
    w = dev_weights(w_st, dtype)
    got = afno.filter_backward(to_dev(x_st, dtype), w["w1"], w["b1"], w["w2"], w["b2"],
                               to_dev(g_st, dtype), nb, wl.lam, wl.keep)
    torch.cuda.synchronize()
    wide = {k: synth.widen(v, dtype) for k, v in w_st.items()}
    ref = ob.filter_backward(synth.widen(x_st, dtype), wide["w1"], wide["b1"], wide["w2"],
                             wide["b2"], synth.widen(g_st, dtype), nb, wl.lam, wl.keep)
    for k in ("dx", "dw1", "db1", "dw2", "db2"):
        err = float(np.max(np.abs(to_f64(got[k]) - ref[k])) / np.max(np.abs(ref[k])))
        say(f"  {k} {err:.2e}")
        assert err <= TIGHT[dtype], (k, err)
