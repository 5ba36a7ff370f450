"""The size-generic column kernels, forward and backward, at every height H = 2^a 3^b 5^c <= 192
(every split of the H transforms, every count of 16-row tiles) against the float64 oracle, over
block sizes of 16 to 128, hidden sizes below and above the block size, cutoffs that empty whole
row tiles, and both storage types; and the forward without prepared weight words, which the
allocation-free entry point takes where they would not fit its workspace.

Bars: fp32 6e-6 (gpu_util.TIGHT), bf16 2e-2 of max |r|.  The backward's biases have
magnitude 1 to 1.5 and its weights a standard deviation of 0.01, so that v and o stay within
0.01 sqrt(2 128 1.6) = 0.2 (one deviation, the widest block, hidden units up to 1.6) of their
biases: a kink is five deviations off, and a decision within bf16 rounding of one is not expected
in the 10^5 of a case (weights of 0.02 put one there in a case of 108 x 128).  The gradients then
have one value."""
import numpy as np
import pytest

import paper_2208_05419_amd as afno
from oracle import backward as ob
from paper_2208_05419_amd import synth
from gpu_util import TIGHT, dev_weights, max_rel, oracle_run, say, to_dev, to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HEIGHTS = [n for n in range(1, 193)
           if any(n == 2 ** a * 3 ** b * 5 ** c for a in range(8) for b in range(5) for c in range(4))]
BLOCKS = (16, 48, 128, 80, 112, 32, 96, 64)


@pytest.fixture(scope="module", autouse=True)
def _generic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    afno.set_kernel_path(afno.AFNO_PATH_GENERIC)
    yield
    afno.set_kernel_path(afno.AFNO_PATH_AUTO)


def _fits(H, bs, hs, dtype):
    es, pad, h16 = (4, 4, (H + 15) // 16 * 16) if dtype == "fp32" else (2, 8, (H + 15) // 16 * 16)
    lds = h16 * (2 * bs + pad) * es + H * 8 * (33 if bs % 32 == 0 else 17)
    lds += h16 * (2 * hs + pad) * es if hs != bs else 0
    return lds <= 160 * 1024


def _choose(H, dtype):
    i = HEIGHTS.index(H)
    for k in range(len(BLOCKS)):
        bs = BLOCKS[(i + k) % len(BLOCKS)]
        for hs in ((bs, 2 * bs, max(16, bs // 2 // 16 * 16))[i % 3], bs):
            if hs <= 256 and _fits(H, bs, hs, dtype):
                return bs, hs, (1.0, 0.7, 0.3)[(i // 3) % 3]
    raise AssertionError


@pytest.mark.parametrize("H", HEIGHTS)
def test_forward_height(H):
    for dtype in ("fp32", "bf16"):
        bs, hs, keep = _choose(H, dtype)
        keep = keep if int((H // 2 + 1) * keep) and int(3 * keep) else 1.0
        wl = synth.Workload("height", 2, H, 4, 2 * bs, 2, dtype, 0.01, keep, weight_std=0.1, hidden=hs)
        say(f"[height] H={H} bs={bs} hs={hs} {dtype} keep={keep}")
        x_st, w_st = synth.make_x(wl, seed=H), synth.make_weights(wl, seed=H)
        x, w = to_dev(x_st, dtype), dev_weights(w_st, dtype)
        args = (x, w["w1"], w["b1"], w["w2"], w["b2"], 2, wl.lam, keep)
        out, delta = afno.filter_forward(*args), afno.filter_stage(*args, afno.AFNO_STAGE_DELTA)
        mixed = afno.filter_stage(*args, afno.AFNO_STAGE_MIXED)
        torch.cuda.synchronize()
        ref, st = oracle_run(x_st, w_st, wl, stages=True)
        m = to_f64(mixed)
        errs = (max_rel(to_f64(out), ref), max_rel(to_f64(delta), st["delta"]),
                max_rel(m[..., 0] + 1j * m[..., 1], st["spec_mlp"]))
        say("  out {:.2e}  delta {:.2e}  mixed {:.2e}".format(*errs))
        assert max(errs) <= TIGHT[dtype], errs


@pytest.mark.parametrize("H", HEIGHTS)
def test_backward_height(H):
    for dtype in ("fp32", "bf16"):
        bs, _, keep = _choose(H, dtype)
        keep = keep if int((H // 2 + 1) * keep) and int(3 * keep) else 1.0
        if not _fits(H + 16, bs, bs, dtype):  # the masks' share of the limit
            bs = 16
        wl = synth.Workload("height", 1, H, 4, bs, 1, dtype, 0.01, keep, weight_std=0.01)
        say(f"[height backward] H={H} bs={bs} {dtype} keep={keep}")
        rng = np.random.default_rng(H)
        x_st, w_st = synth.make_x(wl, seed=H), synth.make_weights(wl, seed=H)
        for k in ("b1", "b2"):
            b = rng.choice([-1.0, 1.0], w_st[k].shape) * rng.uniform(1.0, 1.5, w_st[k].shape)
            w_st[k] = synth.quantize(b, dtype)
        g_st = synth.quantize(rng.standard_normal(x_st.shape), dtype)
        w = dev_weights(w_st, dtype)
        got = afno.filter_backward(to_dev(x_st, dtype), w["w1"], w["b1"], w["w2"], w["b2"],
                                   to_dev(g_st, dtype), 1, wl.lam, keep)
        torch.cuda.synchronize()
        wide = {k: synth.widen(v, dtype) for k, v in w_st.items()}
        ref = ob.filter_backward(synth.widen(x_st, dtype), wide["w1"], wide["b1"], wide["w2"],
                                 wide["b2"], synth.widen(g_st, dtype), 1, wl.lam, keep)
        for k in ("dx", "dw1", "db1", "dw2", "db2"):
            den = float(np.max(np.abs(ref[k]))) or 1.0
            err = float(np.max(np.abs(to_f64(got[k]) - ref[k]))) / den
            say(f"  {k} {err:.2e}")
            assert err <= TIGHT[dtype], (dtype, bs, k, err)


@pytest.mark.parametrize("dtype,nb", [("fp32", 256), ("bf16", 512)])
def test_noalloc_without_room_for_prepared_words(dtype, nb):
    """Blocks of 128 whose words alone take 128 MiB; same bits without them."""
    wl = synth.Workload("plain", 2, 3, 4, nb * 128, nb, dtype, 0.01, 1.0)
    x, w = to_dev(synth.make_x(wl, seed=1), dtype), dev_weights(synth.make_weights(wl, seed=1), dtype)
    args = (x, w["w1"], w["b1"], w["w2"], w["b2"], wl.num_blocks, wl.lam, wl.keep)
    want = afno.filter_forward(*args)
    got = torch.full_like(x, float("nan"))
    afno.filter_forward_noalloc(*args, got)
    torch.cuda.synchronize()
    assert torch.equal(want, got)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_softshrink_of_nan_is_zero(dtype):
    """S(v) = v - lam, v + lam, else 0: a value that is neither above lam nor below -lam gives 0,
    NaN included (the oracle's definition)."""
    wl = synth.Workload("nan", 1, 24, 12, 96, 2, dtype, 0.01, 0.7, weight_std=0.1)
    x_st, w_st = synth.make_x(wl, seed=5), synth.make_weights(wl, seed=5)
    w_st["b2"] = w_st["b2"].copy()
    w_st["b2"][1, 7, 0] = np.float32("nan") if dtype == "fp32" else 0x7FC0
    x, w = to_dev(x_st, dtype), dev_weights(w_st, dtype)
    out = afno.filter_forward(x, w["w1"], w["b1"], w["w2"], w["b2"], 2, wl.lam, wl.keep)
    torch.cuda.synchronize()
    ref, _ = oracle_run(x_st, w_st, wl, stages=True)
    assert np.isfinite(ref).all()
    assert max_rel(to_f64(out), ref) <= TIGHT[dtype]
