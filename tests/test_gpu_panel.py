"""The panel GEMM: each workgroup shape and K-slice count against
the oracle, at the sizes where tiles, stages and slices do not divide.

Tolerance.  Every product carries its activation as a bf16 value and its bf16 remainder, a relative error of
at most 2^-17 per site, on f32 sums.  A pass of two layers has seven such sites per layer and the final norm:
at most 15 * 2^-17 = 1.2e-4 where nothing amplifies them; the oracle's own f32 sums are below 1e-5.
"""
import numpy as np
import pytest

from gpu_common import ArraySource, BF16_ONE, int_to_bf16_bits, log, rel_err
import synth
from oracle import nld_oracle as O
from synth.workloads import LazyWeights, ModelShape, SHAPE_TINY, tokens as synth_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TOL = 1.2e-4

# hidden 160: five k-steps (no whole number of stages); ffn 88: two k-steps and a partial one, 11 gate/up
# tiles; vocab 333: a partial column tile; a LoRA rank of one k-step
ODD = ModelShape(n_layers=2, hidden=160, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=88, vocab=333, lora_rank=32,
                 lora_alpha=64.0)
LONG = ModelShape(**{**SHAPE_TINY.__dict__, "hidden": 512, "ffn": 1072})   # enough stages for several slices
SHAPES = {2: range(0, 5), 4: range(5, 9), 8: range(9, 13), 1: range(13, 17)}   # by row tiles
STAGE = {1: 4, 2: 4, 4: 4, 6: 4, 13: 4, 14: 4, 15: 4, 16: 8}                   # k-steps per stage (2 else)
NAMES = ("O", "DOWN", "QKV", "GU", "LM")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_05722_amd import runtime
    return runtime


@pytest.fixture(scope="module", params=["odd", "long"])
def model(R, request):
    shape = ODD if request.param == "odd" else LONG
    src = LazyWeights(shape, 11)
    return {"shape": shape, "w": O.OracleWeights(shape, src, np.float32), "m": R.DeviceModel(shape, src)}


def run(R, t, batch, k, mode):
    shape = t["shape"]
    tok = synth_tokens(shape, 11, "panel.%d.%d" % (batch, k), (batch, k))
    okv = O.OracleKV(shape, batch, 128, np.float32)
    ref, _, _ = O.block_forward(t["w"], okv, tok, mode)
    cache, ws = R.DeviceCache(shape, batch, 128), R.Workspace(t["m"], batch, k, 128)
    m = R.VERIFY if mode == O.VERIFY else R.DRAFT
    got = [R.block_forward(t["m"], cache, ws, torch.from_numpy(tok).cuda(), m) for _ in range(2)]
    assert R.read_device_status(ws) == 0
    g = got[0][0].cpu().numpy()
    assert torch.equal(got[0][0], got[1][0])   # slices add up in one order, whichever arrives last
    assert np.array_equal(got[0][1].cpu().numpy(), np.argmax(g, axis=-1))
    return rel_err(g, ref)


@pytest.mark.parametrize("batch,k", [(1, 1), (3, 3), (1, 16), (1, 17), (1, 32), (3, 11), (1, 64), (5, 13), (2, 64), (3, 43)])
@pytest.mark.parametrize("slices", [1, 3])
def test_every_shape(R, model, monkeypatch, batch, k, slices):
    """Up to 16, 32, 64 and more than 64 rows (one and two row groups), every shape forced on every projection
    that takes it (up to 16 rows O has a kernel of its own, and down up to 8)."""
    rt = 1 if batch * k <= 16 else 2 if batch * k <= 32 else 4 if batch * k <= 64 else 8
    for i in SHAPES[rt]:
        for n in NAMES:
            steps = (model["shape"].ffn if n == "DOWN" else model["shape"].hidden) // 32
            monkeypatch.setenv("NLD_PANEL_" + n, "%d,%d" % (i, max(1, min(slices, steps // STAGE.get(i, 2)))))
        for mode in (O.VERIFY, O.DRAFT):
            e = run(R, model, batch, k, mode)
            log("panel shape %d slices %d rows %d %s: rel err %.2e" % (i, slices, batch * k, mode, e))
            assert e <= TOL


@pytest.mark.parametrize("batch,k", [(1, 8), (1, 9), (1, 16), (1, 17), (2, 32), (2, 33), (9, 15)])
def test_planned(R, model, batch, k):
    """The plans the library picks, on both sides of each row-tile boundary."""
    for mode in (O.VERIFY, O.DRAFT):
        assert run(R, model, batch, k, mode) <= TOL


@pytest.mark.parametrize("batch,k", [(1, 1), (3, 2), (1, 8)])
def test_down_of_few_rows(R, model, monkeypatch, batch, k):
    """Down of up to 8 rows on the panel GEMM, as where the split-K kernel's groups leave no room for two slices."""
    monkeypatch.setenv("NLD_NO_SPLITK", "1")
    for mode in (O.VERIFY, O.DRAFT):
        assert run(R, model, batch, k, mode) <= TOL


def bf16_parts(v):
    """v as a sum of three bf16 values (bits)."""
    parts, rest = [], np.float64(v)
    for _ in range(3):
        bits = np.uint16(np.float32(rest).view(np.uint32) >> 16)   # truncated, so that the rest is exact
        parts.append(bits)
        rest -= np.float64(np.array(np.uint32(bits) << 16, np.uint32).view(np.float32))
    return parts


@pytest.mark.parametrize("batch,k", [(1, 1), (1, 8), (1, 32), (1, 64), (2, 64)])
@pytest.mark.parametrize("large", [False, True])
def test_swiglu_of_large_gates(R, batch, k, large):
    """Gates past the point where exp(-gate) overflows (88.73) give -0 like any other large negative gate,
    large positive ones the gate itself.  Every token's embedding is one and the gates are set by
    the weights: gate f goes to column f of the residual.  One gate in eight is ordinary."""
    shape = ModelShape(n_layers=1, hidden=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=96, vocab=200, rms_eps=0.0)
    h, f = shape.hidden, shape.ffn
    gates = list(np.linspace(-104.0, -88.73, 72)) + [-80.0, -88.7, -88.72, -88.8, -93.0, -95.0, -97.0, -99.0, -101.0,
                                                     -103.97, -110.0, -1e4]
    gates += [1e4] * 2 if large else [-1e30] * 2
    gates += [0.5, -0.5, 2.0, -2.0, 5.0, -5.0, 20.0, -20.0, 1.0, -1.0]
    zero = lambda o, i: np.zeros((o, i), dtype=np.uint16)   # noqa: E731
    gate, up, down = zero(f, h), zero(f, h), zero(h, f)
    for i, g in enumerate(gates):
        gate[i, :3] = bf16_parts(g)
        up[i, 0] = down[i, i] = BF16_ONE
    ones = lambda n: np.full(n, BF16_ONE, dtype=np.uint16)   # noqa: E731
    layer = {"attn_norm": ones(h), "wq": zero(shape.q_dim, h), "wk": zero(shape.kv_dim, h), "wv": zero(shape.kv_dim, h),
             "wo": zero(h, shape.q_dim), "ffn_norm": ones(h), "w_gate": gate, "w_up": up, "w_down": down}
    lm = int_to_bf16_bits(synth.uniform_int(3, "swiglu.lm", (shape.vocab, h), -8, 8))
    src = ArraySource([layer], np.full((shape.vocab, h), BF16_ONE, dtype=np.uint16), lm, ones(h))
    t = {"shape": shape, "w": O.OracleWeights(shape, src, np.float64), "m": R.DeviceModel(shape, src)}
    with np.errstate(over="ignore"):
        for mode in (O.VERIFY, O.DRAFT):
            assert run(R, t, batch, k, mode) <= TOL   # false for a NaN


@pytest.mark.parametrize("k", [8, 32, 64, 100])
@pytest.mark.parametrize("bits", [0x7FC0, 0xFFC0])
@pytest.mark.parametrize("columns", [slice(17, 18), slice(0, 48)])
def test_nan_logit_reaches_the_confidence(R, k, bits, columns):
    """A NaN logit of either sign is part of its row's softmax sum: the confidence is NaN, also where every column that
    a wavefront takes (16, 32 or 48 of them) is NaN."""
    shape = ModelShape(n_layers=1, hidden=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=96, vocab=200)
    src = LazyWeights(shape, 5)
    lm = np.array(src.lm_head, copy=True)
    lm[columns] = bits
    model = R.DeviceModel(shape, ArraySource([src.layer(0)], src.embed, lm, src.final_norm))
    batch, k = (2, 50) if k > 64 else (1, k)
    cache, ws = R.DeviceCache(shape, batch, 128), R.Workspace(model, batch, k, 128)
    block = torch.from_numpy(synth_tokens(shape, 5, "panel.nan", (batch, k))).cuda()
    block[:, 1:] = shape.mask_token_id
    out = R.denoise_step(model, cache, ws, block, 0.5)
    assert torch.isnan(out["confidence"]).all()
    assert R.read_device_status(ws) == 0


@pytest.mark.parametrize("batch,k", [(1, 1), (1, 33), (1, 64), (4, 25), (2, 64)])
def test_narrowest_model(R, batch, k):
    """Hidden 32, the smallest there is: two sums of squares per row are all that its statistics have room for."""
    shape = ModelShape(n_layers=2, hidden=32, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=40, vocab=77)
    src = LazyWeights(shape, 13)
    t = {"shape": shape, "w": O.OracleWeights(shape, src, np.float32), "m": R.DeviceModel(shape, src)}
    for mode in (O.VERIFY, O.DRAFT):
        e = run(R, t, batch, k, mode)
        log("hidden 32 rows %d %s: rel err %.2e" % (batch * k, mode, e))
        assert e <= TOL


@pytest.mark.parametrize("shape_env", ["", "15,1"])
def test_small_products_are_not_lost(R, monkeypatch, shape_env):
    """At up to 16 rows the lo halves' products have a sum of their own.  One value in 32 is
    (1 + 2^-7)^2 = (1 + 2^-6) + 2^-14 and the others are 1, against weights of 1: the hi sums are exact, and of one
    wavefront's 128 lo products of 2^-14 the half that meets a hi sum above 2048 would round away, 1e-6 of the
    result.  What is left is the rounding of 1/rms, the scaling and the sum: 4 * 2^-24, taken twice."""
    shape = ModelShape(n_layers=1, hidden=4096, n_q_heads=1, n_kv_heads=1, head_dim=64, ffn=8, vocab=256, rms_eps=0.0)
    h = shape.hidden
    v = np.full(h, BF16_ONE, dtype=np.uint16)
    v[::32] += 1   # the next bf16 value, 1 + 2^-7
    zero = lambda o, i: np.zeros((o, i), dtype=np.uint16)   # noqa: E731
    layer = {"attn_norm": v, "wq": zero(64, h), "wk": zero(64, h), "wv": zero(64, h), "wo": zero(h, 64), "ffn_norm": v,
             "w_gate": zero(8, h), "w_up": zero(8, h), "w_down": zero(h, 8)}
    src = ArraySource([layer], np.tile(v, (shape.vocab, 1)), np.full((shape.vocab, h), BF16_ONE, dtype=np.uint16), v)
    if shape_env:
        monkeypatch.setenv("NLD_PANEL_LM", shape_env)
    model, cache = R.DeviceModel(shape, src), R.DeviceCache(shape, 1, 64)
    ws = R.Workspace(model, 1, 8, 64)
    logits, _ = R.block_forward(model, cache, ws, torch.zeros(1, 8, dtype=torch.int32, device="cuda"), R.VERIFY)
    a = 1 + 2.0 ** -7
    ref = h / 32 * (31 + a * a) / np.sqrt((31 + a * a) / 32)
    e = np.max(np.abs(logits.cpu().numpy().astype(np.float64) / ref - 1))
    log("small products: rel err %.2e" % e)
    assert e <= 8 * 2.0 ** -24
