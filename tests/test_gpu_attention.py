"""The attention at every number of row tiles, with committed prefixes that end on, before and after a stage
of 64 keys, one sequence (splits of the committed length) and a ragged batch (work items), against the oracle.

Tolerance.  As for the other products: queries, probabilities and outputs carry 16 bits (2^-17 per site), sums
are f32; one layer has seven such sites and the final norm, 8 * 2^-17 = 6e-5.  The softmax weights come from a
hardware exp2 of 1 ulp on arguments below 2^4 in magnitude: 2^-20.
"""
import numpy as np
import pytest

from gpu_common import log, rel_err
from oracle import nld_oracle as O
from synth.workloads import LazyWeights, ModelShape, prefix_kv, tokens as synth_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TOL = 6.5e-5
CAP = 448


def shape(D):
    return ModelShape(n_layers=1, hidden=128, n_q_heads=4, n_kv_heads=1, head_dim=D, ffn=96, vocab=200)


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_05722_amd import runtime
    return runtime


@pytest.fixture(scope="module", params=[64, 128])
def model(R, request):
    s = shape(request.param)
    src = LazyWeights(s, 21)
    return {"shape": s, "w": O.OracleWeights(s, src, np.float32), "m": R.DeviceModel(s, src)}


def check(R, t, lens, k, mode, bidir=0):
    s, batch = t["shape"], len(lens)
    okv, cache = O.OracleKV(s, batch, CAP, np.float32), R.DeviceCache(s, batch, CAP)
    kb, vb = prefix_kv(s, 21, 0, batch, CAP)
    okv.set_prefix_bf16(0, kb, vb, np.asarray(lens))
    cache.load_prefix(0, kb, vb)   # rows at and past a length hold keys that must not be seen
    cache.set_lengths(lens)
    tok = synth_tokens(s, 21, "attn.%d.%d" % (batch, k), (batch, k))
    ref, _, _ = O.block_forward(t["w"], okv, tok, mode, bidir)
    ws = R.Workspace(t["m"], batch, k, CAP)
    logits, _ = R.block_forward(t["m"], cache, ws, torch.from_numpy(tok).cuda(),
                                R.VERIFY if mode == O.VERIFY else R.DRAFT, bidir)
    assert R.read_device_status(ws) == 0
    e = rel_err(logits.cpu().numpy(), ref)
    log("attention D %d lengths %s k %d %s: rel err %.2e" % (s.head_dim, lens, k, mode, e))
    assert e <= TOL


# with 4 query heads per KV head: 1, 1, 2, 3, 4 (two wavefronts per row tile), 5, 8, 9, 12 (one each), 13, 16 row
# tiles (two row slices)
KS = [1, 4, 5, 12, 16, 17, 32, 33, 48, 50, 64]


@pytest.mark.parametrize("k", KS)
def test_one_sequence(R, model, k):
    for P in (0, 1, 63, 64, 65, 200, CAP - 64):
        check(R, model, [P], k, O.VERIFY)
    check(R, model, [130], k, O.DRAFT, min(1, k))


@pytest.mark.parametrize("keys", [64, 128, 384])
@pytest.mark.parametrize("k", KS)
def test_ragged_batch(R, model, monkeypatch, k, keys):
    monkeypatch.setenv("NLD_ATTN_ITEM_KEYS", str(keys))
    check(R, model, [0, 64, 1, CAP - 64, 63, 129, 192], k, O.VERIFY)
    check(R, model, [65, 0, 128], k, O.DRAFT)


@pytest.mark.parametrize("batch,k", [(515, 1), (200, 17)])
def test_merge_of_many_rows(R, model, monkeypatch, batch, k):
    """The merge that takes a row to D / 8 lanes (from 512 workgroups on): rows that do not fill its last
    workgroup, one to seven parts a row, sequences without a prefix."""
    monkeypatch.setenv("NLD_ATTN_ITEM_KEYS", "64")
    lens = [(i * 53) % (CAP - 17) for i in range(batch)]
    check(R, model, lens, k, O.VERIFY)
