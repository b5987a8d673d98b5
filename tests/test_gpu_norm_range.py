"""Norms of few-row passes over residual streams whose scale jumps inside one projection: up by an outlier
channel, up from an (almost) empty row, down by a cancellation.  A normalised row is at most sqrt(d_model) per
unit gain whatever the stream does, so the stage has to agree with the oracle there as it does elsewhere."""
from dataclasses import replace

import pytest

from tests import stage_harness as H
from workload import CONFIGS

pytestmark = pytest.mark.gpu

_GPT2S = CONFIGS["gpt2s"]
_MODEL = replace(_GPT2S.model, n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=448, vocab=515)
_WIDE = replace(_MODEL, d_model=1088)
_MANY_COLUMNS = replace(_MODEL, ffn=9664, vocab=19300)        # two weight blocks a workgroup in gate||up and head
_CH = 37


def _outlier(w):
    """The first down projection adds some thousands to one channel of a row of rms 0.02."""
    w["w_down"][0, _CH] *= 2.0 ** 18


def _empty_rows(w):
    """Every other token has a zero embedding row; with a tiny eps the first norm scales by 1e6."""
    w["embed"][::2] = 0
    w["wo"][0] *= 64.0


def _cancelled(w):
    """A channel of 2^20 that the first attention takes back exactly: the normed row is 16 there and 0
    elsewhere, so every value is 16, and 256 of them times -256 are -2^20.  The rest of the row, rms 0.02,
    is what the second norm sees."""
    w["embed"][:, _CH] = 2.0 ** 20
    w["g_attn"][0] = 1.0
    w["wqkv"][0, 512:, _CH] = 1.0
    w["wo"][0] *= 2.0 ** -10
    w["wo"][0, _CH] = -256.0


_JUMPS = {"outlier": (_outlier, {}), "empty_rows": (_empty_rows, {"rms_eps": 1e-12}), "cancelled": (_cancelled, {})}


# (the cancellation is exact for 256 channels and half values only)
@pytest.mark.parametrize("model,n,jump", [(m, n, j) for m, n in ((_MODEL, 3), (_MODEL, 16), (_MODEL, 20), (_MODEL, 40), (_MANY_COLUMNS, 6)) for j in _JUMPS]
                         + [(m, n, j) for m, n in ((_WIDE, 5), (_WIDE, 20), (replace(_MODEL, dtype="fp32"), 9))
                            for j in ("outlier", "empty_rows")])
def test_stream_that_jumps(model, n, jump):
    change, fields = _JUMPS[jump]
    cfg = _GPT2S.with_(name="norm_range", model=replace(model, **fields), n_samples=n, prompt_len=(3, 5), gain_jitter=0.05)
    inp = H.make_inputs(cfg, n=n, max_len=4)
    for w in inp["weights"]:
        change(w)
    ref = H.oracle_stage(cfg, inp=inp)
    got = H.run_gpu_stage(cfg, ref, fused=False, R_t=0, chunk_tokens=64)
    H.compare_stage(cfg, ref, got)
