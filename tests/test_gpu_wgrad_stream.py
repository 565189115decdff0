"""Stages whose weight gradients and token sort run on the second stream (more than 2^17 activation
elements: smaller ones run them in order): the waits between the streams with an fp32 stage, a tied head
beside the embedding scatter and several microbatches in flight, against the oracle and run against run."""
import numpy as np
import pytest

import datagen
import oracle
from gpu_common import hp_of, log, run_gpu, run_oracle
from test_gpu_stage import _compare

pytestmark = pytest.mark.gpu

BASE = dict(n_blocks=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=512, seq_len=256, micro_batch=3,
            microbatches_per_step=3, max_inflight=2)
# name: (dtype, first, last, tied, overlap mode)
CASES = {
    "f32-tied": ("f32", True, True, True, 0),
    "f32-middle": ("f32", False, False, False, 1),
    "f32-last": ("f32", False, True, False, 2),
    "bf16-tied": ("bf16", True, True, True, 2),
    "bf16-first": ("bf16", True, False, False, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_second_stream(name):
    dt, first, last, tied, mode = CASES[name]
    w = datagen.SMALL.with_(name=name, dtype=dt, vocab=500 if first or last else 0, first_stage=first,
                            last_stage=last, tie_embedding=tied, **BASE)
    assert w.seq_len * w.micro_batch * w.d_model > 1 << 17
    steps, grads, ys = 4, (0, 3), () if last else (0,)
    log(f"second stream: {name}")
    p0 = datagen.init_params(w)
    runs = [run_gpu(w, steps, hp_of(w), p0, grad_steps=grads, y_steps=ys, upd_steps=(1, 2), early_update=mode > 0,
                    overlap_mode=max(mode, 1)) for _ in range(2)]
    a, b = runs
    assert a["losses"] == b["losses"]
    for t in grads:
        for n in p0:
            assert np.array_equal(a["grads"][t][n], b["grads"][t][n]), f"gradient {n} of step {t}"
    for pre in ("", "m.", "v.", "u_prev."):
        for n in p0:
            assert np.array_equal(a["final"][pre][n], b["final"][pre][n]), f"final {pre}{n}"
    o = run_oracle(w, steps, oracle.hparams_of(w), p0, grad_steps=grads, y_steps=ys)
    _compare(w, a, o, 1e-4 if dt == "f32" else 2e-2, grads, name, w.ef_lambda, state_tol=None if dt == "f32" else 5e-2)
