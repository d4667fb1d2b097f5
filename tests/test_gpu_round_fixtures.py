"""One full outer round (N sync events = one Delayed-Nesterov period, Alg. 3) at FULL model shapes
and batch on the GPU against fixtures the CPU oracle wrote (tests/golden/make_full_size_round.py,
which calls only oracle/ and als_inputs): lm20m (20M-class, H = 50: 128 + 53 worker
steps), lm150m (150M-class) and lm20m_k16 (16 workers), the last two with the DyLU maximum H
lowered to the value stored in the fixture so that the numpy oracle finishes in minutes.

Checked: DyLU step counts and event order bit for bit; every per-step loss; the server
parameters after every group of events and the outer momentum, element by element on a strided
sample of every tensor; per-tensor norms over the WHOLE tensors."""
import os

import numpy as np
import pytest
import torch

import als_inputs as I
import paper_2401_09135_amd as A
from oracle import lm

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")

# the task's bars for bf16 operands with fp32 accumulation
LOSS_RTOL, THETA_REL_L2 = 2e-3, 5e-3
# Per-step loss while the loss is still falling fast: a relative error eps of a parameter update
# changes the next loss by about eps x (the loss change that update causes), to first order.  With
# bf16 operands the update error is a few 1e-2 of the update (measured against the oracle here, and
# the oracle with bf16-rounded operands sits as far from the plain one: test_gpu_parity.py,
# test_bf16_operand_rounding_sets_the_scale_of_the_deviation), so a step across which the reference
# loss changes by D may deviate by UPDATE_REL x D on top of the 2e-3 bar.  In the first steps from
# random weights at lr 1e-3 the loss falls by up to 2 nats per step; once it changes by less than
# 2 % per step the plain bar is all that is left.
UPDATE_REL = 0.1


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def _tensor_norms(v, w):
    out, off = [], 0
    for _n, shape, _k in lm.param_layout(w):
        n = int(np.prod(shape))
        out.append(float(np.sqrt(np.sum(np.square(v[off:off + n], dtype=np.float64)))))
        off += n
    return np.asarray(out)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name", ["lm20m", "lm150m", "lm20m_k16"])
def test_one_outer_round_full_size_against_oracle_fixture(name):
    path = os.path.join(GOLDEN, f"round_{name}.npz")
    if not os.path.exists(path):
        pytest.skip(f"{path} has not been generated")
    fx = np.load(path)
    w = I.workload(name)
    w["H"] = int(fx["H"])
    n_events = int(fx["n_events"])
    assert n_events == w["N"]
    theta0 = I.theta0(lm.param_layout(w), w["seed"])
    idx = fx["idx"]
    ev_idx = idx[::int(fx["ev_stride"])]
    seen = {}

    def on_group(ctx, last_event):
        seen[last_event] = ctx.get_vector("theta")[ev_idx]

    got = A.run_async(w, theta0, lambda i: I.TokenStream(w["seed"], i, w["B"], w["S"], w["V"]),
                      n_events=n_events, on_group=on_group)
    got["ctx"].close()

    # bit-exact quantities
    assert got["steps"].tolist() == fx["steps"].tolist()
    assert got["ev_worker"].tolist() == fx["ev_worker"].tolist()
    assert got["ev_time"].tolist() == fx["ev_time"].tolist()
    assert got["t"] == n_events

    # every per-step loss
    worst_loss = worst_calm = 0.0
    n_calm = n_steps = 0
    for i in range(w["k"]):
        ref = fx[f"loss_{i}"]
        assert len(got["losses"][i]) == len(ref), i
        if len(ref):
            g_l = np.asarray(got["losses"][i], np.float64)
            change = np.abs(np.diff(ref, prepend=ref[0]))
            err = np.abs(g_l - ref)
            assert (err <= LOSS_RTOL * np.abs(ref) + UPDATE_REL * change).all(), (i, g_l.tolist(), ref.tolist())
            worst_loss = max(worst_loss, float(np.max(err / np.abs(ref))))
            calm = change < 0.02 * np.abs(ref)
            if calm.any():
                worst_calm = max(worst_calm, float(np.max(err[calm] / np.abs(ref[calm]))))
            n_calm += int(calm.sum())
            n_steps += len(ref)

    # server parameters after every applied group, on the sample: the growth over the round
    growth = {e: _rel(v, fx["theta_ev"][e]) for e, v in sorted(seen.items())}
    th, mo, de = got["theta"], got["m"], got["delta"]
    rel_theta = _rel(th[idx], fx["theta"])
    rel_upd = _rel(th[idx] - theta0[idx], fx["theta"] - theta0[idx])
    rel_m = _rel(mo[idx], fx["m"])
    tn = _tensor_norms(th, w)
    worst_norm = float(np.max(np.abs(tn - fx["tnorm_theta"]) / fx["tnorm_theta"]))
    line = (f"round {name} H={w['H']} ({n_steps} worker steps): max loss rel {worst_loss:.3e} over all steps, "
            f"{worst_calm:.3e} over the {n_calm} steps across which the loss changes by < 2 %, "
            f"theta rel-L2 after each group {', '.join(f'{e + 1}: {r:.3e}' for e, r in growth.items())}, "
            f"final theta rel-L2 {rel_theta:.3e} (update {rel_upd:.3e}, momentum {rel_m:.3e}), "
            f"worst per-tensor norm deviation {worst_norm:.3e}")
    print(line)
    log = os.environ.get("ALS_PARITY_LOG")
    if log:
        with open(log, "a") as f:
            f.write(line + "\n")
    assert worst_calm < LOSS_RTOL
    assert rel_theta < THETA_REL_L2
    assert max(growth.values()) < THETA_REL_L2
    assert worst_norm < THETA_REL_L2
    assert not de.any()                                  # the N-th event leaves Delta exactly zero
    assert not fx["delta"].any()
    # element by element: no sampled parameter further from the oracle's than 10 x the norm-level
    # bar times the RMS of its tensor, plus half the largest update any sampled element of that
    # tensor received.  (In its first steps AdamW moves every element by about the learning rate
    # whatever the size of its gradient, so an element whose gradient is rounding noise moves by
    # +-lr per step in a direction bf16 and float32 need not agree on: single elements may differ
    # by a fraction of the update scale.  A wrong element, as opposed to rounding, is far outside.)
    off = 0
    pos = 0
    for tname, shape, _k in lm.param_layout(w):
        n = int(np.prod(shape))
        sel = (idx >= off) & (idx < off + n)
        cnt = int(sel.sum())
        ref_t, got_t = fx["theta"][pos:pos + cnt], th[idx[pos:pos + cnt]]
        rms = float(np.sqrt(np.mean(np.square(ref_t, dtype=np.float64))))
        upd = float(np.max(np.abs(ref_t - theta0[idx[pos:pos + cnt]])))
        np.testing.assert_allclose(got_t, ref_t, rtol=0, atol=10 * THETA_REL_L2 * rms + 0.5 * upd, err_msg=tname)
        off += n
        pos += cnt
    assert pos == idx.size
