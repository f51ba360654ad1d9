"""GPU parity of the fp32 server step of the paper's VGG-5 (config 9: Table 4's
VGG-5 after its second pool) against the fp64 oracle, through the C ABI.

fp32 path, graded like the tiny CNN: loss, logits, every parameter's gradient
and the update within 1e-4 (normwise), for the workload batch and small
batches, for the re-forward after the update, and for three steps in a row,
each checked from the library's parameters just before it.  Batch-norm
statistics, the pool's argmax routing and the ReLU masks are all inside the
step, so a single wrong index shows up in the convolution's gradient."""
import numpy as np
import pytest

import fo_synth as S
import oracle
from tests.gpu_util import announce, normwise, per_tensor_errors, to_dev, torch_cuda

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2504_13850_amd.api")

CID = 9
TOL = 1e-4


def _step(model, x, lab, B):
    A.fo_server_step(model, (x, None, B), lab, 0)
    return dict(loss=A.fo_model_read(model, A.FO_BUF_LOSS)[0],
                logits=A.fo_model_read(model, A.FO_BUF_LOGITS).reshape(B, 10),
                grads=A.fo_model_read(model, A.FO_BUF_GRADS),
                params=A.fo_model_read(model, A.FO_BUF_PARAMS).astype(np.float64))


def _check(out, theta, acts, labels):
    r = oracle.server_step(CID, theta, acts, labels)
    assert abs(out["loss"] - r["loss"]) <= TOL * abs(r["loss"]), (out["loss"], r["loss"])
    assert normwise(out["logits"], r["logits"]) <= TOL
    errs = per_tensor_errors(CID, out["grads"], r["grads"])
    worst = max(errs, key=errs.get)
    assert errs[worst] <= TOL, (worst, errs[worst])
    assert normwise(out["params"] - theta, r["params"] - theta) <= TOL
    return r


@pytest.mark.parametrize("B,sub", [(32, 1), (5, 2), (2, 3)])
def test_step_parity(B, sub):
    torch = torch_cuda()
    announce(f"config 9 step B={B}")
    theta = S.init_params(CID)
    acts = S.make_acts(CID, 1, batch=B, sub=sub)[0]
    labels = S.make_labels(CID, 1, batch=B, sub=sub)[0]
    model = A.fo_model_create(CID, B, theta, torch.cuda.current_stream())
    try:
        x, lab = to_dev(acts), to_dev(labels)
        out = _step(model, x, lab, B)
        r = _check(out, theta.astype(np.float64), acts, labels)
        A.fo_server_step(model, (x, None, B), lab, 0)
        z2 = A.fo_model_read(model, A.FO_BUF_LOGITS).reshape(B, 10)
        assert normwise(z2, oracle.server_forward(CID, r["params"], acts)) <= TOL
    finally:
        A.fo_model_destroy(model)


def test_three_steps_in_a_row():
    torch = torch_cuda()
    B = 32
    announce("config 9 chain of 3")
    model = A.fo_model_create(CID, B, S.init_params(CID), torch.cuda.current_stream())
    try:
        prev = S.init_params(CID).astype(np.float64)
        for i in range(3):
            acts = S.make_acts(CID, 1, batch=B, sub=30 + i)[0]
            labels = S.make_labels(CID, 1, batch=B, sub=30 + i)[0]
            out = _step(model, to_dev(acts), to_dev(labels), B)
            _check(out, prev, acts, labels)
            prev = out["params"]
    finally:
        A.fo_model_destroy(model)


# Batches around the edges of the fused step (one sample, 16 and 17 padded
# samples, more samples than shares of the weight gradient, its largest batch)
# and one beyond it.  Bounds as above; seeds in which no ReLU input or pool
# margin is within 9e-6 of the other branch.
@pytest.mark.parametrize("B,sub", [(1, 60), (16, 60), (17, 61), (33, 61), (128, 63), (130, 63)])
def test_batch_edges(B, sub):
    torch = torch_cuda()
    announce(f"config 9 step B={B}")
    theta = S.init_params(CID)
    acts = S.make_acts(CID, 1, batch=B, sub=sub)[0]
    labels = S.make_labels(CID, 1, batch=B, sub=sub)[0]
    model = A.fo_model_create(CID, max(B, 40), theta, torch.cuda.current_stream())
    try:
        _check(_step(model, to_dev(acts), to_dev(labels), B), theta.astype(np.float64), acts, labels)
    finally:
        A.fo_model_destroy(model)
