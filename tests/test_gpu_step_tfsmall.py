"""GPU parity of the fp32 server steps of the paper's own transformers
(configs 7 and 8: Transformer-6 and Transformer-12 of Table 4 after their
embedding) against the fp64 oracle, through the C ABI.

fp32 path, graded like the tiny CNN: loss, logits, every parameter's gradient
and the update within 1e-4 (normwise; the logits relative to their largest),
for the full workload batch and for small ragged batches (lengths 1 and L
included), for the re-forward after the update, and for three steps in a
row, each checked from the library's parameters just before it."""
import numpy as np
import pytest

import fo_synth as S
import oracle
from tests.gpu_util import announce, normwise, per_tensor_errors, to_dev, torch_cuda

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2504_13850_amd.api")

TOL = 1e-4


def _step(model, x, lab, ln, B):
    A.fo_server_step(model, (x, ln, B), lab, 0)
    return dict(loss=A.fo_model_read(model, A.FO_BUF_LOSS)[0],
                logits=A.fo_model_read(model, A.FO_BUF_LOGITS).reshape(B, 2),
                grads=A.fo_model_read(model, A.FO_BUF_GRADS),
                params=A.fo_model_read(model, A.FO_BUF_PARAMS).astype(np.float64))


def _check(cid, out, theta, acts, labels, lengths):
    r = oracle.server_step(cid, theta, acts, labels, lengths)
    assert abs(out["loss"] - r["loss"]) <= TOL * abs(r["loss"]), (out["loss"], r["loss"])
    assert normwise(out["logits"], r["logits"]) <= TOL
    errs = per_tensor_errors(cid, out["grads"], r["grads"])
    worst = max(errs, key=errs.get)
    assert errs[worst] <= TOL, (worst, errs[worst])
    assert normwise(out["params"] - theta, r["params"] - theta) <= TOL
    return r


def _batch(cid, B, sub, lengths=None):
    acts = S.make_acts(cid, 1, batch=B, sub=sub)[0]
    labels = S.make_labels(cid, 1, batch=B, sub=sub)[0]
    ln = S.make_lengths(cid, 1, batch=B, sub=sub)[0] if lengths is None else np.asarray(lengths, np.int32)
    return acts, labels, ln


@pytest.mark.parametrize("cid,B,lengths,sub", [
    (7, 16, None, 1), (7, 3, [1, 64, 33], 2), (7, 1, [64], 3),
    (8, 16, None, 1), (8, 2, [1, 256], 2)])
def test_step_parity(cid, B, lengths, sub):
    torch = torch_cuda()
    acts, labels, ln = _batch(cid, B, sub, lengths)
    announce(f"config {cid} step B={B} lengths={ln.tolist()}")
    theta = S.init_params(cid)
    model = A.fo_model_create(cid, B, theta, torch.cuda.current_stream())
    try:
        x, lab, L = to_dev(acts), to_dev(labels), to_dev(ln)
        out = _step(model, x, lab, L, B)
        r = _check(cid, out, theta.astype(np.float64), acts, labels, ln)
        # the second step's forward, from the updated parameters
        A.fo_server_step(model, (x, L, B), lab, 0)
        z2 = A.fo_model_read(model, A.FO_BUF_LOGITS).reshape(B, 2)
        assert normwise(z2, oracle.server_forward(cid, r["params"], acts, ln)) <= TOL
    finally:
        A.fo_model_destroy(model)


@pytest.mark.parametrize("cid", [7, 8])
def test_three_steps_in_a_row(cid):
    torch = torch_cuda()
    B = 4
    announce(f"config {cid} chain of 3, B={B}")
    model = A.fo_model_create(cid, B, S.init_params(cid), torch.cuda.current_stream())
    try:
        prev = S.init_params(cid).astype(np.float64)
        for i in range(3):
            acts, labels, ln = _batch(cid, B, 20 + i)
            out = _step(model, to_dev(acts), to_dev(labels), to_dev(ln), B)
            _check(cid, out, prev, acts, labels, ln)
            prev = out["params"]
    finally:
        A.fo_model_destroy(model)


def test_lengths_outside_the_sequence_are_reported():
    torch = torch_cuda()
    announce("config 7 bad lengths")
    B = 2
    acts, labels, _ = _batch(7, B, 5)
    model = A.fo_model_create(7, B, S.init_params(7), torch.cuda.current_stream())
    try:
        A.fo_server_step(model, (to_dev(acts), to_dev(np.array([0, 65], np.int32)), B), to_dev(labels), 0)
        with pytest.raises(A.FoError) as e:
            A.fo_model_read(model, A.FO_BUF_LOSS)
        assert "2 sequence length(s)" in str(e.value)
    finally:
        A.fo_model_destroy(model)


# The rows are computed in blocks of 16 of one sequence, and (Transformer-12)
# halves of a block against eighths of the other side: lengths around their
# edges, shorter than the eighths, and padded positions that hold NaN (no
# output may read them).  Bound as above; the batches are seeds without a ReLU
# input within 1e-5 of zero, where another order of summation could take
# the other branch.
@pytest.mark.parametrize("cid,lengths,sub", [(7, [1, 15, 16, 17, 48, 49, 64], 33),
                                             (8, [8, 9, 16, 17, 31, 33, 255], 44)])
def test_block_edges(cid, lengths, sub):
    torch = torch_cuda()
    B = len(lengths)
    acts, labels, ln = _batch(cid, B, sub, lengths)
    announce(f"config {cid} block edges lengths={lengths}")
    padded = acts.copy()
    for b in range(B):
        padded[b, lengths[b]:] = np.nan
    theta = S.init_params(cid)
    model = A.fo_model_create(cid, B + 2, theta, torch.cuda.current_stream())
    try:
        out = _step(model, to_dev(padded), to_dev(labels), to_dev(ln), B)
        _check(cid, out, theta.astype(np.float64), acts, labels, ln)
    finally:
        A.fo_model_destroy(model)
