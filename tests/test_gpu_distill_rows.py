"""GPU parity of the adaptation objective at the sizes where its row kernel changes
shape: vocabularies of one chunk and less, around a workgroup size's register capacity
(64 threads x 19 chunks of 8 bf16 logits, x 9 of fp32), past the largest one (the rest
of a row is streamed), padded and unpadded strides, tokens that one side or both rule
out (-inf), and few rows with many threads each.  Bars as in test_gpu_distill.py:
losses 2e-4 + 1e-4 relative, gradients 1e-4 (fp32) or 2^-8 (bf16) relative plus 1e-3 of
the row's largest magnitude."""
import numpy as np
import pytest

from oracle.distill import KIND_NONE, distill_losses
from synth.distill import make_distill_batch
from tests.test_gpu_distill import _check_grad, _check_losses, _run

pytestmark = pytest.mark.gpu


def _check(b, vocab, added, dtype, T, kind=None):
    kind = b.kind if kind is None else kind
    ref = distill_losses(b.student, b.teacher, kind, b.target, b.dec_group, b.turn_group, T)
    for with_grad in (True, False):
        lo, gr, _ = _run(b, vocab, added, dtype, T, with_grad=with_grad, kind=kind)
        _check_losses(lo, ref.losses)
        if with_grad:
            _check_grad(gr[:, :vocab + added], ref.grad, dtype)
            assert not gr[:, vocab + added:].any()


@pytest.mark.parametrize("dtype,T,vocab,added", [
    ("f32", 1.0, 1, 2), ("bf16", 2.0, 6, 2), ("bf16", 1.0, 8, 1), ("f32", 0.5, 63, 1),
    ("f32", 1.0, 64 * 9 * 8 - 2, 2), ("f32", 2.0, 64 * 9 * 8 - 1, 2),
    ("bf16", 1.0, 64 * 19 * 8 - 2, 2), ("bf16", 0.5, 64 * 19 * 8 - 1, 2),
    ("bf16", 1.0, 128 * 19 * 8 + 5, 7), ("f32", 1.0, 512 * 9 * 8 + 3, 2),
])
def test_row_sizes(gpu, dtype, T, vocab, added):
    b = make_distill_batch(seed=21, n_utt=2, units=3, vocab=vocab, added=added, dtype=dtype)
    kind = b.kind.copy()
    kind[2] = KIND_NONE
    _check(b, vocab, added, dtype, T, kind)


@pytest.mark.parametrize("dtype,vocab", [("bf16", 1024 * 19 * 8 + 9), ("f32", 1024 * 9 * 8 + 8191)])
def test_rows_past_the_registers(gpu, dtype, vocab):
    b = make_distill_batch(seed=22, n_utt=1, units=2, vocab=vocab, added=2, dtype=dtype)
    _check(b, vocab, 2, dtype, 1.0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ruled_out_tokens(gpu, dtype):
    """-inf logits: the teacher's alone (no contribution there), and both sides' (no
    contribution, zero gradient), in every chunk of a stretch and at the row's ends."""
    vocab = 1500
    b = make_distill_batch(seed=23, n_utt=2, units=3, vocab=vocab, added=2, dtype=dtype)
    student, teacher = b.student.copy(), b.teacher.copy()
    teacher[:, 100:900] = -np.inf
    teacher[:, -3:] = -np.inf
    student[:, 300:600] = -np.inf
    b = type(b)(student, teacher, b.kind, np.where((b.target >= 300) & (b.target < 600), 7, b.target).astype(np.int32),
                b.dec_group, b.turn_group)
    # the oracle's logs of the tokens without mass drop out of its sums as 0 * -inf: a
    # finite logit far below the others has the same sums
    low = type(b)(np.maximum(student, -1e4), np.maximum(teacher, -1e4), b.kind, b.target, b.dec_group, b.turn_group)
    ref = distill_losses(low.student, low.teacher, b.kind, b.target, b.dec_group, b.turn_group, 1.0)
    lo, gr, _ = _run(b, vocab, 2, dtype, 1.0)
    _check_losses(lo, ref.losses)
    _check_grad(gr[:, :vocab + 2], ref.grad, dtype)


def _rounded(x, dtype):
    import torch
    t = torch.from_numpy(np.asarray(x, np.float32))
    return (t if dtype == "f32" else t.bfloat16().float()).numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [0.5, 1.0, 2.0])
@pytest.mark.parametrize("mask", [-1e10, -1e30, "lowest"])
def test_masked_spans(gpu, dtype, T, mask):
    """Logits masked by a large finite value instead of -inf, in spans that leave some
    threads of a row's workgroup nothing else."""
    import torch
    if mask == "lowest":
        mask = torch.finfo(torch.float32 if dtype == "f32" else torch.bfloat16).min
    vocab, added = 1500, 2
    b = make_distill_batch(seed=24, n_utt=2, units=3, vocab=vocab, added=added, dtype=dtype)
    student, teacher = b.student.copy(), b.teacher.copy()
    for x in (student, teacher):
        x[:, 40:1400] = _rounded(mask, dtype)
    b = type(b)(student, teacher, b.kind, np.where((b.target >= 40) & (b.target < 1400), 7, b.target).astype(np.int32),
                b.dec_group, b.turn_group)
    _check(b, vocab, added, dtype, T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,offset", [(1.0, 3e9), (0.5, -3e9), (2.0, 1e12), (1.0, -1e30), (1e-6, 0.0)])
def test_far_logits(gpu, dtype, T, offset):
    """Rows whose logits all lie far from 0, or far apart at the temperature (also with rows
    past the register capacity): exponents come from differences, not from the logits."""
    for vocab in (1500, 64 * 19 * 8 + 77):
        b = make_distill_batch(seed=25, n_utt=1, units=3, vocab=vocab, added=2, dtype=dtype)
        b = type(b)(_rounded(b.student * 3 + offset, dtype), _rounded(b.teacher * 3 + offset, dtype), b.kind, b.target,
                    b.dec_group, b.turn_group)
        _check(b, vocab, 2, dtype, T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_of_the_lowest_value(gpu, dtype):
    """Transcription rows without a single unmasked logit are uniform."""
    import torch
    low = torch.finfo(torch.float32 if dtype == "f32" else torch.bfloat16).min
    vocab, added = 700, 2
    b = make_distill_batch(seed=26, n_utt=1, units=3, vocab=vocab, added=added, dtype=dtype)
    student = b.student.copy()
    student[b.target >= 0] = low
    _check(type(b)(student, b.teacher, b.kind, b.target, b.dec_group, b.turn_group), vocab, added, dtype, 1.0)


@pytest.mark.parametrize("dtype,logits,batch", [
    ("bf16", 2 * 64 * 8, (2, 3)), ("f32", 2 * 64 * 8 - 1, (2, 3)),             # one workgroup size and the next
    ("bf16", 4 * 256 * 8, (2, 3)), ("bf16", 4 * 256 * 8 + 1, (2, 3)),          # 4 rounds and 5, 256 threads
    ("f32", 4 * 256 * 8, (2, 3)), ("f32", 4 * 256 * 8 + 1, (2, 3)),
    ("bf16", 8 * 256 * 8 - 8, (2, 3)), ("bf16", 8 * 256 * 8 - 7, (2, 3)),      # 8 rounds of 256 threads, 4 of 512
    ("bf16", 8 * 1024 * 8, (1, 2)), ("bf16", 8 * 1024 * 8 + 1, (1, 2)),        # 8 rounds and 9, 1,024 threads
    ("bf16", 1500, (16, 12)), ("f32", 3500, (12, 12)),                         # many rows, few threads each
])
def test_rounds_of_a_row(gpu, dtype, logits, batch):
    """Row lengths around those at which a row's kernel holds more chunks a thread, and short
    rows in batches large and small."""
    b = make_distill_batch(seed=27, n_utt=batch[0], units=batch[1], vocab=logits - 2, added=2, dtype=dtype)
    _check(b, logits - 2, 2, dtype, 2.0)
