"""Prefill chunk size (GPU property, no oracle): the prompts are processed in
chunks of max_rows rows, and every kernel's arithmetic for a row depends only
on that row's own data and keys (K reductions split by (N, K), attention
splits at fixed absolute positions), so prefilling with 128-, 384-, 512- and
1024-row chunks must leave bit-identical state: the same first tokens, and
the following rounds' drafter logits, verify logits, acceptance and
committed tokens equal bit for bit.  Prompts of 700 and 300 tokens make the
chunks ragged (700 = 5 x 128 + 60 = 384 + 316 = 512 + 188)."""
import numpy as np
import pytest

from workload import get_config
from workload.synth import make_weights

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROUNDS = 2


def _run(max_rows, dims, B, prompts, w, V):
    from paper_2609_06498_amd import Runtime
    from paper_2609_06498_amd.session import Session
    b = len(prompts)
    rt = Runtime(dims, B, b, max(len(p) for p in prompts) + (ROUNDS + 2) * B, w, "suffix", max_rows=max_rows)
    sess = Session(rt, b)
    sess.prefill(prompts)
    out = [sess.anchor.cpu().numpy().copy()]
    for _ in range(ROUNDS):
        lg = torch.zeros(b * B, V, dtype=torch.float32, device="cuda")
        dl = torch.zeros(b * B, V, dtype=torch.float32, device="cuda")
        sess.round(True, draft_logits=dl, logits=lg)
        torch.cuda.synchronize()
        out += [dl.cpu().numpy(), lg.cpu().numpy(), sess.accept.cpu().numpy().copy(),
                sess.committed.cpu().numpy().copy(), sess.seq_len.cpu().numpy().copy()]
    assert rt.status() == 0
    return out


def test_prefill_chunk_size_invariance():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = get_config("small-bf16-b24")
    dims, B, V = wl.dims, wl.block, wl.dims.vocab
    r = np.random.default_rng(0x5EED_0C4)
    prompts = [r.integers(0, V, size=n).astype(np.int32) for n in (700, 300)]
    w = make_weights(dims, wl.seed_w)
    ref = None
    for mr in (128, 384, 512, 1024):
        print(f"[prefill-chunks] max_rows={mr}", flush=True)
        out = _run(mr, dims, B, prompts, w, V)
        if ref is None:
            ref = out
            continue
        for i, (a, b) in enumerate(zip(ref, out)):
            assert np.array_equal(a, b), f"max_rows {mr}: output {i} differs from the 128-row chunks"


@pytest.mark.parametrize("seq", [-2**31, -1, 2, 2**31 - 1])
def test_prefill_refuses_slots_outside_the_batch(seq):
    """Nothing is launched for a slot that the context does not have, the largest int among them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import DFlowError, Runtime
    wl = get_config("tiny-f32")
    rt = Runtime(wl.dims, wl.block, 2, 64, make_weights(wl.dims, wl.seed_w))
    tok = torch.zeros(4, dtype=torch.int32, device="cuda")
    first = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    smp = rt.sampler(1.0, 5, torch.zeros(1, dtype=torch.int64, device="cuda"))
    with pytest.raises(DFlowError, match="seq"):
        rt.prefill(seq, tok, first)
    with pytest.raises(DFlowError, match="seq"):
        rt.prefill_sampled(seq, tok, smp, first)
    assert int(first) == -7 and rt.status() == 0
    assert not bool((rt.k_pool != 0).any())
    rt.close()
