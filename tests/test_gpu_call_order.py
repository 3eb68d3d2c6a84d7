"""A prompt processed in a spare slot between two calls of a round leaves the
round's sequences alone (GPU property, no oracle).  The captured states of
verify_block are read by accept and the projected features of accept by
kv_commit, so a prefill of another slot after verify, after accept or after both
must give, bit for bit, what it gives between rounds: the same drafter context
and target caches, drafts, acceptance, bonus tokens and feature rows, and the
same caches and first token of the spare slot's own prompt."""
import numpy as np
import pytest

from tests.gpu_common import gpu_trajectory
from workload import get_config
from workload.synth import make_prompts, make_schedule, make_weights, trajectory_length_needed

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROUNDS = 3


def _run(rt, prompts, extra, after, force, sampled):
    """ROUNDS rounds with one prefill of the spare slot per round after the named calls; everything observable."""
    from paper_2609_06498_amd.session import Session
    b, B, dm = len(prompts), rt.block, rt.dims
    for t in (rt.k_pool, rt.v_pool, rt.ck_pool, rt.cv_pool):
        t.zero_()
    s = Session(rt, b)
    s.prefill(prompts)
    first = torch.zeros(1, dtype=torch.int32, device="cuda")
    feat = torch.zeros(b * B, dm.d, dtype=rt.elt_torch, device="cuda")
    stream = torch.arange(b, dtype=torch.int64, device="cuda")
    smp = rt.sampler(1.0, 5, stream)
    out = []
    for r in range(ROUNDS):
        def maybe(call):
            if call in after:
                rt.prefill(b, extra[r], first)
        maybe("commit")
        if sampled:
            dl, lg = s.logit_buffers()
            rt.draft_block(b, s.anchor, s.seq_len, True, None, None, dl)
            rt.sample_draft(b, dl, s.anchor, s.seq_len, smp, s.draft_tok, s.block)
            rt.verify_block(b, s.block, s.seq_len, None, lg)
            maybe("verify")
            rt.accept_sampled(b, s.block, s.seq_len, lg, dl, smp, s.accept, s.anchor, s.committed, s.n_carry, feat)
        else:
            traj, mode, tok = force
            rt.draft_block(b, s.anchor, s.seq_len, True, s.draft_tok, s.block)
            rt.force_drafts(b, traj, traj.shape[1], mode[r], tok[r], s.anchor, s.seq_len, s.block)
            rt.verify_block(b, s.block, s.seq_len, s.tgt)
            maybe("verify")
            rt.accept_and_carry(b, s.block, s.tgt, s.accept, s.anchor, s.committed, s.n_carry, feat)
        maybe("accept")
        rt.kv_commit(b, s.accept, s.seq_len)
        out += [x.clone() for x in (s.draft_tok, s.block, s.accept, s.anchor, s.committed, s.n_carry, s.seq_len,
                                    feat, first)]
    assert rt.status() == 0
    return out + [x.clone() for x in (rt.k_pool, rt.v_pool, rt.ck_pool, rt.cv_pool)]


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("name", ["tiny-f32", "small-bf16"])
def test_prefill_between_calls_of_a_round(name, sampled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    from paper_2609_06498_amd.session import Session
    wl = get_config(name)
    dm, B, b = wl.dims, wl.block, wl.batch
    prompts = make_prompts(wl)
    sched = make_schedule(wl, ROUNDS)
    need = trajectory_length_needed(wl, sched)
    # a slot more than the round's sequences; chunks of 64 rows, prompts longer and shorter than one
    rt = Runtime(dm, B, b + 1, max(need) + 2 * B, make_weights(dm, wl.seed_w), wl.carry_window, max_rows=64)
    traj = torch.from_numpy(gpu_trajectory(rt, Session(rt, b), prompts, need)).cuda()
    force = (traj, torch.from_numpy(sched["mode"]).cuda(), torch.from_numpy(sched["tok"]).cuda())
    rng = np.random.default_rng(3)
    extra = [torch.from_numpy(rng.integers(0, dm.vocab, size=n).astype(np.int32)).cuda() for n in (90, 64, 33)]
    ref = _run(rt, prompts, extra, ("commit",), force, sampled)
    n = (len(ref) - 4) // ROUNDS
    # first tokens are written at the same prefill, whichever call it follows
    for after in (("verify",), ("accept",), ("verify", "accept")):
        print(f"[order] {name} sampled={sampled} prefill after {after}", flush=True)
        got = _run(rt, prompts, extra, after, force, sampled)
        for i, (x, y) in enumerate(zip(ref, got)):
            what = ("k_pool", "v_pool", "ck_pool", "cv_pool")[i - ROUNDS * n] if i >= ROUNDS * n else \
                f"round {i // n} " + ("draft_tok", "block", "accept", "bonus", "committed", "n_carry", "seq_len",
                                      "features", "first token")[i % n]
            assert torch.equal(x, y), f"{name}: {what} differs with a prefill after {after}"
    rt.close()
