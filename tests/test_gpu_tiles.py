"""The tiled GEMM against the weight-streaming one, and prompt attention at every
tile (GPU property, no oracle): a prompt processed in chunks of at most 48 rows
takes the weight-streaming kernels, larger chunks the tiles, their K parts and
the reduce kernels, and every row's arithmetic is the same in both, so the
target KV and the drafter context must agree bit for bit.  The longer prompt
crosses the first boundary of the attention splits (2048 keys), so its rows are
written directly, or merged from one or two partials, depending on the chunk.
  The chunk sizes sit at the edges of the tiles
(64 and 128 rows), of the split rules (49, 256/257, 512/513 rows) and off the
16-row tiles; the widths give odd strip and k-tile counts, K ranges of unequal
length and reductions shorter than the load ring.  A prompt's LM head has one row
and never reaches a tile, and no prompt runs the relay: rounds of many sequences
do, compared with the same sequences a few at a time."""
import numpy as np
import pytest

from workload import get_config
from workload.configs import ModelDims
from workload.synth import make_weights

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DIMS = {
    "bf16": get_config("small-bf16").dims,
    "f32": get_config("small-f32").dims,
    # 3, 4 and 5 k tiles per projection
    "bf16-narrow": ModelDims("bf16", 96, 2, 2, 1, 64, 160, 272, 1, (0, 1)),
    "f32-narrow": ModelDims("f32", 48, 2, 2, 1, 64, 112, 272, 1, (0, 1)),
    # gate/up of 257 column tiles: 256-row tiles at 1000 and 1024 rows
    "bf16-wide": ModelDims("bf16", 256, 2, 4, 2, 64, 16416, 272, 1, (0, 1)),
}
ROWS = (48, 49, 64, 65, 127, 129, 200, 256, 257, 384, 512, 513, 1024)


@pytest.mark.parametrize("name", sorted(DIMS))
def test_chunk_rows_bitwise(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    dims = DIMS[name]
    r = np.random.default_rng(7)
    prompts = [r.integers(0, dims.vocab, size=n).astype(np.int32) for n in (2300, 310)]
    tok = torch.from_numpy(np.concatenate(prompts)).cuda()
    w = make_weights(dims, 11)
    ref = None
    for rows in (48, 512, 1000, 1024) if name == "bf16-wide" else ROWS:
        print(f"[tiles] {name} rows={rows}", flush=True)
        rt = Runtime(dims, 16, 2, 2400, w, max_rows=rows)
        first = torch.zeros(2, dtype=torch.int32, device="cuda")
        rt.prefill_batch(tok, [len(p) for p in prompts], first)
        assert rt.status() == 0
        got = [x.clone() for x in (rt.k_pool, rt.v_pool, rt.ck_pool, rt.cv_pool, first)]
        rt.close()
        if ref is None:
            ref = got
            assert any(bool((x != 0).any()) for x in ref)
            continue
        for i, (a, b) in enumerate(zip(ref, got)):
            assert torch.equal(a, b), f"{name}: output {i} with {rows}-row chunks differs from 48-row chunks"


@pytest.mark.parametrize("rows", [32, 64, 200, 1024])
def test_prompts_sharing_chunks_bitwise(rows):
    """Prompts of a batch share chunks: the caches and first tokens are those of
    the same prompts taken one at a time (one-row prompts, prompts that end at
    a chunk's edge and prompts cut by it)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    dims = DIMS["bf16"]
    r = np.random.default_rng(9)
    lens = [1, 63, 130, 6, 1, 300, 11]
    prompts = [r.integers(0, dims.vocab, size=n).astype(np.int32) for n in lens]
    w = make_weights(dims, 11)
    got = []
    for batch in (False, True):
        rt = Runtime(dims, 16, len(lens), 400, w, max_rows=rows)
        first = torch.zeros(len(lens), dtype=torch.int32, device="cuda")
        if batch:
            rt.prefill_batch(torch.from_numpy(np.concatenate(prompts)).cuda(), lens, first)
        else:
            for s, p in enumerate(prompts):
                rt.prefill(s, torch.from_numpy(p).cuda(), first[s:s + 1])
        assert rt.status() == 0
        got.append([x.clone() for x in (rt.k_pool, rt.v_pool, rt.ck_pool, rt.cv_pool, first)])
        rt.close()
    assert bool((got[0][0] != 0).any())
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), f"output {i} differs"


@pytest.mark.parametrize("b", [25, 50])
def test_round_rows_bitwise(b):
    """Rounds of 250 and 500 rows (the last 16-row and 256-row tiles not full)
    against the same sequences four at a time (40 rows, the weight-streaming
    kernels).  The LM heads take the 256 x 128 tile (3073 strips: 385 strip
    tiles, the last of a single strip).  The second round runs the relay, whose two projections take the
    tiles' bias epilogues."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    from paper_2609_06498_amd.session import Session
    dims = ModelDims("bf16", 96, 2, 2, 1, 64, 160, 49168, 1, (0, 1))
    B, rounds = 10, 2
    r = np.random.default_rng(13)
    prompts = [r.integers(0, dims.vocab, size=n).astype(np.int32) for n in r.integers(3, 40, size=b)]
    rt = Runtime(dims, B, b, 64 + rounds * B, make_weights(dims, 11))

    def run(seqs):
        s = Session(rt, len(seqs))
        s.prefill([prompts[i] for i in seqs])
        out = []
        for _ in range(rounds):
            lg = torch.zeros(len(seqs) * B, dims.vocab, dtype=torch.float32, device="cuda")
            dl = torch.zeros_like(lg)
            s.round(True, draft_logits=dl, logits=lg)
            out.append([dl.view(len(seqs), B, -1), lg.view(len(seqs), B, -1)] +
                       [x.clone() for x in (s.block, s.tgt, s.committed, s.accept, s.n_carry, s.seq_len)])
        assert rt.status() == 0
        return out

    print(f"[tiles] round of {b * B} rows", flush=True)
    many = run(list(range(b)))
    assert int(many[0][6].max()) > 0        # something is carried, so the second round relays rows
    for lo in range(0, b, 4):
        seqs = list(range(lo, min(lo + 4, b)))
        for k, (x, y) in enumerate(zip(run(seqs), many)):
            for i, (p, q) in enumerate(zip(x, y)):
                assert torch.equal(p, q[lo:lo + len(seqs)]), f"sequences {seqs}, round {k}: output {i} differs"
    # the argmax of the logits themselves
    assert torch.equal(many[1][1].argmax(-1).int(), many[1][3])
    rt.close()


def test_logits_at_any_float():
    """The logits buffers are the caller's: one that starts between two 16-byte
    boundaries takes the same values (64 rows, the tiles' vector stores)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    from paper_2609_06498_amd.session import Session
    dims, B, b = DIMS["bf16-narrow"], 16, 4
    r = np.random.default_rng(17)
    prompts = [r.integers(0, dims.vocab, size=n).astype(np.int32) for n in (5, 30, 17, 9)]
    rt = Runtime(dims, B, b, 64, make_weights(dims, 11))
    got = []
    for off in (0, 1):
        s = Session(rt, b)
        s.prefill(prompts)
        n = b * B * dims.vocab
        lg, dl = (torch.full((n + 8,), -7.0, dtype=torch.float32, device="cuda") for _ in range(2))
        s.round(True, draft_logits=dl[off:off + n], logits=lg[off:off + n])
        assert rt.status() == 0
        for x in (dl, lg):      # nothing outside
            assert bool((x[:off] == -7).all()) and bool((x[off + n:] == -7).all())
        got.append([dl[off:off + n].clone(), lg[off:off + n].clone(), s.tgt.clone(), s.block.clone()])
    rt.close()
    for i, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), f"output {i} differs"
