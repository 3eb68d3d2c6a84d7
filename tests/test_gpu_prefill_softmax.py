"""Prompt attention keeps the largest probability of a key page exact: the bf16
probabilities are relative to the page's own largest score, not to that of the
pages before it (GPU property against a 64-bit softmax).

Every weight is a power of two or zero, so that the attention output of the
first layer's one head can be read bit for bit from the second layer's value
cache.  Key A (page 0, value 0) scores highest, key B (page 1, value 1) up to six
powers of two lower, every other key (value 0) next to nothing, so the output is
p_B / (p_A + p_B + rest) in bf16.  With p_B exact that is the 64-bit value rounded
once: only ties within the fp32 arithmetic's few 1e-7 of a rounding boundary (the
boundaries lie 2^-9 to 2^-8 apart: about one row in a thousand) may go the other
way; 2 % are allowed.  With p_B rounded to bf16 beside an exact p_A, a quarter of
the rows comes out one unit off."""
import numpy as np
import pytest

from workload.configs import ModelDims
from workload.synth import make_weights

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

D, DH, V = 256, 64, 272
C = DH // 2 - 1          # the head channel that counts: the slowest rotation pair (angle 0 at this theta)
A, F, B, Q0 = 0, 1, 2, 3   # token ids: the two keys, the filler, the first query


def _bits(x):
    """fp32 / fp64 -> bf16 bit patterns, rounded to nearest even."""
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + (u >> 16 & 1)) >> 16).astype(np.uint16)


def _val(b):
    return (b.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("max_rows", [64, 512])
def test_top_probability_of_a_page_is_exact(max_rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    dims = ModelDims("bf16", D, 2, 1, 1, DH, 64, V, 1, (0, 1), rope_theta=1e30)
    rng = np.random.default_rng(5)
    # embedding: 0 carries the row's norm (2^10, so its scale is 2^-6), 1 / 2 the query's two raw channels,
    # 3 / 4 the key's, 5 the value; 6 stays 0 and takes the attention output
    emb = np.zeros((V, D))
    emb[:, 0] = 1024.0
    emb[:, 3] = -1.0
    emb[A, 3] = 1.0
    emb[B, 3:6] = 1.0, 1.734375, 1.0
    emb[Q0:, 1] = 1.0
    emb[Q0:, 2] = _val(_bits(rng.uniform(0.0, 3.0, V - Q0)))
    w = make_weights(dims, 11)
    w["embed"] = _bits(emb)

    def unit(rows, cols, *at):     # 64 undoes the row scale
        m = np.zeros((rows, cols), np.float32)
        for r, c, x in at:
            m[r, c] = x
        return _bits(m)
    gain = unit(1, DH, (0, C, 1.0))[0]
    for l in range(2):
        p = f"layers.{l}."
        w[p + "attn_norm"] = w[p + "ffn_norm"] = _bits(np.ones(D))
        w[p + "q_norm"] = w[p + "k_norm"] = gain
        w[p + "wq"] = unit(DH, D, (C, 1, 64.0), (0, 2, 64.0))
        w[p + "wk"] = unit(DH, D, (C, 3, 64.0), (0, 4, 64.0))
        w[p + "wv"] = unit(DH, D, (0, 5 + l, 64.0))
        w[p + "wo"] = unit(D, DH, (6, 0, 1.0 - l))
        w[p + "w_down"] = _bits(np.zeros((D, 64)))
    n = 2500                       # past the first boundary of the attention splits
    tok = rng.integers(Q0, V, size=n).astype(np.int32)
    tok[:128] = F
    tok[0], tok[64] = A, B
    rt = Runtime(dims, 2, 1, n + 2, w, max_rows=max_rows)
    first = torch.zeros(1, dtype=torch.int32, device="cuda")
    rt.prefill(0, torch.from_numpy(tok).cuda(), first)
    assert rt.status() == 0
    s, pages = np.arange(n) % 64, np.arange(n) // 64
    off = (s // 32 * (DH // 16) * 64 + s % 16 // 4 * 16) * 8 + s % 32 // 16 * 4 + s % 4   # value channel 0
    pool = rt.v_pool.cpu().numpy().view(np.uint16).reshape(2, rt.num_pages, 64 * DH)
    got = pool[1, pages, off]
    assert np.array_equal(_val(pool[0, pages, off]), emb[tok, 5])
    rt.close()
    # 64-bit softmax of the bf16 queries and keys
    norm = lambda x, y: _val(_bits(x / np.sqrt((x * x + y * y) / DH + dims.rms_eps)))
    q = norm(emb[tok, 1], emb[tok, 2])
    kA, kB, kF = norm(np.array([1.0, 1.0, -1.0]), np.array([0.0, 1.734375, 0.0]))
    rows = np.arange(128, n)
    sc = q[rows] / np.sqrt(DH)
    pA, pB, pF = np.exp(sc * kA), np.exp(sc * kB), np.exp(sc * kF)
    want = _bits(pB / (pA + pB + (rows - 1) * pF))
    off_by = np.abs(got[rows].astype(int) - want.astype(int))
    print(f"[softmax] {np.count_nonzero(off_by)} of {len(rows)} rows differ, by {off_by.max()} units at most", flush=True)
    assert off_by.max() <= 1
    assert np.count_nonzero(off_by) <= 0.02 * len(rows)
