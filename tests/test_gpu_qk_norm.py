"""QK-norm's sum of squares is a binary tree over the rotation pairs of a head
(GPU property, no oracle): permuting the pairs of a row by any xor permutes its
normalised values and changes no bit of them.  Two key heads read the same
inputs, one of them permuted, through unit-vector projections (exact), at
position 0, where RoPE is the identity; fp32, where one unit in the last place
of the sum reaches the cached keys."""
import numpy as np
import pytest

from workload.configs import ModelDims
from workload.synth import make_weights

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [64, 128])
def test_pair_permutations_bitwise(dh):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_06498_amd import Runtime
    d, n, half = 2 * dh, 32, dh // 2
    dims = ModelDims("f32", d, 1, 2, 2, dh, 64, 272, 1, (0,))
    w = make_weights(dims, 11)
    w["layers.0.attn_norm"] = np.ones(d, np.float32)
    w["layers.0.k_norm"] = np.ones(dh, np.float32)
    e = np.arange(dh)
    off = e // 16 * 256 + e % 16 // 4 * 64 + e % 4      # element e of slot 0 in a fp32 key block
    tok = torch.arange(n, dtype=torch.int32, device="cuda")
    first = torch.zeros(n, dtype=torch.int32, device="cuda")
    for k in (1, 2, 3, 4, half // 2, half - 1):
        perm = (e % half ^ k) + e // half * half
        w["layers.0.wk"] = np.concatenate([np.eye(dh, d), np.eye(dh, d)[perm]]).astype(np.float32)
        rt = Runtime(dims, 2, n, 8, w)
        rt.prefill_batch(tok, [1] * n, first)
        assert rt.status() == 0
        keys = rt.k_pool.cpu().numpy().reshape(n, 2, 64 * dh)[:, :, off]   # one page a sequence
        rt.close()
        a, b = keys[:, 0][:, perm], keys[:, 1]
        assert np.all(a != 0)
        assert np.array_equal(a, b), f"xor {k}: {np.count_nonzero((a != b).any(axis=1))} of {n} rows differ"
