"""Product sumchecks at the sizes where the round kernels change over, byte for byte against the oracle's C tier:
one block per evaluation in the last rounds (512, 256, 128, 64 and fewer pairs), few and many partial sums per round
(one, up to 64, more than 512)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 5, 8, 10, 11, 12, 13, 14, 17, 19, 20])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_product_rounds(lib, ctx, k, d):
    from oracle import c_oracle
    from workloads import uniform_fr_limbs
    rng = np.random.default_rng(100 * k + d)
    raws = [uniform_fr_limbs(rng, 1 << d).tobytes() for _ in range(k)]
    if d == 12:     # the largest element everywhere: sums of lazy values at the top of their range
        from oracle.field import R_MOD
        raws = [int(R_MOD - 1).to_bytes(32, "little") * (1 << d) for _ in range(k)]
    tabs = [lib.fr_tensor_upload(ctx, r, (1 << d,)) for r in raws]
    tr = lib.Transcript(7)
    got = lib.sumcheck_product(ctx, tabs, tr)
    proof, chal, digest = c_oracle.product_prove(raws, 7)
    assert got["proof"] == proof and got["points"] == chal and tr.digest() == digest
