"""Binary16 forward: input values that round to an infinity, in queries,
references and both, on every variant.  A query holding one costs +inf with
end position 0 (every path passes its row; the oracle's own minimum is not
defined there, where the reference holds an infinity too: inf - inf is NaN);
one in the reference only makes its column impassable, and the other queries
agree with the oracle bit for bit.  A NaN acts as an infinity."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_bit_exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("ref_len", [60, 1500])
def test_infinite_values(kind, ref_len):
    import paper_2403_06931_amd as P
    rng = np.random.default_rng(77 + kind)
    lens = np.array([5, 5, 70, 70, 3, 3, 9], np.int32)
    q = rng.standard_normal(int(lens.sum())).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(lens)])
    q[off[0] + 2] = 1e5                    # first of a pair
    q[off[3] + 69] = -65520.0              # second of a pair, its last row: the tie rounds away
    q[off[4]] = 65519.996                  # largest value that stays finite
    q[off[6] + 8] = 7e4                    # last query of an odd batch
    r = rng.standard_normal(ref_len).astype(np.float32)
    r[[0, 7, ref_len - 1]] = 1e5, -1e5, 65520.0
    want_c, want_e = oracle.sdtw_f16(q, lens, r, kind)
    r[7] = np.nan                          # as impassable as the infinity it replaces
    assert np.isfinite(want_c[[1, 2, 5]]).all()
    want_c[[0, 3, 6]] = np.inf
    want_e[[0, 3, 6]] = 0
    dev = torch.device("cuda:0")
    qd, ld, rd = (torch.from_numpy(x).to(dev) for x in (q, lens, r))
    for v in range(P.sdtw_variant_count()):
        print(f"variant {v} kind {kind} M {ref_len}", flush=True)
        c, e = P.sdtw_forward_f16(qd, lens, ld, rd, kind, variant=v)
        torch.cuda.synchronize()
        assert_bit_exact(c.cpu().numpy(), e.cpu().numpy(), want_c, want_e, f"variant {v}")
