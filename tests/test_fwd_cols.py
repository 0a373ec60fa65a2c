"""The column-owning forward (lanes own reference columns, segments handed
from wavefront to wavefront): bit for bit against the oracle at the edges of
its segments (64 C columns), workgroups (four segments), step groups (eight
rows) and handover rings (128 rows)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_bit_exact, gpu_forward

pytestmark = pytest.mark.gpu

LENS = [1, 7, 8, 9, 63, 64, 65, 72, 127, 128, 129, 300]


def _cols_variants():
    import paper_2403_06931_amd as P
    return [v for v in range(P.sdtw_variant_count()) if P.sdtw_variant_info(v)[0] == 1]


@pytest.mark.parametrize("ref_len", [1, 1023, 1024, 1025, 2049, 4096, 4097, 8193, 12289])
def test_segment_edges(ref_len):
    import paper_2403_06931_amd as P
    kind = ref_len % 2
    w = workloads.make_random(len(LENS), LENS, max(ref_len, 64), seed=900 + ref_len,
                              excerpt_every=0)
    w.reference = np.ascontiguousarray(w.reference[:ref_len])
    want_c, want_e = oracle.sdtw_f32(w.queries, w.lens, w.reference, kind)
    for v in _cols_variants():
        # the persistent flag's grid sizes change the number of workgroups
        for flags in (0, P.SDTW_F_PERSISTENT | P.SDTW_F_WAVES_PER_SIMD(1)):
            print(f"variant {v} M {ref_len} flags {flags}", flush=True)
            c, e = gpu_forward(w, kind, variant=v, flags=flags)
            assert_bit_exact(c, e, want_c, want_e, f"variant {v} M {ref_len} flags {flags}")


def test_more_items_than_workgroups():
    """More (four segments, query) items than the grid holds, and a batch whose
    offsets come from the table kernel with a single segment."""
    rng = np.random.default_rng(31)
    lens = rng.integers(1, 40, 3000)
    w = workloads.make_random(lens.size, list(lens), 9000, seed=32, excerpt_every=0)
    idx = np.arange(0, lens.size, 97)
    sub = w.subset(idx)
    want_c, want_e = oracle.sdtw_f32(sub.queries, sub.lens, sub.reference, 0)
    for v in _cols_variants():
        c, e = gpu_forward(w, 0, variant=v)
        assert_bit_exact(c[idx], e[idx], want_c, want_e, f"variant {v}, 3,000 queries")
    w = workloads.make_random(16500, 3, 500, seed=33, excerpt_every=0)
    want_c, want_e = oracle.sdtw_f32(w.queries, w.lens, w.reference, 0)
    for v in _cols_variants():
        c, e = gpu_forward(w, 0, variant=v)
        assert_bit_exact(c, e, want_c, want_e, f"variant {v}, 16,500 queries")
