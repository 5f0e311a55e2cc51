"""GPU parity of the float32 MFMA attention kernel at the edges of its tiles, and against the vector-ALU kernel
(path option 2) where values are not finite."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import _gpu as G

pytestmark = pytest.mark.gpu
OPT_SPLITS, OPT_PATH = 0, 1


def _case(heads, n, lens, mode="step", page=16, extra=0, seed=71):
    kw = dict(step_offsets=[extra] * len(lens), max_draft=n + extra) if mode == "step" else {}
    return W.make_case(mode=mode, batch=len(lens), ctx_lens=list(lens), n_new=n, dtype="fp32", page_size=page,
                       num_q_heads=heads[0], num_kv_heads=heads[1], seed=seed, **kw)


# rows = G * n: one 16-row tile, two, and several groups of two with a ragged last tile; prefixes around
# the 16-key block, one round of the 8 waves (128 keys) and past it; draft keys 1 to 64
@pytest.mark.parametrize("heads,n,extra,mode", [((8, 8), 1, 0, "step"), ((32, 8), 4, 0, "step"), ((32, 8), 4, 3, "step"),
                                               ((16, 2), 2, 13, "step"), ((32, 8), 5, 1, "step"), ((8, 1), 4, 0, "step"),
                                               ((6, 2), 17, 0, "step"), ((32, 8), 64, 0, "step"), ((32, 8), 17, 0, "tree"),
                                               ((16, 8), 64, 0, "tree"), ((32, 8), 60, 0, "tree")])
@pytest.mark.parametrize("lens", [(0, 1, 15), (16, 17, 127, 128, 129), (700, 33)])
@pytest.mark.parametrize("splits", [0, 3])
def test_fp32_tiles(heads, n, extra, mode, lens, splits):
    c = _case(heads, n, lens, mode=mode, extra=extra, page=64 if splits else 16)
    dc = G.DevCase(c)
    with G.handle_for(c) as att:
        att.set_option(OPT_SPLITS, splits)
        gpu, lse = G.run(att, dc, want_lse=True)
    ref, ref_lse = oracle.draft_attention(c)
    G.assert_parity(gpu, ref, "fp32", f"{heads} n={n} lens={lens}")
    assert np.abs(lse - ref_lse).max() <= 1e-4, np.abs(lse - ref_lse).max()


@pytest.mark.parametrize("n", [4, 8])
def test_fp32_same_as_vector_kernel_where_values_are_not_finite(n):
    """A key of weight zero contributes nothing even if its value is inf or NaN; one with weight makes the row
    non-finite in the same channels.  Query rows see a draft key's value only if it is not after them."""
    c = _case((32, 8), n, (40, 300), seed=72)
    c.draft_v[0, n - 1, 2, 5] = np.inf       # seen by the last query row only
    c.draft_v[1, n - 2, 3, 100] = np.nan     # seen by the last two
    dc = G.DevCase(c)
    with G.handle_for(c) as att:
        got = G.run(att, dc)
        att.set_option(OPT_PATH, 2)
        ref = G.run(att, dc)
    assert not np.isfinite(ref).all()
    np.testing.assert_array_equal(np.isfinite(got), np.isfinite(ref))
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= G.FP32_MAX_ABS


def test_fp32_automatic_plans_fit_the_no_allocation_scratch():
    """Whatever the batch, query count and prefix: split partials of an automatic plan take less than 32 MiB."""
    c = _case((32, 8), 64, (16,))
    G.torch().zeros(1, device="cuda")
    with G.handle_for(c, max_batch=64, max_pages_per_seq=2048) as att:
        for b in (1, 2, 5, 16, 31, 33, 64):
            for n in (1, 4, 5, 8, 9, 33, 64):
                for ctx in (0, 16, 100, 255, 256, 1000, 8192, 32768):
                    pl = att.plan(b, n, ctx)
                    rows_pad = 32 * pl["row_tiles"]
                    assert pl["splits"] == 1 or b * 8 * rows_pad * pl["splits"] * (128 * 4 + 8) + 512 <= 32 << 20, (b, n, ctx)
