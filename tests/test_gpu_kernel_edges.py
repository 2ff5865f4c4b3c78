"""Kernels at the edges of their tiles, chunks and dispatch rules, against the fp64 oracle."""
import numpy as np
import pytest

from ea_inputs import CONFIGS, make_layer, widen
from oracle import ea_extensions as X
from oracle import ea_oracle as O
from tests import parity as P
import paper_2510_00636_amd as ea

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 127, 129, 2047, 66000])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (256, "f32")])
def test_keydiff_chunk_edges(n, d, dtype):
    """One row, one row around a 128-row chunk, and heads long enough for several chunks of both
    passes.  Tolerance: fp32 sums of n unit vectors, n 2^-24 / sqrt(n) of the anchor's length, and a
    d-term fp32 dot product; below 2e-6 absolute (scores lie in [0, 2])."""
    import torch
    cfg = CONFIGS["c2"].with_(dtype=dtype, head_dim=d, n_q_heads=2, n_kv_heads=2)
    if n > 10000 and d == 256:
        cfg = cfg.with_(n_q_heads=1, n_kv_heads=1)
    lay = make_layer(cfg, n=n, window=min(n, 2))
    p = P.params_for(cfg)
    sc = torch.full((1, cfg.n_kv_heads, n), -1.0, device="cuda")
    ea.score_baseline(p, ea.SCORER_KEYDIFF, P.to_dev(lay["k"]), n, n, 0, sc, P.workspace(p, n, 1))
    torch.cuda.synchronize()
    assert np.abs(sc.cpu().numpy() - X.keydiff_scores(widen(lay["k"]))).max() <= 2e-6
