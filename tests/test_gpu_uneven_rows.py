"""Passes of 5 to 16 sequences whose hidden width leaves the 16-column
workgroups of the FCs uneven over the compute units (4128 columns: 258
workgroups): their GEMMs run as K slices with a finish launch, K ragged in
64-wide chunks (16 sequences), or stay whole where the workspace, made for at
most 16 rows of the two layers, holds no slices (5 sequences)."""
import numpy as np
import pytest

from fe_synth import configs as C
from tests.gpu_case import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [5, 16])
def test_uneven_width_matches_oracle(batch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = C.SMALL_MHA_BF16_D128.with_(name="uneven", hidden=4128, n_q_heads=4, n_kv_heads=4,
                                      intermediate=3552, n_layers=2, draft_vocab=1040,
                                      target_vocab=1040, batch=batch, topk=4)
    lens = np.arange(batch, dtype=np.int32) * 13 % 70
    run_case(cfg, seed=2, prefix_lens=lens)
