"""The autotuner chooses between different launches only: a configuration that launches the same kernels on
the same grids as the default is never preferred to it by the noise of a timing."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 10, 17, 30, 50])
@pytest.mark.parametrize("lo,hi", [(4, 16), (17, 32), (33, 48), (49, 64)])
def test_no_choice_by_noise(lib, n, lo, hi, monkeypatch):
    import torch
    monkeypatch.delenv("RWPSF_AUTOTUNE_CACHE", raising=False)
    rng = np.random.default_rng(n)
    batch = lib.Batch(na=1.4, wavelength=600.0, n_i=1.518, pixel=100.0, plane_pitch=50.0, max_emitters=n, n_pupil=32)
    crop = rng.integers(lo, hi + 1, n)
    em = lib.make_emitters(np.zeros(n), np.zeros(n), np.zeros(n), crop, np.ones(n, dtype=int), np.zeros((n, 21)))
    I = torch.empty(lib.batch_offsets(em)[-1], device="cuda")
    cfg, ms = batch.autotune(em, I)
    batch.close()
    # fewer items than workgroups at one per CU: more per CU is the same grid; buckets that are not in use, and
    # 48 rows on the 64-row tile, launch nothing else
    rows = list(cfg["tile_rows"])
    assert cfg["wg_per_cu"] == 2 and ms > 0
    for q, (default, taller) in enumerate([(16, 64), (32, 64), (48, 48), (64, 64)]):
        assert rows[q] in ((default, taller) if lo <= 16 * (q + 1) <= hi else (default,))
