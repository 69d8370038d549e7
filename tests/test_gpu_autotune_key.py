"""Which handles share a recorded layout choice (ALGMORTAR_AUTOTUNE_CACHE):
those of the same sizes and kernels.  Two chains of 1024 cells in two
subdomains differ in their longest subdomain only, 640 and 1000 rows; a record
without the set of layouts it was made with is not read at all."""
import numpy as np
import pytest

pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from tests.test_gpu_block_inverse import BOX, _band_matrix  # noqa: E402

pytestmark = pytest.mark.gpu


def _choice(sizes):
    A, _, part = _band_matrix(sizes, BOX, 1)
    h = am.AlgMortar(A, part, 2)
    c, us = h.tile_choice(1)
    h.close()
    assert len(us) == 3
    return c, any(u > 0 for u in us)


def test_key(tmp_path, monkeypatch):
    path = tmp_path / "cache.txt"
    monkeypatch.delenv("ALGMORTAR_TILE", raising=False)
    monkeypatch.setenv("ALGMORTAR_AUTOTUNE_CACHE", str(path))
    # a record of the band kernels, which had three layouts of other meanings
    path.write_text("n1024_m2_nl1_b2x0_p0_f1_pl0_nr1_c3 2\n")
    c, timed = _choice((640, 384))
    assert timed
    assert _choice((640, 384)) == (c, False)
    assert _choice((1000, 24))[1]
    keys = [line.split()[0] for line in path.read_text().splitlines()]
    assert len(set(keys)) == len(keys) == 3
