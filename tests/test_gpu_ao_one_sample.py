"""Ambient-occlusion rays of one sample a ray, which a workgroup takes 256 at a
time: whole workgroups, one ray more and one less, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2603_00292_amd import workloads as wl
from test_gpu_ao import _check_pixels, _run, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width, height", [(17, 15), (16, 16), (32, 16), (27, 19)])
def test_one_sample(gpu, orc, width, height):  # noqa: F811
    W = wl.ao_terrain(width, height, 1, k=336, nq=16)
    acc, (ao, h, ar, occ) = _run(gpu, W)
    S = orc.OracleScene.from_scene(W.scene)
    _check_pixels(orc, W, S, np.arange(width * height), h, ar, occ, ao, f"ao {width}x{height}x1")
    acc.close()
