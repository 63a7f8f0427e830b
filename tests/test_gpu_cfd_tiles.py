"""Convolution of the depth layers where its 16 x 16 tiles and its responses'
half-widths can go wrong, against the oracle at the bars of the other
convolution tests (FP32 scores in Q31.32 layers, FP64 sums): detectors of one
tile, one pixel more and fewer, and several; the largest response from one
pixel to 8 (four columns per thread) and beyond (one output per thread)."""
import math

import pytest

import phantoms
from test_gpu_cfd import cfd_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu,nv,angle", [
    (16, 16, 0.4), (17, 33, 1.0), (15, 31, 4.0), (32, 17, 6.0), (33, 16, 8.0), (33, 47, 8.9), (33, 47, 9.5), (40, 18, 12.0),
    (48, 48, 11.0)])
def test_cfd_tiles(nu, nv, angle):
    p = phantoms.thorax_problem("cfd_tiles", 24, 1.6, 3, 3, 180.0, nu, 38.4 / min(nu, nv), 200_000)
    cfd_parity(p.with_(nv=nv, accept_half_angle_rad=math.radians(angle)))
