"""Near ties of the joining rule that single precision cannot see: the other end
lies near the centre of the first one's circle (a tenth of its radius away), where
the rounding of the positions weighs ten times as much in the arc and the tangent.
Each pair is at a cut to 1e-9 in double precision and more than a part in a
thousand beyond it in single precision; both sides flag it."""
import numpy as np
import pytest

import oracle

from _helix_frames import NROW
from test_gpu_merge import _gpu_merge

pytestmark = pytest.mark.gpu

# sector, row, y and z of both ends (2^-16 cm), q/pT, sin phi and tan lambda of the
# first one, sin phi of the second (a line): at the drift cut
DRIFT = [
    (6, 130, -551619, -490685, 6553600, 6588357, -644.9884033203125, 0.021186798810958862,
     7.979897975921631, 0.0),
    (2, 108, -342412, -282686, 6553600, 6547729, -657.1669921875, 0.012889130972325802,
     7.985280513763428, 0.0),
    (15, 113, -59778, 937, 6553600, 6501391, -647.4371948242188, 0.0027840808033943176,
     7.977591514587402, 0.0),
    (15, 140, -30663, 29598, 6553600, 6553772, -651.7422485351562, -0.013964196667075157,
     7.966055393218994, 0.0)]
# at the cut on the angle between the tangents
ANGLE = [
    (2, 130, -395406, -334848, 6553600, 6553600, -648.5043334960938, -0.010335724800825119, 0.0,
     -0.0011135792592540383),
    (2, 130, 613204, 673762, 6553600, 6553600, -648.5043334960938, -0.010335724800825119, 0.0,
     -0.0011135792592540383)]


@pytest.mark.parametrize("case", DRIFT + ANGLE)
def test_ties_near_a_centre(case):
    sector, row, ya, yb, za, zb, qpt, sa, tgl, sb = case
    y, z = np.array([ya, yb], np.int32), np.array([za, zb], np.int32)
    ur = sector * NROW + row
    cl = dict(crow_start=np.where(np.arange(18 * NROW + 1) > ur, 2, 0).astype(np.uint32), y_fx=y,
              z_fx=z, qtot=np.ones(2, np.uint16), qmax=np.ones(2, np.uint16),
              flags=np.zeros(2, np.uint8))
    par = np.array([[ya / 65536, 0, sa, tgl, qpt], [yb / 65536, 0, sb, 0, 0]], np.float32)
    tr = dict(par=par, row=np.full(2, row, np.uint8), z_anchor=z,
              hit_start=np.arange(3, dtype=np.uint32), hits=np.arange(2, dtype=np.uint32))
    o, g = oracle.merge_tracks(cl, tr, 18), _gpu_merge(cl, tr, 18, 1000)
    assert o["near_tie"].all()
    assert g["near_tie"].astype(bool).all()
    assert np.array_equal(g["label"].astype(np.int64), o["label"])
