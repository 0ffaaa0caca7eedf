"""nbody_forces / nbody_accel on both sides of the entry counts from which they
build j records for fewer than one entry in 16 (1024 entries in FP64; elsewhere
2048 and 2^29 pairs, or 2^28 for FP64 and mixed accelerations, 2^27 in
double-single with jerk), and one wide item a CU, where its waves start to share
the j.  Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_0909_0879_amd import binding, ics
from tests.gpu_util import check_parity, is_mixed, require_gpu, to_np

pytestmark = pytest.mark.gpu

FP64, MIXED, DS = binding.FP64, binding.MIXED, binding.MIXED_DS


@pytest.mark.parametrize("prec,n,counts", [
    (FP64, 20000, (1023, 1024)),          # with jerk
    (FP64, 131072, (2047, 2048)),         # acceleration only: 2^28 pairs
    (MIXED, 131072, (2047, 2048)),        # the same
    (MIXED, 262144, (2047, 2048)),        # with jerk: 2^29 pairs
    (DS, 65536, (2047, 2048)),            # the same: 2^27
    (DS, 262144, (2047, 2048)),           # acceleration only: 2^29
    (MIXED, 4096, (3840, 4096)),          # 240 and 256 items of 256 slots
    (DS, 4096, (3840, 4096)),
])
def test_counts_around_the_lines(prec, n, counts):
    require_gpu()
    m, x, v = ics.plummer(n, 91)
    g = binding.NBody(m, x, v, eps=1e-3, precision=prec)
    g.set_tuning({"variant": binding.VARIANT_S1, "acc_variant": binding.VARIANT_S1,
                  "i_slots": [256] * 25})
    rng = np.random.default_rng(92)
    for na in counts:
        idx = np.sort(rng.choice(n, na, replace=False)).astype(np.int32)
        pick = np.sort(rng.choice(na, 256, replace=False))
        a_ref, j_ref = oracle.forces(x, v, m, 1e-3, idx=idx[pick].astype(np.int64))
        acc, jerk = (to_np(t) for t in g.forces(x, v, m, i_active=idx))
        only = to_np(g.accel(x, m, i_active=idx))
        g.sync()
        check_parity(acc[pick], jerk[pick], a_ref, j_ref, is_mixed(prec), f"n {n} na {na}")
        check_parity(only[pick], jerk[pick], a_ref, j_ref, is_mixed(prec), f"accel n {n} na {na}")
    g.close()
