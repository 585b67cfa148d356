"""What the host table builder lays out, through kx_mech_info's device_bytes."""
import numpy as np
import pytest

from paper_2411_02640_amd import inputs as I
from paper_2411_02640_amd import kx


def _bytes(mech):
    h = kx.HostMechanism(mech)
    n = h.device_bytes
    h.close()
    return n


@pytest.mark.parametrize("spec", [I.MECH_9, I.MECH_53], ids=lambda s: s.name)
def test_all_zero_qss_flags(spec):
    """Flags that name no QSS species lay out the same tables as no flags."""
    mech = I.make_mechanism(spec)
    flagged = dict(mech, qss=np.zeros(mech["n_species"], np.int32))
    assert _bytes(flagged) == _bytes(dict(mech, qss=None))
