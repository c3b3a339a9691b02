"""The staging orders that the vector kernels read are found on the device; the rule is the host's, to the last tie: element for
element the same, for every tiling, on both sides of the channel counts where the device's search takes two, four or eight
blocks of chunks, with groups that are not full and filters that keep nothing."""
import numpy as np
import pytest

import paper_2001_07710_amd as pc
from workloads import layers as L

pytestmark = pytest.mark.gpu

TILINGS = [(16, 2, 32), (16, 1, 32), (8, 1, 32), (16, 2, 16), (16, 1, 16)]
NONE = 0xFFFFFFFF


@pytest.mark.parametrize("C,F,keep", [(1, 1, 1.0), (3, 70, 1.0), (31, 16, 0.5), (100, 72, 0.4), (256, 33, 0.3), (1008, 47, 0.2),
                                      (257, 17, 0.3), (512, 40, 0.25), (513, 16, 0.3),
                                      (1024, 16, 0.3), (1025, 40, 0.25), (1040, 33, 0.02), (2048, 65, 0.3), (2049, 32, 0.1)])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_the_orders_on_the_device_are_the_hosts(C, F, keep, dtype):
    print("[case]", C, F, keep, dtype, flush=True)
    r = np.random.default_rng(C * 7 + F)
    w = r.standard_normal((F, C, 3, 3)).astype(np.float16 if dtype == "f16" else np.float32)
    lib = np.array(L.drawn_library(4, 8), dtype=np.uint16)
    pid = r.integers(0, 8, (F, C)).astype(np.uint8)
    mask = (r.random((F, C)) < keep * r.uniform(0.2, 1.8, (F, 1))).astype(np.uint8)
    mask[r.random(F) < 0.1] = 0                              # filters that keep nothing
    host, device = pc.pack(w, lib, pid, mask, pc.PACK_HOST_ONLY), pc.pack(w, lib, pid, mask)
    filters = pc.packed_export(device)[0]
    for waves, nf, cc in TILINGS:
        got = pc.packed_order(device, waves, nf, cc)
        np.testing.assert_array_equal(got, pc.packed_order(host, waves, nf, cc))
        for g, row in enumerate(got):                        # (and it is an order: what the group's filters keep, once each)
            group = filters[g * waves * nf:(g + 1) * waves * nf]
            np.testing.assert_array_equal(np.sort(row[row != NONE]), np.nonzero(mask[group].any(axis=0))[0])
        if cc == 32:
            assert pc.packed_balance(device, waves, nf, True) == pc.packed_balance(host, waves, nf, True)
    with pytest.raises(pc.PconvError):
        pc.packed_order(device, 4, 1, 32)
    host.free()
    device.free()
