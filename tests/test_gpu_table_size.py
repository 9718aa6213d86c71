"""Energy tables around the sizes where they stop fitting a block's LDS beside the stepper's own
arrays: every such model binds and gives the oracle's bits at either block size."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_1912_10596_amd as nb
    nb.lib()
    return nb


# doubles of a table: two flavours (2 + species rows) N_E, three (7 + species rows) N_E, and
# 2 N_phi; those of up to 96 KB (12288) may be staged in LDS
CASES = [(2, ne, 0, 3) for ne in (2300, 2360, 2500, 3070, 3073)] + \
        [(2, ne, 1, 3) for ne in (1560, 2047, 2049)] + \
        [(3, ne, 0, 3) for ne in (1364, 1366)] + [(3, ne, 1, 3) for ne in (944, 946)] + \
        [(2, 3072, 0, 0), (2, 3073, 0, 0), (3, 1365, 0, 0), (3, 1366, 0, 0)]


@pytest.mark.parametrize("nf,n_energy,track_all,n_phi", CASES)
def test_models_bind_at_every_table_size(nb, oracle, nf, n_energy, track_all, n_phi):
    d = dict(workloads.small_params(n_flavor=nf, n_energy=n_energy, n_u=3, n_steps=2), n_phi=n_phi,
             track_all=track_all)
    print(f"tables: {nf} flavours, {n_energy} energies, track_all {track_all}, n_phi {n_phi}", flush=True)
    o = oracle.Model(d, species4=track_all)
    o.run()
    m = nb.Model(d)
    m.run()
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())
    for bs in (256, 512):
        m.set_tuning(bs)
        assert m.get_tuning()["block_threads"] == bs
        m.reset()
        m.run()
        np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())
