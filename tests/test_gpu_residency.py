"""Grids of the full resident capacity at table sizes where a block's LDS, rounded up to the units it
is given out in, decides how many blocks a CU holds: every block of the launch is resident
(the grid barriers complete), and the bits are those of a grid of one block per CU."""
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


# more rows than two 256-thread blocks per CU have wavefronts (2048), so that a third block per
# CU is launched wherever one counts as resident
CASES = [("2f", dict(n_flavor=2, n_energy=ne, n_u=1100)) for ne in (1063, 1070, 1089, 1090, 1943, 1944)] + \
        [("2f-all", dict(n_flavor=2, n_energy=ne, n_u=550, track_all=1)) for ne in (709, 715, 727)] + \
        [("2f-ext", dict(n_flavor=2, n_energy=ne, n_u=120, n_phi=10)) for ne in (248, 260, 276)] + \
        [("2f-ext-all", dict(n_flavor=2, n_energy=ne, n_u=60, n_phi=10, track_all=1)) for ne in (175,)]


@pytest.mark.parametrize("name,kw", CASES, ids=[f"{c[0]}-{c[1]['n_energy']}" for c in CASES])
def test_full_grids_are_resident(nb, name, kw):
    d = workloads.small_params(n_steps=2, **kw)
    m = nb.Model(d)
    got = {}
    for blocks in (0, 256):
        m.set_tuning(256, blocks)
        print(f"{name} {kw['n_energy']} energies: {m.get_tuning()['blocks']} blocks of 256", flush=True)
        m.reset()
        m.run()
        got[blocks] = m.get_state().cpu().numpy()
    np.testing.assert_array_equal(got[0], got[256])


# grids bounded by LDS (one block per CU at either size), and three-flavour grids bounded by
# max_blocks, give more rows a wavefront of their own at 512 threads; others keep 256
BLOCKS = [(dict(n_flavor=2, n_energy=1943, n_u=600), 256), (dict(n_flavor=2, n_energy=1944, n_u=512), 256),
          (dict(n_flavor=2, n_energy=1944, n_u=513), 512), (dict(n_flavor=2, n_energy=1350, n_u=300, track_all=1), 512),
          (dict(n_flavor=2, n_energy=1200, n_u=60, n_phi=9), 512),
          (dict(n_flavor=2, n_energy=20, n_u=40, max_blocks=20), 256),
          (dict(n_flavor=2, n_energy=20, n_u=41, max_blocks=20), 256),
          (dict(n_flavor=3, n_energy=20, n_u=40, max_blocks=20), 256),
          (dict(n_flavor=3, n_energy=20, n_u=41, max_blocks=20), 512),
          (dict(n_flavor=3, n_energy=20, n_u=512), 256), (dict(n_flavor=3, n_energy=20, n_u=513), 512)]


@pytest.mark.parametrize("kw,bs", BLOCKS, ids=["-".join(f"{k}{v}" for k, v in c[0].items()) for c in BLOCKS])
def test_default_block_size(nb, kw, bs):
    d = workloads.small_params(n_steps=2, **kw)
    m = nb.Model(d)
    print(kw, m.get_tuning(), flush=True)
    assert m.get_tuning()["block_threads"] == bs
    m.run()
    want = m.get_state().cpu().numpy()
    m.set_tuning(768 - bs)
    m.reset()
    m.run()
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), want)


def test_default_block_size_of_batches(nb):
    """Batches keep 256 threads, also where max_blocks bounds the grid."""
    ds = [workloads.small_params(n_flavor=2, n_energy=20, n_u=n, n_steps=2, max_blocks=4) for n in (9, 20)]
    assert nb.Model(ds).get_tuning() == dict(nb.Model(ds).get_tuning(), block_threads=256, blocks=4)


@pytest.mark.parametrize("kw", [dict(n_flavor=2, n_energy=1945, n_u=520), dict(n_flavor=2, n_energy=40, n_u=30, max_blocks=9),
                                dict(n_flavor=3, n_energy=40, n_u=30, max_blocks=9)],
                         ids=["lds", "2f-max_blocks", "3f-max_blocks"])
def test_adaptive_runs_in_bounded_grids(nb, oracle, kw):
    """Adaptive runs where the block size follows from the bound on the grid."""
    d = workloads.small_params(n_steps=4, r_start_km=600.0, r_end_km=600.2, **kw)
    o = oracle.Model(d)
    so = o.run_adaptive(1e-7)
    m = nb.Model(d, adaptive=True)
    st = m.run_adaptive(1e-7)
    assert (st["accepted"], st["rejected"]) == (so["accepted"], so["rejected"])
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())
