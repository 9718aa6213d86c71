"""The grid reduction of the stage moments at the edges of its grid sizes and epoch tags: one
block (no exchange), at most eight (every copy has one block), nine and more (some or all
copies have several), past 512 barriers (the 9-bit tags and counts wrap); against the oracle,
bit for bit."""
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


@pytest.mark.parametrize("nf", [2, 3])
@pytest.mark.parametrize("blocks", [1, 2, 7, 8, 9, 16, 18])
def test_grid_sizes_and_tag_wrap(nb, oracle, nf, blocks):
    d = workloads.small_params(n_flavor=nf, n_energy=9, n_u=72, n_steps=300)
    print(f"reduction: {nf} flavours, {blocks} blocks, 1200 barriers", flush=True)
    m = nb.Model(d)
    m.set_tuning(512, blocks)
    assert m.get_tuning()["blocks"] == blocks
    m.run()
    o = oracle.Model(d)
    o.run()
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())


@pytest.mark.parametrize("n_u", [3, 40, 90])
def test_adaptive_grid_sizes(nb, oracle, n_u):
    d = workloads.small_params(n_flavor=2, n_energy=7, n_u=n_u, n_steps=200, r_start_km=600.0,
                               r_end_km=604.0)
    print(f"reduction: adaptive, {2 * n_u} rows", flush=True)
    m = nb.Model(d, adaptive=True)
    st = m.run_adaptive(1e-7)
    o = oracle.Model(d)
    so = o.run_adaptive(1e-7)
    assert (st["accepted"], st["rejected"]) == (so["accepted"], so["rejected"])
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())


@pytest.mark.parametrize("kw", [dict(), dict(n_phi=3)], ids=["bulb", "extended"])
@pytest.mark.parametrize("nf", [2, 3])
@pytest.mark.parametrize("n_energy", [1, 63, 64, 65, 1984, 1985, 2048, 2049, 4100])
def test_row_lengths(nb, oracle, nf, n_energy, kw):
    """Row sums at the edges of the lane chunks and of the 2048-energy row segments."""
    d = dict(workloads.small_params(n_flavor=nf, n_energy=n_energy, n_u=3, n_steps=3), **kw)
    print(f"row fold: {nf} flavours, {n_energy} energies, {kw}", flush=True)
    m = nb.Model(d)
    m.run()
    o = oracle.Model(d)
    o.run()
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())


@pytest.mark.parametrize("n_energy,n_u", [(65, 4), (96, 8), (130, 8), (2000, 4)])
def test_packed_tails_at_512_threads(nb, oracle, n_energy, n_u):
    """One row per wavefront of 512-thread blocks: the packed-row-tail variant."""
    d = workloads.small_params(n_flavor=3, n_energy=n_energy, n_u=n_u, n_steps=4)
    print(f"packed tails: {n_energy} x {n_u}", flush=True)
    m = nb.Model(d)
    m.set_tuning(512)
    m.run()
    o = oracle.Model(d)
    o.run()
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())


@pytest.mark.parametrize("nf,n_u", [(2, 4), (2, 5), (3, 4), (3, 5), (3, 512), (3, 513)])
def test_adaptive_block_sizes(nb, oracle, nf, n_u):
    """Adaptive runs at the row counts where the threads per block change."""
    d = workloads.small_params(n_flavor=nf, n_energy=5, n_u=n_u, n_steps=30, r_start_km=600.0,
                               r_end_km=601.0)
    print(f"adaptive: {nf} flavours, {2 * n_u} rows", flush=True)
    m = nb.Model(d, adaptive=True)
    st = m.run_adaptive(1e-7)
    o = oracle.Model(d)
    so = o.run_adaptive(1e-7)
    assert (st["accepted"], st["rejected"]) == (so["accepted"], so["rejected"])
    np.testing.assert_array_equal(m.get_state().cpu().numpy(), o.get_state())


@pytest.mark.parametrize("bs,blocks,steps", [(256, 0, 4200), (256, 1, 30), (256, 3, 30), (512, 1, 30)])
def test_batch_models_wait_for_their_own_rows(nb, oracle, bs, blocks, steps):
    """Batches in one launch: a wavefront per row, past 16384 epochs (the 14-bit tags and counts
    wrap); wavefronts with more rows than they keep, of several models (blocks meet after
    every step)."""
    ds = [workloads.small_params(n_energy=ne, n_u=nu, n_steps=steps, r_start_km=500.0,
                                 r_end_km=500.0 + 0.01 * steps, lum_erg_s=[le, 1e51, 2e51])
          for ne, nu, le in ((5, 3, 1e51), (70, 1, 2e51), (3, 40, 1.5e51), (64, 2, 3e51), (9, 11, 1e51))]
    print(f"batch: {bs} threads, {blocks} blocks, {steps} steps", flush=True)
    m = nb.Model(ds)
    m.set_tuning(bs, blocks)
    m.run()
    got = m.get_state().cpu().numpy()
    off = m.offsets()
    for i, d in enumerate(ds):
        o = oracle.Model(d)
        o.run()
        np.testing.assert_array_equal(got[:, off[i]:off[i + 1]], o.get_state())


@pytest.mark.parametrize("n_energy,n_u", [(8, 16), (8, 17), (64, 16), (64, 17), (64, 18), (128, 256), (129, 256),
                                          (512, 257), (1024, 257)])
def test_adjoint_grid_sizes(nb, oracle, n_energy, n_u):
    """The adjoint's sums at one block, at most eight, more than eight and many blocks, and at the
    beam counts where the block size and the beams per thread change; parameters and
    tolerance of the adjoint's own oracle test."""
    import torch
    d = workloads.small_params(n_flavor=2, n_energy=n_energy, n_u=n_u, n_steps=5, r_start_km=60.0,
                               r_end_km=61.5, n0_cm3=1e31, lum_erg_s=[3e50, 2e50, 1e50], theta=[0.5, 0.0, 0.0])
    print(f"adjoint: {2 * n_energy * n_u} beams", flush=True)
    o = oracle.Model(d)
    c = np.random.default_rng(5).uniform(-1.0, 1.0, o.nb) / o.nb
    _, go, sbo = o.adjoint(3, c, want_state_bar=True)
    m = nb.Model(d, adjoint_ckpt=3)
    g, sb = m.adjoint(torch.as_tensor(c, device="cuda"), want_state_bar=True)
    np.testing.assert_allclose(g, go, rtol=1e-9, atol=0)
    np.testing.assert_allclose(sb.cpu().numpy(), sbo, rtol=1e-9, atol=1e-9 * np.abs(sbo).max())
    m.reset()
    np.testing.assert_array_equal(m.adjoint(torch.as_tensor(c, device="cuda")), g)


@pytest.mark.parametrize("n_energy", [1, 21, 32, 63, 64, 65, 127, 128, 129, 1984, 1985])
@pytest.mark.parametrize("n_phi", [0, 2])
def test_row_groups_across_chunks(nb, oracle, n_energy, n_phi):
    """Rows streamed in groups, where a lane's next beam lies 64 beams further: rows that divide a
    64-lane chunk, fill it, or end one short of or one past it, and the longest row that is
    grouped.  n_phi = 0: a batch of two such models on one block (many rows to a wavefront);
    otherwise the extended model."""
    n_u = 4 if n_energy > 1000 else 37
    ds = [workloads.small_params(n_flavor=2, n_energy=n_energy, n_u=n_u + i, n_steps=3, r_start_km=100.0,
                                 r_end_km=100.1, n0_cm3=1e32, n_phi=n_phi) for i in range(1 if n_phi else 2)]
    print(f"row groups: {n_energy} energies, n_phi {n_phi}", flush=True)
    m = nb.Model(ds[0] if n_phi else ds)
    m.set_tuning(256, 1)
    m.run()
    got = m.get_state().cpu().numpy()
    at = 0
    for d in ds:
        o = oracle.Model(d)
        o.run()
        np.testing.assert_array_equal(got[:, at:at + o.nb], o.get_state())
        at += o.nb
