"""Edges of the kernels' tilings and of the dispatch rules between them, on the
GPU against the serial oracle: fixed point bit for bit, FP64 within 1e-12 of
each field's largest magnitude (the accumulation's rounding, as in the other
parity tests)."""
import dataclasses

import numpy as np
import pytest

from paper_2509_18261_amd import workloads as W

from test_gpu_snr import B, check  # noqa: F401  (B is the binding fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("acc", ["fix64", "f64"])
@pytest.mark.parametrize("r_k,sub", [(0.0, 16), (0.5, 2), (1.0, 1), (2.5, 8), (5.0, 2), (9.25, 1),
                                     (16.0, 16)])
def test_snr_kernel_sizes(B, orc, r_k, sub, acc):  # noqa: F811
    """Remnant kernels from the host cell alone to the largest radius and
    finest sampling (the longest cell list in LDS), with remnants on cell
    corners, centres and sample points (exact ties of the distance test) and
    at domain corners (kernels that wrap)."""
    w = W.snr_box(nx=36, n_snr=3, seed=31, dtype=np.float64)
    pts = np.array([[18.0, 18.0, 18.0], [7.5, 20.5, 30.5], [0.0, 35.999, 0.25],
                    [12.0 + 0.5 / sub, 9.0 + 0.5 / sub, 17.0 + 0.5 / sub], [3.3, 30.1, 11.7]])
    n = len(pts)
    f = {"m": np.full(n, W.SNR_M_EJ), "e": np.full(n, W.SNR_E_SN)}
    vel = np.random.default_rng(5).standard_normal((3, n))
    f.update(vx=vel[0], vy=vel[1], vz=vel[2])
    w = dataclasses.replace(w, name=f"snr_r{r_k}_s{sub}", ghost=17, snr=W._one_box(pts, f),
                            snr_params=dataclasses.replace(w.snr_params, r_k=r_k, sub=sub))
    check(B, orc, w, acc)


@pytest.mark.parametrize("kind", ["cic", "sn"])
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8193])
def test_binning_slices(B, orc, n, kind):  # noqa: F811
    """One tile's entries around the slice length of the second sorting level,
    every other bucket empty, and one particle kind absent (more tiles than
    the sort of small deposits takes)."""
    from test_gpu_parity import check as check_deposit
    rng = np.random.default_rng(n)
    pos = 20.0 + 0.9 * rng.random((n, 3))
    w = W.c2(nx=80, n_cic=1, n_sn=1, dtype=np.float64)
    if kind == "cic":
        w = dataclasses.replace(w, name=f"slice_cic_{n}", sn=None,
                                cic=W._one_box(pos, W.cic_fields(rng, n)))
    else:
        w = dataclasses.replace(w, name=f"slice_sn_{n}", cic=None,
                                sn=W._one_box(pos, W.sn_fields(n, 1.5)))
    check_deposit(B, orc, w, "fix64", tuning={"deposit_path": 1, "tile_x": 16, "tile_yz": 2})


@pytest.mark.parametrize("fuse", [0, 2])
@pytest.mark.parametrize("n_cic,n_sn,nx,tile", [
    (0, 1, 24, (16, 8)), (1, 0, 24, (16, 8)), (256, 64, 40, (64, 4)), (257, 65, 40, (32, 2)),
    (5000, 1025, 61, (16, 2)), (12000, 2000, 62, (16, 2)),   # 3844 to 8192 and more tiles
    (199992, 1, 33, (32, 4)), (199993, 1, 33, (32, 4)),      # either side of the entry limit
    (100000, 100, 96, (16, 4)),
])
def test_sort_of_small_deposits(B, orc, n_cic, n_sn, nx, tile, fuse):  # noqa: F811
    """Deposits on either side of the rule that sends a sort to the short
    launches (8192 tiles, 200000 entries), around the block sizes of its
    kernels, on uneven boxes too, and with tiles split into chunks."""
    from test_gpu_parity import step_vs_oracle
    rng = np.random.default_rng(n_cic + n_sn + nx)
    edges = ([nx], [nx], [nx]) if nx % 2 == 0 else ([nx // 3, nx - nx // 3], [nx],
                                                     [nx // 2, nx - nx // 2])
    dom = (nx, nx, nx)
    pc = W.clumped_positions(rng, n_cic, dom, nclump=2, a=3.0) if n_cic else None
    ps = W.uniform_positions(rng, n_sn, dom) if n_sn else None
    w = W.multibox(*edges, 4, positions_cic=pc, positions_sn=ps, sn_radius=3.0, seed=nx)
    step_vs_oracle(B, orc, w, "fix64",
                   tuning=dict(deposit_path=1, tile_x=tile[0], tile_yz=tile[1], chunk_cic=1024,
                               chunk_sn=64, fuse_apply=fuse))


@pytest.mark.parametrize("form", ["calls", "owner"])
def test_binning_beside_the_member_count(B, orc, form):  # noqa: F811
    """Supernovae are binned without knowing their member counts: spheres that
    hold no cell centre, one, or (a particle on a cell corner, r^2 at its eight
    centres' distance) eight by an exact tie, from every lane count; then ones
    skipped for a mass or an energy that is not finite or overflows."""
    from test_gpu_parity import _add_particle, _flags, compare, run_gpu, step_vs_oracle
    rng = np.random.default_rng(8)
    tie = float(np.sqrt(0.75))
    rad = [0.0, 0.3, 0.5, np.nextafter(tie, 0.0), np.nextafter(tie, 1.0), 0.87, 2.0, 4.0]
    pos, r = [], []
    for q in rad:
        for p in ([10.0, 20.0, 30.0], [7.5, 8.5, 9.5], [0.0, 0.0, 0.0], [79.999, 0.25, 40.0],
                  *(80.0 * rng.random((5, 3)))):
            pos.append(p)
            r.append(q)
    f = W.sn_fields(len(r), 4.0)
    f["r"][:] = r
    w = W.c2(nx=80, n_cic=500, n_sn=1, dtype=np.float64)
    w = dataclasses.replace(w, sn=W._one_box(np.array(pos), f))
    tun = {"deposit_path": 1, "tile_x": 16, "tile_yz": 2}  # more tiles than the short sort takes
    for lanes in (1, 2, 4, 8, 16) if form == "owner" else (4,):
        if form == "owner":
            step_vs_oracle(B, orc, w, "fix64", tuning=dict(tun, fuse_apply=2, count_lanes=lanes))
            continue
        sn = _add_particle(w.sn, (40.1, 41.2, 42.3), e=float("nan"))
        sn = _add_particle(sn, (50.1, 41.2, 42.3), m=float("inf"), r=0.3)
        sn = _add_particle(sn, (60.5, 61.5, 62.5), m=1e7, r=0.0)
        got = run_gpu(B, dataclasses.replace(w, sn=sn), "fix64", tuning=tun)
        assert _flags(got) & 0x8 and "OVERFLOW" in got["status"]["flag_names"], got["status"]
        compare(w, "fix64", got, orc.step(w, "fix64", want_eta=True))


@pytest.mark.parametrize("acc", ["fix64", "f64"])
@pytest.mark.parametrize("r_k,sub", [(0.3, 2), (3.0, 4), (4.5, 2), (4.75, 2), (8.25, 1)])
def test_snr_many_remnants(B, orc, r_k, sub, acc):  # noqa: F811
    """More remnants than workgroups of four wavefronts fit the chip, on either
    side of the radius up to which one wavefront takes a whole remnant, and
    with kernels too wide for a cell list."""
    w = W.snr_box(nx=40, n_snr=2100, seed=33, dtype=np.float64)
    w = dataclasses.replace(w, name=f"many_r{r_k}_s{sub}", ghost=10,
                            snr_params=dataclasses.replace(w.snr_params, r_k=r_k, sub=sub))
    check(B, orc, w, acc)
