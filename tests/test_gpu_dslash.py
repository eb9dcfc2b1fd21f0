"""GPU parity of the multi-rhs half Dslash, the M operator and the reductions against the oracle.

Tolerances: FP64 per element 1e-13 relative (floor 1e-2 rms for elements that cancel), FP32
relative L2 1e-6, FP32 arithmetic with FP16 link storage relative L2 2e-3 (binary16 rounds links
to 4.9e-4 relative).  Multi-rhs output must be bit-identical to single-rhs calls.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import DEV, check_f64_elem, make_lattice, rel_elem, rel_l2

torch = pytest.importorskip("torch")
from paper_1409_1510_amd import hisq  # noqa: E402

pytestmark = pytest.mark.gpu

# (dims, n): extents 4 alias the +3/-1 hops; 6 aliases +3/-3; ragged V/2 (not a multiple of the
# 256-site workgroup) and rhs counts that leave partial register tiles.
CASES = [((4, 4, 4, 4), 1), ((6, 4, 4, 8), 3), ((8, 6, 4, 10), 5), ((8, 8, 8, 8), 16),
         ((12, 4, 6, 8), 9)]


def _vecs(dims, n, seed):
    return synth.sources(dims, n, seed)


@pytest.mark.parametrize("dims,n", CASES)
@pytest.mark.parametrize("out_parity", [0, 1])
def test_f64_matches_oracle(dims, n, out_parity):
    lat, fat, naik = make_lattice(dims, 100)
    v = _vecs(dims, n, 101)
    got = lat.dslash(out_parity, hisq.HISQ_F64, torch.from_numpy(v).to(DEV)).cpu().numpy()
    ref = oracle.dslash_half(fat, naik, v, dims, out_parity)
    check_f64_elem(got, ref, f"dims={dims} n={n} parity={out_parity}")
    lat.close()


@pytest.mark.parametrize("dims,n", CASES)
@pytest.mark.parametrize("recon", [18, 14, 13, 9])
def test_f32_matches_oracle(dims, n, recon):
    lat, fat, naik = make_lattice(dims, 102, recon=recon)
    v = _vecs(dims, n, 103)
    for par in (0, 1):
        got = lat.dslash(par, hisq.HISQ_F32, torch.from_numpy(v).to(DEV).to(torch.complex64))
        ref = oracle.dslash_half(fat, naik, v, dims, par)
        err = rel_l2(got.cpu().numpy(), ref)
        print(f"FP32 r{recon} dims={dims} n={n} parity={par}: rel L2 {err:.3g}")
        assert err <= 1e-6
    lat.close()


@pytest.mark.parametrize("recon", [18, 14, 13, 9])
def test_f16_links_matches_oracle(recon):
    dims, n = (8, 6, 4, 10), 5
    lat, fat, naik = make_lattice(dims, 104, recon=recon)
    v = _vecs(dims, n, 105)
    for par in (0, 1):
        got = lat.dslash(par, hisq.HISQ_F16, torch.from_numpy(v).to(DEV).to(torch.complex64))
        ref = oracle.dslash_half(fat, naik, v, dims, par)
        err = rel_l2(got.cpu().numpy(), ref)
        print(f"FP16 links r{recon} parity={par}: rel L2 {err:.3g}")
        assert 1e-5 < err <= 2e-3  # above FP32 level: the links really are binary16
    lat.close()


@pytest.mark.parametrize("prec,recon", [(hisq.HISQ_F64, 18), (hisq.HISQ_F32, 18),
                                        (hisq.HISQ_F32, 14), (hisq.HISQ_F16, 18),
                                        (hisq.HISQ_F16, 14), (hisq.HISQ_F32, 13),
                                        (hisq.HISQ_F32, 9), (hisq.HISQ_F16, 9)])
def test_multi_rhs_bit_identical_to_single(prec, recon):
    dims = (8, 6, 4, 10)
    lat, fat, naik = make_lattice(dims, 106, recon=recon)
    dt = torch.complex128 if prec == hisq.HISQ_F64 else torch.complex64
    for n in (2, 7, 16, 23):
        v = torch.from_numpy(_vecs(dims, n, 107 + n)).to(DEV).to(dt)
        for par in (0, 1):
            multi = lat.dslash(par, prec, v)
            singles = torch.stack([lat.dslash(par, prec, v[i:i + 1].contiguous())[0] for i in range(n)])
            assert torch.equal(multi.view(torch.float64 if dt == torch.complex128 else torch.float32),
                               singles.view(torch.float64 if dt == torch.complex128 else torch.float32))
    lat.close()


def test_max_rhs_and_errors():
    dims = (4, 4, 4, 6)
    lat, fat, naik = make_lattice(dims, 108)
    n = hisq.HISQ_MAX_RHS
    v = _vecs(dims, n, 109)
    got = lat.dslash(1, hisq.HISQ_F64, torch.from_numpy(v).to(DEV)).cpu().numpy()
    ref = oracle.dslash_half(fat, naik, v, dims, 1)
    check_f64_elem(got, ref, f"n={n}")
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, n + 1, torch.from_numpy(v).to(DEV),
                              torch.from_numpy(v).to(DEV))
    assert e.value.code == hisq.HISQ_ERR_ARG
    x = torch.from_numpy(v[:1]).to(DEV)
    for bad_n in (0, -1):  # an empty bundle is an argument error, not a no-op launch
        for fn in (lambda: hisq.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, bad_n, x, x.clone()),
                   lambda: hisq.hisq_apply_m(lat.ctx, hisq.HISQ_F64, 0.1, bad_n, x, x.clone(), None),
                   lambda: hisq.hisq_dot_mrhs(lat.ctx, hisq.HISQ_F64, bad_n, x, x,
                                              torch.zeros(2, dtype=torch.float64, device=DEV))):
            with pytest.raises(hisq.HisqError) as e:
                fn()
            assert e.value.code == hisq.HISQ_ERR_ARG
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, 1, x, x)
    assert e.value.code == hisq.HISQ_ERR_ARG
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_dslash_mrhs(lat.ctx, 2, hisq.HISQ_F64, 1, x, x.clone())
    assert e.value.code == hisq.HISQ_ERR_ARG
    lat.close()


def test_misaligned_vectors_rejected():
    """A vector pointer that is not a multiple of its complex element size is refused with
    HISQ_ERR_ARG before anything is launched (the offset buffers stay in bounds either way)."""
    import ctypes
    dims = (4, 4, 4, 4)
    lat, fat, naik = make_lattice(dims, 111)
    lib = hisq.library()
    vp = ctypes.c_void_p
    for prec, dt, off in ((hisq.HISQ_F64, torch.complex128, 8), (hisq.HISQ_F32, torch.complex64, 4)):
        a = torch.zeros((2, 3, lat.vh), dtype=dt, device=DEV)
        b = torch.zeros_like(a)
        mis = vp(a.data_ptr() + off)
        assert lib.hisq_dslash_mrhs(lat.ctx, 1, prec, 1, mis, hisq._ptr(b)) == hisq.HISQ_ERR_ARG
        assert lib.hisq_dslash_mrhs(lat.ctx, 1, prec, 1, hisq._ptr(b), mis) == hisq.HISQ_ERR_ARG
        assert "aligned" in lib.hisq_last_error(lat.ctx).decode()
        assert lib.hisq_apply_m(lat.ctx, prec, 0.1, 1, mis, hisq._ptr(b), None) == hisq.HISQ_ERR_ARG
        dots = torch.zeros(4, dtype=torch.float64, device=DEV)
        assert lib.hisq_dot_mrhs(lat.ctx, prec, 1, mis, hisq._ptr(b), hisq._ptr(dots)) == hisq.HISQ_ERR_ARG
        assert lib.hisq_dot_mrhs(lat.ctx, prec, 1, hisq._ptr(a), hisq._ptr(b), vp(dots.data_ptr() + 4)) == hisq.HISQ_ERR_ARG
    x = torch.zeros((2, 3, lat.vh), dtype=torch.complex128, device=DEV)
    y = torch.zeros_like(x)
    prm = hisq.hisq_cg_params(kind=hisq.HISQ_CG_F64, tol=1e-8, max_iter=10, reliable_every=50,
                              link_prec=hisq.HISQ_F32, use_x0=0, check_every=0)
    assert lib.hisq_cg_mrhs(lat.ctx, 0.1, 1, vp(x.data_ptr() + 8), hisq._ptr(y), ctypes.byref(prm), None) == hisq.HISQ_ERR_ARG
    assert lib.hisq_z2_noise(lat.ctx, 1, 0, 1, vp(x.data_ptr() + 8)) == hisq.HISQ_ERR_ARG
    # the aligned calls still work afterwards
    assert lib.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, 1, hisq._ptr(x), hisq._ptr(y)) == hisq.HISQ_OK
    torch.cuda.synchronize()
    lat.close()


def test_binding_rejects_mismatched_rhs_counts():
    """The binding checks that every vector of a call holds the rhs count the library will read
    or write (a shorter output would be written past its end), before anything is launched."""
    dims = (4, 4, 4, 4)
    lat, fat, naik = make_lattice(dims, 112)
    a = torch.zeros((2, 3, lat.vh), dtype=torch.complex128, device=DEV)
    short = torch.zeros((1, 3, lat.vh), dtype=torch.complex128, device=DEV)
    with pytest.raises(ValueError):
        lat.dslash(1, hisq.HISQ_F64, a, short)
    with pytest.raises(ValueError):
        lat.apply_m(hisq.HISQ_F64, 0.1, a, short)
    with pytest.raises(ValueError):
        lat.dot(hisq.HISQ_F64, a, short)
    with pytest.raises(ValueError):
        lat.cg(0.1, a, x0=short)
    with pytest.raises(ValueError):  # wrong dtype for the precision
        lat.dslash(1, hisq.HISQ_F32, a)
    torch.cuda.synchronize()
    lat.close()


def test_state_and_link_errors():
    dims = (4, 4, 4, 4)
    lat = hisq.Lattice(dims, 0)
    x = torch.zeros((1, 3, lat.vh), dtype=torch.complex128, device=DEV)
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, 1, x, x.clone())
    assert e.value.code == hisq.HISQ_ERR_STATE
    fat, naik = synth.gauge_links(dims, 110)
    bad = fat.copy()
    bad[3, 1, 2, 2] = np.nan
    with pytest.raises(hisq.HisqError) as e:
        lat.load_links(bad, naik)
    assert e.value.code == hisq.HISQ_ERR_NONFINITE
    for recon in (14, 13, 9):  # fat links are not c * U(3): the compressed formats must refuse
        with pytest.raises(hisq.HisqError) as e:
            lat.load_links(naik, fat, naik_recon=recon)
        assert e.value.code == hisq.HISQ_ERR_ARG
    u1 = naik * np.exp(0.3j)  # c complex: U(3) but not a real multiple of SU(3)
    lat.load_links(fat, u1, naik_recon=14)
    for recon in (13, 9):
        with pytest.raises(hisq.HisqError) as e:
            lat.load_links(fat, u1, naik_recon=recon)
        assert e.value.code == hisq.HISQ_ERR_ARG
    # only the FP32 copy: FP64 calls fail cleanly
    lat.load_links(fat, naik, copies=hisq.HISQ_LINKS_F32)
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_dslash_mrhs(lat.ctx, 1, hisq.HISQ_F64, 1, x, x.clone())
    assert e.value.code == hisq.HISQ_ERR_STATE
    lat.close()


def test_links_from_device_memory():
    dims = (6, 4, 4, 8)
    fat, naik = synth.gauge_links(dims, 111)
    lat = hisq.Lattice(dims, 0)
    lat.load_links(torch.from_numpy(fat).to(DEV), torch.from_numpy(naik).to(DEV))
    with pytest.raises(ValueError):  # a device array of the wrong size is refused by the binding
        lat.load_links(torch.from_numpy(fat[:-1]).to(DEV), torch.from_numpy(naik[:-1]).to(DEV))
    v = _vecs(dims, 2, 112)
    got = lat.dslash(0, hisq.HISQ_F64, torch.from_numpy(v).to(DEV)).cpu().numpy()
    check_f64_elem(got, oracle.dslash_half(fat, naik, v, dims, 0), "links from device memory")
    lat.close()


@pytest.mark.parametrize("prec,tol", [(hisq.HISQ_F64, 1e-13), (hisq.HISQ_F32, 1e-6)])
def test_apply_m_and_pq(prec, tol):
    dims, n, mass = (8, 6, 4, 10), 6, 0.1
    lat, fat, naik = make_lattice(dims, 113)
    v = _vecs(dims, n, 114)
    dt = torch.complex128 if prec == hisq.HISQ_F64 else torch.complex64
    out, pq = lat.apply_m(prec, mass, torch.from_numpy(v).to(DEV).to(dt), with_pq=True)
    ref = oracle.m_ee(fat, naik, v, dims, mass)
    got = out.cpu().numpy()
    if prec == hisq.HISQ_F64:
        check_f64_elem(got, ref, "M operator", tol)
    else:
        assert rel_l2(got, ref) <= tol
    pq_ref = np.array([np.vdot(v[i], ref[i]).real for i in range(n)])
    assert np.max(np.abs(pq.cpu().numpy() - pq_ref) / pq_ref) <= (1e-12 if prec == hisq.HISQ_F64 else 1e-6)
    lat.close()


@pytest.mark.parametrize("prec", [hisq.HISQ_F64, hisq.HISQ_F32])
def test_dot(prec):
    dims, n = (8, 6, 4, 10), 5
    lat = hisq.Lattice(dims, 0)
    a = _vecs(dims, n, 115)
    b = _vecs(dims, n, 116)
    dt = torch.complex128 if prec == hisq.HISQ_F64 else torch.complex64
    ta, tb = torch.from_numpy(a).to(DEV).to(dt), torch.from_numpy(b).to(DEV).to(dt)
    got = lat.dot(prec, ta, tb).cpu().numpy()
    a2, b2 = ta.cpu().numpy().astype(np.complex128), tb.cpu().numpy().astype(np.complex128)
    ref = np.array([np.vdot(a2[i], b2[i]) for i in range(n)])
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
    # deterministic: same bits on a second call
    assert np.array_equal(got, lat.dot(prec, ta, tb).cpu().numpy())
    lat.close()


def test_full_size_32c8_sampled_sites():
    """The workload lattice 32^3 x 8 with 16 rhs, FP64 and FP32, in the benchmarked launch
    configuration: sampled output sites against the per-site oracle, plus the exact identity
    <a, D_oe b> = -<D_eo a, b> over the whole lattice."""
    cfg = synth.WORKLOADS["c1"]
    dims, n = cfg["dims"], 16
    lat, fat, naik = make_lattice(dims, synth.workload_seed("c1"))
    v = synth.sources(dims, n, synth.workload_seed("c1") + 1)
    rng = np.random.default_rng(5)
    sites = np.concatenate([[0, 1, lat.vh - 1], rng.choice(lat.vh, 40, replace=False)])
    tv = torch.from_numpy(v).to(DEV)
    for par in (0, 1):
        ref = oracle.dslash_sites(fat, naik, v, dims, par, sites)
        got64 = lat.dslash(par, hisq.HISQ_F64, tv).cpu().numpy()[:, :, sites]
        check_f64_elem(got64, ref, f"32^3x8 parity {par}")
        got32 = lat.dslash(par, hisq.HISQ_F32, tv.to(torch.complex64)).cpu().numpy()[:, :, sites]
        assert rel_l2(got32, ref) <= 1e-6
    a = torch.from_numpy(synth.sources(dims, n, 7)).to(DEV)
    b = torch.from_numpy(synth.sources(dims, n, 8)).to(DEV)
    lhs = lat.dot(hisq.HISQ_F64, lat.dslash(1, hisq.HISQ_F64, a), b)   # <D_oe a, b>  (odd)
    rhs = lat.dot(hisq.HISQ_F64, a, lat.dslash(0, hisq.HISQ_F64, b))   # <a, D_eo b>  (even)
    assert torch.max(torch.abs(lhs + rhs)) <= 1e-10 * torch.max(torch.abs(lhs))
    lat.close()


ALL_CFGS = ([(rt, spb, nt, 0, 0) for rt in (1, 2, 4, 8, 16) for spb in (256, 64) for nt in (0, 1)]
            + [(rt, 64, nt, lds, xm) for rt in (1, 2, 4) for lds in (1, 2, 3, 4, 5, 6) for xm in (0, 1, 2, 3)
               for nt in (0, 1)]
            + [(rt, 32, nt, lds, xm) for rt in (1, 2, 4) for lds in (0, 1, 2, 3) for xm in (0, 1, 2, 3)
               for nt in (0, 1)])


def _cfg_valid(prec, cfg, dims, recon=18):
    """The launch rules of the header: FP64 has no 16-rhs tile and no direction-pipelined form;
    the 16-wave LDS form and the direction-pipelined forms take at most 2 rhs per thread; the
    z-slab map needs (Lx/2)*Ly % 64 == 0 and Lz % 8 == 0, the y-slab map (Lx/2)*Ly % 512 == 0
    and its z-tiled walk also Lz % 4 == 0; 13- and 9-real Naik links have no 32-site and no
    direction-pipelined form."""
    rt, spb, nt, lds, xm = cfg
    plane = dims[0] // 2 * dims[1]
    if prec == hisq.HISQ_F64 and (rt == 16 or lds >= 4):
        return False
    if recon in (13, 9) and lds and (spb == 32 or lds >= 4):
        return False
    if spb == 32 and not (lds in (1, 2) and rt <= 2):
        return False
    if lds >= 3 and rt > 2:
        return False
    if xm == 1 and not (plane % 64 == 0 and dims[2] % 8 == 0):
        return False
    if xm in (2, 3) and plane % 512 != 0:
        return False
    if xm == 3 and dims[2] % 4 != 0:
        return False
    return True


@pytest.mark.parametrize("dims", [(8, 6, 4, 10), (16, 8, 8, 4), (16, 64, 8, 4), (6, 6, 4, 6)])
@pytest.mark.parametrize("prec,recon", [(hisq.HISQ_F64, 18), (hisq.HISQ_F32, 18),
                                        (hisq.HISQ_F32, 14), (hisq.HISQ_F16, 14),
                                        (hisq.HISQ_F32, 9), (hisq.HISQ_F16, 13)])
def test_every_launch_config_bit_identical(prec, recon, dims):
    """All register tiles, workgroup shapes, cache hints, the LDS-staged form and the XCD maps give
    the same bits, for the plain half Dslash and for the fused M operator (including its FP64
    <p, Mp> reduction; the 32-site form is plain-only and leaves the fused configuration as it
    was), and the autotuned choice is one of them.  Exactly the configurations the
    header rules out are refused.  (16, 8, 8, 4) admits the z-slab XCD map, (16, 64, 8, 4) the
    y-slab maps (two z tiles for the tiled walk); (6, 6, 4, 6) has V/2 = 432, so the last 64-site
    block of the LDS forms is ragged."""
    n, mass = 11, 0.1
    lat, fat, naik = make_lattice(dims, 120, recon=recon)
    dt = torch.complex128 if prec == hisq.HISQ_F64 else torch.complex64
    rdt = torch.float64 if prec == hisq.HISQ_F64 else torch.float32
    v = torch.from_numpy(_vecs(dims, n, 121)).to(DEV).to(dt)
    ref = oracle.dslash_half(fat, naik, _vecs(dims, n, 121), dims, 1)
    first = None
    tried = 0
    for cfg in ALL_CFGS:
        try:
            hisq.hisq_set_launch(lat.ctx, prec, n, cfg)
        except hisq.HisqError as e:
            assert e.code == hisq.HISQ_ERR_ARG
            assert not _cfg_valid(prec, cfg, dims, recon), cfg
            continue
        assert _cfg_valid(prec, cfg, dims, recon), cfg
        tried += 1
        out = lat.dslash(1, prec, v)
        m, pq = lat.apply_m(prec, mass, v, with_pq=True)
        cur = (out.view(rdt).clone(), m.view(rdt).clone(), pq.clone())
        if first is None:
            first = cur
            got = out.cpu().numpy()
            if prec == hisq.HISQ_F64:
                assert rel_elem(got, ref) <= 1e-13
            else:
                assert rel_l2(got, ref) <= (2e-3 if prec == hisq.HISQ_F16 else 1e-6)
        else:
            assert torch.equal(first[0], cur[0]), cfg
            assert torch.equal(first[1], cur[1]), cfg
            assert torch.equal(first[2], cur[2]), cfg
    assert tried >= 16
    print(f"prec {prec} r{recon}: {tried} launch configurations agree bit for bit")
    hisq.hisq_set_launch(lat.ctx, prec, n, None)
    best, ms = hisq.hisq_autotune(lat.ctx, prec, n, 0)
    assert best in ALL_CFGS and ms > 0
    assert hisq.hisq_get_launch(lat.ctx, prec, n, 0) == best
    assert torch.equal(lat.dslash(1, prec, v).view(rdt), first[0])
    lat.close()


@pytest.mark.parametrize("prec", [hisq.HISQ_F32, hisq.HISQ_F16])
def test_direction_pipelined_tile_limit(prec):
    """The direction-pipelined forms hold 16 (forms 4, 6) or 32 (form 5) rhs tiles per workgroup:
    n = 40 is refused with one rhs per thread and accepted as 20 tiles of 2 by form 5, with the
    same bits as the register-tile kernel."""
    dims, n = (8, 6, 4, 10), 40
    lat, fat, naik = make_lattice(dims, 125)
    v = torch.from_numpy(_vecs(dims, n, 126)).to(DEV).to(torch.complex64)
    hisq.hisq_set_launch(lat.ctx, prec, n, (2, 256, 0, 0, 0))
    ref = lat.dslash(1, prec, v).view(torch.float32).clone()
    for lds in (4, 5, 6):
        with pytest.raises(hisq.HisqError) as e:
            hisq.hisq_set_launch(lat.ctx, prec, n, (1, 64, 0, lds, 0))
        assert e.value.code == hisq.HISQ_ERR_ARG
    hisq.hisq_set_launch(lat.ctx, prec, n, (2, 64, 1, 5, 0))
    assert torch.equal(lat.dslash(1, prec, v).view(torch.float32), ref)
    m1, pq1 = lat.apply_m(prec, 0.1, v, with_pq=True)
    hisq.hisq_set_launch(lat.ctx, prec, n, (2, 256, 0, 0, 0))
    m0, pq0 = lat.apply_m(prec, 0.1, v, with_pq=True)
    assert torch.equal(m1.view(torch.float32), m0.view(torch.float32)) and torch.equal(pq1, pq0)
    lat.close()


_ROTATED = {}


def _rotated_tiled_links(dims):
    """A 4^4 random field tiled over `dims`, then rotated by a random local SU(3) gauge
    transformation: the links no longer repeat with period 4, so a link or neighbour read from a
    site shifted by a multiple of 4 fails the comparison (one lattice is kept at a time)."""
    if dims not in _ROTATED:
        _ROTATED.clear()
        fat, naik = synth.tiled_gauge_links(dims, 130)
        _ROTATED[dims] = synth.gauge_rotated(fat, naik, dims, 132)
    return _ROTATED[dims]


@pytest.mark.parametrize("name,prec,n", [("c3", hisq.HISQ_F32, 16), ("c3", hisq.HISQ_F16, 16),
                                         ("c3", hisq.HISQ_F64, 16), ("c4", hisq.HISQ_F32, 32),
                                         ("c4", hisq.HISQ_F16, 32), ("c4", hisq.HISQ_F64, 8)])
def test_full_size_48c12_64c16_sampled_sites(name, prec, n):
    """The 48^3 x 12 and 64^3 x 16 lattices at their rhs counts (FP64 at 64^3 x 16: 8 rhs), in
    the tuned launch configuration of each: sampled output sites (including the first and last of
    each parity) against the per-site oracle, on gauge-rotated tiled links (no period in the link
    values)."""
    dims = synth.WORKLOADS[name]["dims"]
    fat, naik = _rotated_tiled_links(dims)
    lat = hisq.Lattice(dims, 0)
    copies = hisq.HISQ_LINKS_F64 if prec == hisq.HISQ_F64 else hisq.HISQ_LINKS_F32 | hisq.HISQ_LINKS_F16
    lat.load_links(fat, naik, copies, 18)
    rng = np.random.default_rng(6)
    sites = np.concatenate([[0, 1, lat.vh - 1], rng.choice(lat.vh, 40, replace=False)])
    v = synth.sources(dims, n, 131)
    tv = torch.from_numpy(v).to(DEV)
    if prec != hisq.HISQ_F64:
        tv = tv.to(torch.complex64)
    print("launch", name, prec, n, hisq.hisq_get_launch(lat.ctx, prec, n, 0))
    for par in (0, 1):
        ref = oracle.dslash_sites(fat, naik, v, dims, par, sites)
        got = lat.dslash(par, prec, tv).cpu().numpy()[:, :, sites]
        if prec == hisq.HISQ_F64:
            check_f64_elem(got, ref, f"{name} parity {par}")
        else:
            err = rel_l2(got, ref)
            print(f"{name} prec {prec} parity {par}: rel L2 {err:.3g}")
            assert err <= (2e-3 if prec == hisq.HISQ_F16 else 1e-6)
    lat.close()


@pytest.mark.parametrize("name,prec,n,recon", [("c4", hisq.HISQ_F32, 32, 14), ("c4", hisq.HISQ_F16, 32, 9),
                                               ("c3", hisq.HISQ_F32, 16, 9), ("c3", hisq.HISQ_F16, 16, 13)])
def test_full_size_compressed_naik_sampled_sites(name, prec, n, recon):
    """Naik links stored as 14, 13 or 9 reals at 48^3 x 12 and 64^3 x 16, in an LDS launch under
    the lattice's XCD map (z slabs at 48^3 x 12, z-tiled y slabs at 64^3 x 16): sampled output
    sites against the per-site oracle on the full (uncompressed) gauge-rotated links, so every
    reconstruction is checked at the full volume."""
    dims = synth.WORKLOADS[name]["dims"]
    fat, naik = _rotated_tiled_links(dims)
    lat = hisq.Lattice(dims, 0)
    lat.load_links(fat, naik, hisq.HISQ_LINKS_F32 | hisq.HISQ_LINKS_F16, recon)
    cfg = (2, 64, 1, 2, 3 if name == "c4" else 1)
    hisq.hisq_set_launch(lat.ctx, prec, n, cfg)
    rng = np.random.default_rng(7)
    sites = np.concatenate([[0, 1, lat.vh - 1], rng.choice(lat.vh, 40, replace=False)])
    v = synth.sources(dims, n, 133)
    tv = torch.from_numpy(v).to(DEV).to(torch.complex64)
    for par in (0, 1):
        ref = oracle.dslash_sites(fat, naik, v, dims, par, sites)
        got = lat.dslash(par, prec, tv).cpu().numpy()[:, :, sites]
        err = rel_l2(got, ref)
        print(f"{name} prec {prec} r{recon} parity {par}: rel L2 {err:.3g}")
        assert err <= (2e-3 if prec == hisq.HISQ_F16 else 1e-6)
    lat.close()


def test_tuning_table_round_trip(tmp_path):
    """Tuned choices saved to a table are taken back by a new context on the same lattice and link
    formats; the file keeps other lattices' entries, and lines with an invalid configuration or
    another lattice are skipped on loading."""
    dims, n = (8, 6, 4, 10), 5
    path = tmp_path / "table.txt"
    foreign = "4 4 4 4 1 18 3 0 1 256 0 0 0 0.01000\n"
    path.write_text("# a comment line\n" + foreign)
    lat, fat, naik = make_lattice(dims, 130)
    tuned = {}
    for prec, fused in ((hisq.HISQ_F32, 0), (hisq.HISQ_F16, 1), (hisq.HISQ_F64, 0)):
        tuned[(prec, fused)], ms = hisq.hisq_autotune(lat.ctx, prec, n, fused)
        assert ms > 0
    hisq.hisq_save_tuning(lat.ctx, str(path))
    lat.close()
    text = path.read_text()
    assert foreign in text
    # an invalid register tile (3) and a different lattice for this context's formats
    lx, ly, lz, lt = dims
    path.write_text(text + f"{lx} {ly} {lz} {lt} 1 18 7 0 3 64 0 0 0 0.01000\n"
                           f"{lx} {ly} {lz} {lt + 2} 1 18 7 0 1 64 0 0 0 0.01000\n")
    lat2, _, _ = make_lattice(dims, 130)
    assert hisq.hisq_load_tuning(lat2.ctx, str(path)) == 3
    for (prec, fused), cfg in tuned.items():
        assert hisq.hisq_get_launch(lat2.ctx, prec, n, fused) == cfg
    lat2.close()


def _launch_ms(lat, prec, n, reps=20, sustain_ms=50.0):
    """Mean launch time of D_oe, D_eo pairs after `sustain_ms` of the same launches untimed (the
    device reaches its sustained speed for these kernels after some 30 ms of load)."""
    import time
    a = torch.randn(n, 3, lat.vh, dtype=torch.complex64, device=DEV) * 1e-30
    b = torch.empty_like(a)
    t = time.perf_counter()
    while (time.perf_counter() - t) * 1e3 < sustain_ms:
        for _ in range(5):
            lat.dslash(1, prec, a, b)
            lat.dslash(0, prec, b, a)
        torch.cuda.synchronize()
        a.mul_(1e-30)  # D grows a vector by at most ~9 per application: stay far from overflow
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        lat.dslash(1, prec, a, b)
        lat.dslash(0, prec, b, a)
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / (2 * reps)


def test_multi_rhs_gain_over_single_rhs():
    """The paper's qualitative claim (Section 1 and Table 1): bundling rhs more than doubles the
    Dslash flop rate from 1 to 4 rhs (FP32, 32^3 x 8, tuned launches).  The 14-real Naik gain at
    1 and 8 rhs (about 10 % and 3 % in the paper's model) is printed."""
    dims = (32, 32, 32, 8)
    fat, naik = synth.tiled_gauge_links(dims, 140)
    lat = hisq.Lattice(dims, 0)
    lat.load_links(fat, naik, hisq.HISQ_LINKS_F32, 18)
    ms = {n: _launch_ms(lat, hisq.HISQ_F32, n) for n in (1, 4, 8)}
    gain = (4 / ms[4]) / (1 / ms[1])
    print(f"FP32 ms per launch {ms}; flop-rate gain 1 -> 4 rhs: {gain:.2f}")
    assert gain >= 2.0
    lat.load_links(fat, naik, hisq.HISQ_LINKS_F32, 14)
    for n in (1, 8):
        r14 = _launch_ms(lat, hisq.HISQ_F32, n)
        print(f"r14 at n = {n}: {r14:.4f} ms against {ms[n]:.4f} ms ({100 * (ms[n] / r14 - 1):.1f} % faster)")
    lat.close()


def test_register_tile_offsets_fit_32_bits_on_large_lattices():
    """The register-tile Dslash indexes a rhs tile with 32-bit element offsets: on a lattice with
    V/2 = 100.7M sites (256^3 x 12; only the context is created, nothing is allocated) a tile of
    16 FP32 rhs (3 x 16 x V/2 > 2^32 elements) is refused, 8 are accepted, and the untuned
    heuristic never proposes a tile that does not fit."""
    lat = hisq.Lattice((256, 256, 256, 12), 0)
    with pytest.raises(hisq.HisqError) as e:
        hisq.hisq_set_launch(lat.ctx, hisq.HISQ_F32, 16, (16, 256, 0, 0, 0))
    assert e.value.code == hisq.HISQ_ERR_ARG
    hisq.hisq_set_launch(lat.ctx, hisq.HISQ_F32, 16, (8, 256, 0, 0, 0))
    assert hisq.hisq_get_launch(lat.ctx, hisq.HISQ_F32, 16, 0)[0] == 8
    for prec in (hisq.HISQ_F64, hisq.HISQ_F32):
        for n in (8, 32, 64):
            rt = hisq.hisq_get_launch(lat.ctx, prec, n, 1)[0]
            assert 3 * rt * lat.vh < 2 ** 32
    lat.close()


# ---- two sites per lane (16-byte gathers): lattices with Lx divisible by 4, FP32 and FP16 links ------

@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (4, 6, 4, 10), (8, 4, 6, 4), (12, 4, 4, 6), (20, 6, 4, 4),
                                  (32, 8, 4, 4)])
@pytest.mark.parametrize("recon", [18, 14, 13, 9])
def test_pair_form_is_bit_identical(dims, recon):
    """The LDS form with two sites per lane against the register-tile form, bit for bit: rows of 2
    sites (both x neighbours wrap) up to 16, a partial last block of 64 sites, rhs counts below,
    at and above a tile, vectors aligned to 8 bytes only, and the fused M form's <p, Mp>."""
    lat, _, _ = make_lattice(dims, 77, recon=recon)
    vh = lat.vh
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    for prec in (hisq.HISQ_F32, hisq.HISQ_F16):
        for n in (1, 2, 3, 4, 5, 9, 17):
            flat = torch.randn(2 * n * 3 * vh + 2, generator=g, dtype=torch.float32, device=DEV)
            v = torch.view_as_complex(flat[2:].view(-1, 2)).view(n, 3, vh)  # 8 bytes past a 16-byte boundary
            assert v.data_ptr() % 16 == 8
            ref = {}
            for cfg in [(1, 64, 0, 0, 0)] + [(rt, 64, nt, lds, 0) for rt in (2, 4) for nt in (0, 1)
                                             for lds in (1, 2, 3) if not (rt == 4 and lds == 3)]:
                hisq.hisq_set_launch(lat.ctx, prec, n, cfg)
                buf = torch.zeros(2 * n * 3 * vh + 2, dtype=torch.float32, device=DEV)
                out = torch.view_as_complex(buf[2:].view(-1, 2)).view(n, 3, vh)
                got = []
                for par in (1, 0):
                    lat.dslash(par, prec, v, out)
                    got.append(out.clone())
                q, pq = lat.apply_m(prec, 0.3, v, out, with_pq=True)
                got += [q.clone(), pq]
                if not ref:
                    ref = got
                for a, b in zip(got, ref):
                    assert torch.equal(torch.view_as_real(a) if a.is_complex() else a,
                                       torch.view_as_real(b) if b.is_complex() else b), (cfg, prec, n)
    lat.close()


# ---- launches too small to fill the chip: three waves per 64 sites, one per row --------------------

def _bits_over_configs(lat, prec, n, cfgs, g):
    """Both halves, M v and <v, Mv> of every configuration equal to the first one's, bit for bit."""
    v = torch.randn(n, 3, lat.vh, generator=g, device=DEV,
                    dtype=torch.complex128 if prec == hisq.HISQ_F64 else torch.complex64)
    ref = None
    for cfg in cfgs:
        hisq.hisq_set_launch(lat.ctx, prec, n, cfg)
        out = torch.zeros_like(v)
        got = []
        for par in (1, 0):
            lat.dslash(par, prec, v, out)
            got.append(torch.view_as_real(out).clone())
        q, pq = lat.apply_m(prec, 0.3, v, out, with_pq=True)
        got += [torch.view_as_real(q).clone(), pq]
        ref = ref or got
        for a, b in zip(got, ref):
            assert torch.equal(a, b), (cfg, prec, n)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,counts", [((4, 4, 4, 4), (1, 64)), ((6, 4, 10, 6), (1, 5, 43, 44)),
                                         ((8, 8, 8, 8), (1, 16, 17, 32, 33)), ((30, 10, 6, 4), (1, 9, 18, 19))])
def test_row_form_is_bit_identical(dims, counts):
    """64-site blocks times rhs up to and past the row form's limits (512 in FP64, 1024), and a
    partial last block; (1, 256, ...) is the register-tile kernel at every size."""
    lat, _, _ = make_lattice(dims, 78, recon=18)
    g = torch.Generator(device=DEV)
    g.manual_seed(6)
    for prec in (hisq.HISQ_F64, hisq.HISQ_F32, hisq.HISQ_F16):
        for n in counts:
            _bits_over_configs(lat, prec, n, [(1, 256, 0, 0, 0), (1, 64, 0, 0, 0), (1, 64, 1, 0, 0)], g)
    lat.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 4, 10, 6), (30, 10, 6, 4)])
def test_fp64_gather_ahead_form_is_bit_identical(dims):
    """The FP64 LDS form (one site per lane, gathers ahead) with partial rhs tiles and blocks."""
    lat, _, _ = make_lattice(dims, 79, recon=18)
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    for n in (1, 2, 3, 9, 17):
        _bits_over_configs(lat, hisq.HISQ_F64, n, [(1, 256, 0, 0, 0)] + [
            (rt, 64, nt, lds, 0) for rt in (1, 2) for nt in (0, 1) for lds in (1, 2, 3)], g)
    lat.close()
