"""GPU asqtad link construction (asqtad_build_links through the C ABI) against the FP64 oracle.

The oracle sums the asqtad paths one by one; the kernel evaluates nested
staples.  Both are FP64 and differ only in the order of the sums: each link
entry is a sum of at most 86 products of seven unitary-bounded matrices, so the
two agree to a few units of 1e-16 times |F| ~ 1; the bound used is 1e-13
absolute.  At the full 20^3 x 64 size the oracle computes sampled sites.
Solves on the constructed links are checked by the oracle's own operator built
from the oracle's links: relative true residual <= 1e-10.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

LINK_TOL = 1e-13


@pytest.fixture(scope="module")
def asq():
    import torch

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_1411_2223_amd as m

    m.load()
    return m


def _gpu_links(asq, dims, U, u0):
    import torch

    thin = asq.links_to_device(U.reshape(-1, 4, 3, 3))
    fat, lng = asq.build_links(dims, thin, u0)
    torch.cuda.synchronize()

    def host(t):
        return t.cpu().numpy().view(np.complex128).reshape(-1, 4, 3, 3)

    return host(fat), host(lng)


@pytest.mark.parametrize("dims,u0", [((4, 4, 4, 4), 1.0), ((6, 6, 4, 10), 0.87), ((4, 6, 8, 6), 1.0)])
def test_links_match_oracle(asq, dims, u0):
    # (6, 6, 4, 10): 1440 sites, 22.5 blocks of 64 -- a ragged last block
    print(f"links dims={dims} u0={u0}", flush=True)
    U = synth.thin_links(dims, 0.5, seed=41)
    fat, lng = _gpu_links(asq, dims, U, u0)
    want_f, want_l = oracle.asqtad_links(dims, U.reshape(-1, 4, 3, 3), u0)
    assert np.abs(fat - want_f).max() < LINK_TOL
    assert np.abs(lng - want_l).max() < LINK_TOL


def test_links_deterministic(asq):
    dims = (6, 4, 4, 8)
    U = synth.thin_links(dims, 0.4, seed=42)
    a = _gpu_links(asq, dims, U, 0.9)
    b = _gpu_links(asq, dims, U, 0.9)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_links_full_size_sampled(asq):
    """20^3 x 64 thin links of the single-solve workload, 300 sampled sites incl. the wrap edges."""
    w = synth.WORKLOADS["single_20x20x20x64"]
    dims = w["dims"]
    print(f"links full size dims={dims}", flush=True)
    U = synth.thin_links(dims, w["eps"], synth.gauge_seed(w["index"]))
    fat, lng = _gpu_links(asq, dims, U, 1.0)
    X, Y, Z, T = dims
    V = X * Y * Z * T
    rng = np.random.Generator(np.random.PCG64(7))
    edges = [0, V - 1, X - 1, X * Y - 1, X * Y * Z - 1, (T - 1) * X * Y * Z, V - X, V // 2 + X - 1]
    sites = np.concatenate([edges, rng.integers(0, V, size=300 - len(edges))])
    want_f, want_l = oracle.asqtad_links(dims, U.reshape(-1, 4, 3, 3), 1.0, sites=sites)
    assert np.abs(fat[sites] - want_f).max() < LINK_TOL
    assert np.abs(lng[sites] - want_l).max() < LINK_TOL


@pytest.mark.parametrize("mode", ["f64", "mixed32", "mixed16"])
def test_solve_on_constructed_links(asq, mode):
    import torch

    dims, u0, mass = (8, 8, 8, 8), 0.9, 0.05
    print(f"solve on built links mode={mode}", flush=True)
    U = synth.thin_links(dims, 0.3, seed=43)
    g = asq.Gauge.from_thin(dims, U.reshape(-1, 4, 3, 3), u0)
    b = synth.make_sources(dims, 2, seed=44)
    bd = asq.vec_to_device(b, "f64")
    res = g.solve([mass, 2 * mass], bd, mode=mode)
    torch.cuda.synchronize()
    x = asq.vec_from_device(res.x, 2, g.half, "f64")
    fat, lng = oracle.asqtad_links(dims, U.reshape(-1, 4, 3, 3), u0)
    for c, m in enumerate((mass, 2 * mass)):
        assert res.stats[c]["converged"]
        assert oracle.true_residual(dims, fat, lng, m, b[c], x[c]) <= 1e-10


def test_constructed_fat_links_refuse_compression(asq):
    import torch

    dims = (4, 4, 4, 8)
    U = synth.thin_links(dims, 0.3, seed=45)
    thin = asq.links_to_device(U.reshape(-1, 4, 3, 3))
    fat, lng = asq.build_links(dims, thin, 1.0)
    torch.cuda.synchronize()
    with pytest.raises(asq.AsqError) as e:
        asq.Gauge(dims, fat, lng, precs=("f64", "f32"), recon=12)
    assert e.value.code == asq.ASQ_ENOTSU3


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 4, 10), (20, 20, 20, 64)])
def test_plaquette_matches_oracle(asq, dims):
    # FP64 on both sides, different summation orders: 1e-13 absolute on a mean of order 1
    eps = 0.3 if dims[0] == 20 else 0.5
    U = synth.thin_links(dims, eps, seed=46)
    thin = asq.links_to_device(U.reshape(-1, 4, 3, 3))
    p1 = asq.plaquette(dims, thin)
    p2 = asq.plaquette(dims, thin)
    want = oracle.plaquette(dims, U.reshape(-1, 4, 3, 3))
    print(f"plaquette dims={dims}: gpu {p1!r} oracle {want!r}", flush=True)
    assert p1 == p2
    assert abs(p1 - want) < 1e-13


def test_tadpole_improved_construction(asq):
    # u0 from the plaquette: the links match the oracle's at that u0 and a solve meets the tolerance
    import torch

    dims, mass = (8, 8, 8, 8), 0.05
    U = synth.thin_links(dims, 0.3, seed=47)
    u0 = oracle.plaquette(dims, U.reshape(-1, 4, 3, 3)) ** 0.25
    g = asq.Gauge.from_thin(dims, U.reshape(-1, 4, 3, 3), u0="plaquette")
    fat, lng = oracle.asqtad_links(dims, U.reshape(-1, 4, 3, 3), u0)
    b = synth.make_sources(dims, 1, seed=48)
    res = g.solve([mass], asq.vec_to_device(b, "f64"), mode="mixed32")
    torch.cuda.synchronize()
    x = asq.vec_from_device(res.x, 1, g.half, "f64")
    assert res.rc == 0
    assert oracle.true_residual(dims, fat, lng, mass, b[0], x[0]) <= 1e-10


def _links_by(asq, dims, thin, u0, work_bytes):
    """(rc, fat, long) of asqtad_build_links (work_bytes None) or asqtad_build_links_work."""
    import ctypes

    import torch

    d4 = (ctypes.c_int * 4)(*dims)
    fat, lng = torch.full_like(thin, float("nan")), torch.full_like(thin, float("nan"))
    args = (d4, thin.data_ptr(), float(u0), fat.data_ptr(), lng.data_ptr())
    if work_bytes is None:
        rc = asq.asqtad_build_links(*args, asq.stream_ptr(None))
    else:
        work = torch.full((max(work_bytes, 256),), 255, dtype=torch.uint8, device="cuda")  # NaNs
        rc = asq.asqtad_build_links_work(*args, work.data_ptr(), work_bytes, asq.stream_ptr(None))
    torch.cuda.synchronize()
    return rc, fat, lng


# one block of 64 sites and a ragged one; extents of 4, where a two-site hop wraps to the
# same site both ways; more sites than four directions at a time fit (one per launch there)
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 4, 10, 6), (4, 14, 4, 6), (32, 32, 32, 34)])
def test_links_workspace_matches_workspace_free(asq, dims):
    """The staged form against the nested one on the same matrices.  Entries are sums of at most 86
    products of up to seven matrices with entries of rms 0.4: both round each product by 1e-16 of its
    size, so they agree to 1e-13 of the largest entry."""
    import ctypes

    import torch

    print(f"links with a workspace dims={dims}", flush=True)
    n = int(np.prod(dims)) * 4 * 18
    thin = torch.randn(n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3)) * 0.3
    need = asq.asqtad_links_workspace_bytes((ctypes.c_int * 4)(*dims))
    rc0, f0, l0 = _links_by(asq, dims, thin, 0.9, None)
    rc1, f1, l1 = _links_by(asq, dims, thin, 0.9, need)
    assert rc0 == 0 and rc1 == 0
    for a, b in ((f0, f1), (l0, l1)):
        assert float((a - b).abs().max()) <= 1e-13 * float(a.abs().max())
    assert _links_by(asq, dims, thin, 0.9, need - 256)[0] == asq.ASQ_ENOMEM


def test_build_links_on_side_stream(asq):
    """The binding's workspace belongs to the stream the kernels run on."""
    import torch

    dims = (6, 6, 4, 10)
    thin = asq.links_to_device(synth.thin_links(dims, 0.4, seed=44).reshape(-1, 4, 3, 3))
    want = asq.build_links(dims, thin, 0.9)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = asq.build_links(dims, thin, 0.9, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


# the last lattice of the kernel for small ones, the first beyond it, and a ragged one
@pytest.mark.parametrize("dims", [(16, 16, 16, 8), (16, 16, 10, 14), (18, 14, 22, 10)])
def test_plaquette_kernels_match_torch(asq, dims):
    """Both plaquette kernels against the definition in torch.  The mean of 6 V traces of products of
    three matrices, each rounded to a few 1e-16 of its size, agrees to 1e-13 of the mean trace size."""
    import torch

    X, Y, Z, T = dims
    print(f"plaquette dims={dims}", flush=True)
    n = X * Y * Z * T * 72
    thin = torch.randn(n, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    U = torch.view_as_complex(thin.reshape(T, Z, Y, X, 4, 3, 3, 2))
    want = scale = 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a = U[..., mu, :, :].contiguous() @ torch.roll(U[..., nu, :, :], -1, 3 - mu).contiguous()
            b = U[..., nu, :, :].contiguous() @ torch.roll(U[..., mu, :, :], -1, 3 - nu).contiguous()
            tr = (a * b.conj()).real.sum(dim=(-1, -2)) / 3
            want += float(tr.sum())
            scale += float(tr.abs().sum())
    got = asq.plaquette(dims, thin)
    assert abs(got - want / (6 * X * Y * Z * T)) <= 1e-13 * scale / (6 * X * Y * Z * T)


def _free_form(asq, dims, thin, u0):
    rc, fat, lng = _links_by(asq, dims, thin, u0, None)
    assert rc == 0
    return fat, lng


@pytest.mark.parametrize("side", [False, True])
def test_build_links_without_room_for_a_workspace(asq, monkeypatch, side):
    """Where the device has no room for the workspace, the binding takes the workspace-free call: its bits."""
    import torch

    dims = (8, 6, 10, 12)
    thin = torch.randn(5760 * 72, dtype=torch.float64, device="cuda",
                       generator=torch.Generator("cuda").manual_seed(6)) * 0.3
    want = _free_form(asq, dims, thin, 0.9)
    asked = []

    def full(n, device="cuda"):
        asked.append(n)
        raise torch.OutOfMemoryError("no room")

    monkeypatch.setattr(asq, "empty_bytes", full)
    stream = torch.cuda.Stream() if side else None
    torch.cuda.synchronize()
    print(f"links without room side={side}", flush=True)
    fat, lng = asq.build_links(dims, thin, 0.9, stream=stream)
    torch.cuda.synchronize()
    assert asked == [28 * 5760 * 144]
    assert torch.equal(fat, want[0]) and torch.equal(lng, want[1])


def test_build_links_under_capture(asq):
    """A captured call takes no workspace, which its replays would use after it is someone else's: every
    replay gives the eager bits of the workspace-free call, with other work in between."""
    import torch

    dims = (6, 6, 4, 10)
    thin = asq.links_to_device(synth.thin_links(dims, 0.4, seed=45).reshape(-1, 4, 3, 3))
    want = _free_form(asq, dims, thin, 0.9)
    fat, lng = torch.empty_like(thin), torch.empty_like(thin)
    asq.build_links(dims, thin, 0.9, fat=fat, lng=lng)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print("links under capture", flush=True)
    with torch.cuda.graph(graph):
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        asq.build_links(dims, thin, 0.9, fat=fat, lng=lng)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    for k in range(3):
        fat.zero_()
        lng.zero_()
        other = torch.randn(1 << 20, device="cuda")
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(fat, want[0]) and torch.equal(lng, want[1])
        assert bool(torch.isfinite(other).all())
