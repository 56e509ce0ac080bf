"""GPU parity of the one-colour four-fermion operator (asqtad_npr_fourfermion through
the C ABI) against the FP64 oracle of Eq. (1).

Both sides compute in FP64 from the same links and propagators; they sum the same
terms in different orders, so each output agrees to 1e-12 of the operator's largest
entry (an FP64 sum of 256 products of 3 x 3 matrix products).  Every hypercube of
the small lattices is compared; at 20^3 x 64 a sample of hypercubes is.
"""
import ctypes

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def asq():
    import torch

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_1411_2223_amd as m

    m.load()
    return m


def random_props(dims, seed, n=4):
    V = int(np.prod(dims))
    rng = np.random.Generator(np.random.PCG64(seed))
    return [rng.standard_normal((V, 3, 3)) + 1j * rng.standard_normal((V, 3, 3)) for _ in range(n)]


def run_gpu(asq, dims, U, G, ops):
    import torch

    V = int(np.prod(dims))
    thin = asq.links_to_device(U.reshape(V, 4, 3, 3))
    props = [asq.links_to_device(g.reshape(V, 1, 3, 3)) for g in G]  # canonical complex128 -> float64 views
    out = asq.npr_fourfermion(dims, thin, props, ops)
    out2 = asq.npr_fourfermion(dims, thin, props, ops)
    torch.cuda.synchronize()
    assert torch.equal(out, out2), "not bitwise reproducible"
    a = out.cpu().numpy().view(np.complex128)
    return a.reshape(len(ops), V // 16, 3, 3, 3, 3)


def compare(got, want, label):
    for k in range(want.shape[0]):
        scale = np.abs(want[k]).max()
        err = np.abs(got[k] - want[k]).max() / scale
        print(f"{label} op {k}: max error {err:.2e} of max |V| {scale:.3e}", flush=True)
        assert err <= TOL


ALL_OPS = [(s1, f1, s2, f2) for s1, f1, s2, f2 in
           np.random.Generator(np.random.PCG64(7)).integers(0, 16, size=(40, 4)).tolist()]


@pytest.mark.parametrize("dims,nops", [((4, 4, 4, 4), 5), ((6, 4, 4, 8), 40), ((2, 4, 6, 4), 23)])
def test_npr_every_hypercube_small(asq, dims, nops):
    # 40 operators take two launches (32 per launch) and two passes of the
    # contraction loop (21 per pass); 23 a ragged second pass
    V = int(np.prod(dims))
    U = synth.thin_links(dims, 0.5, 21) if min(dims) >= 4 else None
    if U is None:  # extents of 2 are outside the thin-link generator: random SU(3) per link
        U = synth.su3_exp(np.random.Generator(np.random.PCG64(21)).standard_normal((V * 4, 8)), 0.5)
    U = U.reshape(V, 4, 3, 3)
    G = random_props(dims, 22)
    ops = ALL_OPS[:nops]
    got = run_gpu(asq, dims, U, G, ops)
    want = oracle.npr_fourfermion(dims, U, G, ops)
    compare(got, want, f"{dims}")


def test_npr_same_propagator_four_times(asq):
    # the four propagator arguments may be one array (one flavour)
    dims = (4, 4, 4, 4)
    V = int(np.prod(dims))
    U = synth.thin_links(dims, 0.3, 23).reshape(V, 4, 3, 3)
    G = random_props(dims, 24, n=1) * 4
    ops = [(0, 0, 0, 0), (15, 15, 15, 15), (5, 10, 5, 10)]
    compare(run_gpu(asq, dims, U, G, ops), oracle.npr_fourfermion(dims, U, G, ops), "one flavour")


def test_npr_full_size_sampled(asq):
    # the paper's 20^3 x 64 lattice shape, 16 operators, sampled hypercubes
    import torch

    w = synth.WORKLOADS["single_20x20x20x64"]
    dims = w["dims"]
    V = int(np.prod(dims))
    U = synth.thin_links(dims, w["eps"], synth.gauge_seed(w["index"])).reshape(V, 4, 3, 3)
    G = random_props(dims, 25, n=2)
    G = [G[0], G[0], G[1], G[1]]
    ops = [(s, 15, s, 15) for s in range(16)]
    thin = asq.links_to_device(U)
    props = [asq.links_to_device(g.reshape(V, 1, 3, 3)) for g in G]
    out = asq.npr_fourfermion(dims, thin, props, ops)
    torch.cuda.synchronize()
    nz = V // 16
    zs = np.unique(np.concatenate([[0, nz - 1], np.random.Generator(np.random.PCG64(26)).integers(0, nz, 14)]))
    got = out.view(len(ops), nz, 162)[:, torch.as_tensor(zs, device=out.device)].cpu().numpy()
    got = got.view(np.complex128).reshape(len(ops), len(zs), 3, 3, 3, 3)
    want = oracle.npr_fourfermion(dims, U, G, ops, zs=zs)
    compare(got, want, "20^3x64 sampled")


def test_npr_rejects_bad_arguments(asq):
    import torch

    dims = (4, 4, 4, 4)
    V = int(np.prod(dims))
    thin = torch.zeros(V * 72, dtype=torch.float64, device="cuda")
    g = torch.zeros(V * 18, dtype=torch.float64, device="cuda")
    out = torch.zeros(V // 16 * 162, dtype=torch.float64, device="cuda")
    d4 = (ctypes.c_int * 4)(*dims)

    def call(ops, o=out, dd=d4, gg=g):
        op = np.ascontiguousarray(np.asarray(ops, dtype=np.int32).reshape(-1, 4))
        return asq.asqtad_npr_fourfermion(dd, thin.data_ptr(), gg.data_ptr(), g.data_ptr(), g.data_ptr(),
                                          g.data_ptr(), op.shape[0], op.ctypes.data_as(ctypes.POINTER(ctypes.c_int)),
                                          o.data_ptr(), None)

    assert call([(16, 0, 0, 0)]) == asq.ASQ_EINVAL
    assert call([(0, -1, 0, 0)]) == asq.ASQ_EINVAL
    assert call([(0, 0, 0, 0)], o=g) == asq.ASQ_EINVAL  # output over a propagator
    assert call([(0, 0, 0, 0)], dd=(ctypes.c_int * 4)(4, 4, 3, 4)) == asq.ASQ_EINVAL
    assert call([(0, 0, 0, 0)], gg=g[1:]) == asq.ASQ_EINVAL  # misaligned
    assert call([(0, 0, 0, 0)]) == asq.ASQ_OK
    torch.cuda.synchronize()


def _partner(op):
    return (op[0] ^ 1, op[1], op[2] ^ 1, op[3])


def _op_lists():
    rng = np.random.Generator(np.random.PCG64(27))
    pool = [tuple(o) for o in rng.integers(0, 16, size=(60, 4)).tolist()]
    alone = []
    for o in pool:
        if o not in alone and _partner(o) not in alone:
            alone.append(o)
    mixed = alone[:12] + [_partner(o) for o in alone[:12]] + alone[12:17]
    rng.shuffle(mixed)
    return {"one": alone[:1], "one pair": [alone[0], _partner(alone[0])],
            "eight slots": [o for k in range(6) for o in (alone[k], _partner(alone[k]))] + alone[6:8],
            "nine slots": [(s, 15, s, 15) for s in range(16)] + alone[3:4],
            "no partners": alone[:16],  # a whole pass of the single form
            "mixed, 29": [tuple(int(v) for v in o) for o in mixed],
            "two launches": [tuple(int(v) for v in o) for o in mixed] + alone[17:25]}


@pytest.mark.parametrize("label", list(_op_lists()))
def test_npr_paired_operators(asq, label):
    """Operators and their partners (gamma_x on both bilinears), with every combination of the
    signs that relate them, against the oracle; the halved sums and differences of two operators
    round by 1e-16 of the larger sum of products, as the operators one by one do."""
    dims = (4, 4, 4, 4)
    U = synth.thin_links(dims, 0.5, 28).reshape(256, 4, 3, 3)
    G = random_props(dims, 29)
    ops = _op_lists()[label]
    compare(run_gpu(asq, dims, U, G, ops), oracle.npr_fourfermion(dims, U, G, ops), label)


def _graded_props(dims, seed, e):
    """Random propagators whose odd sites are scaled by e."""
    X, Y, Z, T = dims
    x = np.arange(int(np.prod(dims)))
    odd = (x % X + x // X % Y + x // (X * Y) % Z + x // (X * Y * Z)) & 1
    return [g * np.where(odd, e, 1.0)[:, None, None] for g in random_props(dims, seed)]


# eight pairs of operators that differ by gamma_x on both bilinears, so one of even and one of odd
# spin-taste parity each; and the same with other operators among them
@pytest.mark.parametrize("e", [1.0, 0.1, 1e-2, 1e-4])
@pytest.mark.parametrize("label", ["nine slots", "mixed, 29"])
def test_npr_accuracy_per_operator(asq, label, e):
    """Staggered propagators differ in size between the parities, and with them the operators: every
    operator is accurate relative to its own largest entry.  An entry sums 256 products whose
    roundings, a few 1e-16 of a product each, add up as a random walk, like the products
    themselves: 1e-14 of the largest entry leaves a factor of ten."""
    dims = (4, 4, 4, 4)
    U = synth.thin_links(dims, 0.5, 30).reshape(256, 4, 3, 3)
    G = _graded_props(dims, 31, e)
    ops = _op_lists()[label]
    got, want = run_gpu(asq, dims, U, G, ops), oracle.npr_fourfermion(dims, U, G, ops)
    err = [np.abs(got[k] - want[k]).max() / np.abs(want[k]).max() for k in range(len(ops))]
    print(f"graded by {e} {label}: largest error {max(err):.2e} of an operator's largest entry", flush=True)
    assert max(err) <= 1e-14


def test_npr_operator_does_not_depend_on_the_list(asq):
    """An operator has the same bits alone and among others, and is exactly zero where every product is."""
    dims = (4, 4, 4, 4)
    U = synth.thin_links(dims, 0.5, 32).reshape(256, 4, 3, 3)
    for e in (1.0, 0.0):
        G = _graded_props(dims, 33, e)
        for label in ("nine slots", "mixed, 29", "two launches"):
            ops = _op_lists()[label]
            got = run_gpu(asq, dims, U, G, ops)
            for k, op in enumerate(ops):
                print(f"list {label} e={e} op {k}", flush=True)
                assert np.array_equal(run_gpu(asq, dims, U, G, [op])[0], got[k])
                odd = any(bin(op[j] ^ op[j + 1]).count("1") & 1 for j in (0, 2))
                if e == 0.0 and odd:  # each product holds a propagator of an odd site
                    assert not np.any(got[k])
