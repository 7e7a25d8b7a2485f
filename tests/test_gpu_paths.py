"""Kernel paths that a size rule chooses, against the path they replace or the
FP64 oracle, at the sizes where the split into workgroups can go wrong."""
import numpy as np
import pytest

from paper_2409_13958_amd import meshgen as mg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2409_13958_amd.binding")


def film(nx, ny, nz=1):
    return mg.kuhn_box((nx, ny, nz), 1e-9, periodic=0b011, jitter=0.1, grid=(16, 16, 4))


@pytest.mark.parametrize("lanes", [0, 4, 8, 16])
@pytest.mark.parametrize("nx, ny", [(4, 4), (4, 8), (5, 7), (16, 16)])
def test_products_of_m_in_one_launch_equal_the_single_kernels(nx, ny, lanes):
    """k_mprod (both terms, small cells) against k_exch alone, bit for bit, and
    its charges' sum; rows below, at and past a workgroup's share."""
    prob = film(nx, ny)
    ctx = B.Context.from_problem(prob, device=0)
    ctx.set_variant("spmv", lanes)
    n, _, nou, _ = ctx.query()
    m = torch.tensor(prob.m[nou], dtype=torch.float32, device="cuda")
    h, alone, hex_ = (torch.empty_like(m) for _ in range(3))
    q = torch.empty(n, dtype=torch.float32, device="cuda")
    ctx.heff_parts(m, h, q=q, hex=hex_)
    ctx.heff(m, alone, terms=B.TERM_EX)
    torch.cuda.synchronize()
    assert torch.equal(hex_, alone)
    loc = ctx.export("loc_val").reshape(-1, 8)[:, 1:4].astype(np.float64)
    rp, col = ctx.export("loc_rowptr"), ctx.export("loc_col")
    terms = (loc * m.cpu().numpy().astype(np.float64)[col]).sum(1)
    ref = np.add.reduceat(terms, rp[:-1])
    # FP32 sums of at most a few dozen terms: 64 roundings of the largest sum
    bound = 64 * 2.0 ** -24 * np.add.reduceat(np.abs(terms), rp[:-1]).max()
    assert np.abs(q.cpu().numpy() - ref).max() <= bound


@pytest.mark.parametrize("make", [
    lambda: film(4, 4),                       # one tile holds every row
    lambda: film(40, 33),                     # more than 32 rows per tile
    # spheres in an empty host: tiles without rows beside full ones
    lambda: mg.composite_c3(n_cells=24, grid=(21, 21, 21)),
    lambda: mg.kuhn_box((13, 17, 22), 1e-9, periodic=0b111, jitter=0.2, grid=(14, 18, 24)),
])
def test_interpolation_tiles_do_not_change_the_sums(make):
    """The tile shape only regroups the rows: the narrow tiles and those
    chosen by size give the same bits, alone and in a batch (larger tiles)."""
    prob = make()
    ctx = B.Context.from_problem(prob, device=0)
    _, _, nou, _ = ctx.query()
    m = torch.tensor(prob.m[nou], dtype=torch.float32, device="cuda")
    out = []
    for v in (0, 2, 1):
        ctx.set_variant("interp", v)
        out.append(torch.empty_like(m))
        ctx.heff(m, out[-1])
    other = B.Context.from_problem(film(60, 61), device=0)
    batch = B.Batch([ctx, other], spmv_lanes=4)
    ctx.set_variant("spmv", 4)
    ref = torch.empty_like(m)
    ctx.heff(m, ref)
    mb = torch.cat([m, torch.zeros((other.n, 3), device="cuda")])
    hb = torch.empty_like(mb)
    batch.heff(mb, hb)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    assert torch.equal(hb[:ctx.n], ref)
    batch.close()


@pytest.mark.parametrize("p, rb, nx, grid", [
    (1, 0, 5, (8, 8, 4)), (2, 1, 9, (12, 12, 4)), (3, 2, 16, (16, 16, 4)),
    (3, 2, 40, (16, 16, 4)),      # several batches of 64 nodes per wavefront
    (4, 1, 7, (16, 16, 8)), (5, 1, 12, (16, 16, 8)),
    # tiles of 25 boxes along x and y: the wavefronts that take nodes are two
    (5, 1, 6, (125, 125, 8)),
])
def test_scatter_anterpolation_against_the_tile_gather(p, rb, nx, grid):
    """Every order of the scatter kernel against the gather by tiles, at node
    counts below, at and past a wavefront's batch."""
    prob = mg.kuhn_box((nx, nx + 1, 2), 1e-9, periodic=0b011, jitter=0.1, grid=grid)
    ctx = B.Context.from_problem(prob, device=0, order_p=p, near_boxes=rb)
    _, _, nou, _ = ctx.query()
    m = torch.tensor(prob.m[nou], dtype=torch.float32, device="cuda")
    h = []
    for v in (3, 1):
        ctx.set_variant("anterp", v)
        h.append(torch.empty_like(m))
        ctx.heff(m, h[-1], terms=B.TERM_MS)
    torch.cuda.synchronize()
    # two FP32 sums of the same charges in other orders; the far field is a
    # part of H_ms of at most its size
    assert float((h[0] - h[1]).norm() / h[1].norm()) < 1e-5


@pytest.mark.parametrize("grid", [
    (16, 16, 4), (14, 15, 18), (18, 20, 21), (25, 24, 27), (28, 32, 30), (36, 35, 40),
    (42, 45, 16), (49, 50, 4), (54, 56, 5), (63, 60, 6), (64, 70, 4), (72, 75, 7), (81, 80, 4),
    (90, 84, 4), (96, 98, 4), (100, 105, 4), (108, 112, 5), (120, 125, 4), (126, 128, 4),
    (140, 140, 4), (144, 150, 4), (160, 162, 4), (243, 343, 4), (486, 500, 4), (512, 448, 4),
])
@pytest.mark.parametrize("fft", [1, 2])
def test_grid_convolution_of_every_kind_of_extent(grid, fft):
    """The transform passes against the same convolution by numpy in 64 bits:
    one to five passes, every radix, whole planes (shared by one to eight
    workgroups) and one axis at a time, padded and periodic axes."""
    prob = mg.kuhn_box((4, 4, 2), 1e-9, periodic=0b011, grid=grid, m=[0.0, 0.0, 1.0])
    ctx = B.Context.from_problem(prob, device=0)
    try:
        ctx.set_variant("fft", fft)
    except B.PmfemError:
        pytest.skip("the planes do not fit in LDS")
    info = ctx.export("grid_info")
    N, M = info[:3].astype(int), info[3:6].astype(int)
    rng = np.random.default_rng(grid[0] * 1000 + grid[1])
    q = rng.standard_normal(N[::-1])
    qt = torch.tensor(q, dtype=torch.float32, device="cuda")
    u = torch.empty_like(qt)
    ctx.grid_convolve(qt, u)
    khat = ctx.export("khat").reshape(M[2], M[1], M[0] // 2 + 1).astype(np.float64)
    s = tuple(M[::-1])
    ref = np.fft.irfftn(np.fft.rfftn(qt.cpu().numpy().astype(np.float64), s=s) * khat, s=s)
    ref = ref[:N[2], :N[1], :N[0]] * np.prod(M)
    torch.cuda.synchronize()
    err = np.linalg.norm(u.cpu().numpy() - ref) / np.linalg.norm(ref)
    # about log2(M) roundings of 2^-24 per axis and direction, at most doubled
    assert err < 2 * 2 * np.log2(np.prod(M)) * 2.0 ** -24


@pytest.mark.parametrize("nx, ny", [(4, 4), (5, 7), (9, 16)])
def test_rk4_steps_against_the_formula_and_across_calls(nx, ny):
    """Stage kernels against the RK4 formula on the library's own field; the
    steps of one call, of one call each, of a graph and of a batch agree."""
    probs = [film(nx, ny), film(4, 4)]
    ctxs = [B.Context.from_problem(p, device=0) for p in probs]
    ms = [torch.tensor(p.m[c.query()[2]], dtype=torch.float64, device="cuda")
          for p, c in zip(probs, ctxs)]
    ctx, m0 = ctxs[0], ms[0]
    dt, alpha, happ = 2e-14, 0.3, [1e4, -2e4, 3e4]
    gamma0 = 4e-7 * np.pi * 1.76086e11
    hmax = [0.0]

    def slope(v):
        h = torch.empty(v.shape, dtype=torch.float32, device="cuda")
        ctx.heff(v.to(torch.float32), h, h_applied=happ)
        h = h.to(torch.float64)
        hmax[0] = max(hmax[0], float(h.norm(dim=1).max()))
        c = torch.linalg.cross(v, h)
        return -gamma0 / (1 + alpha ** 2) * (c + alpha * torch.linalg.cross(v, c))

    ref = m0.clone()
    for _ in range(3):
        k1 = slope(ref)
        k2 = slope(ref + dt / 2 * k1)
        k3 = slope(ref + dt / 2 * k2)
        k4 = slope(ref + dt * k3)
        ref = ref + dt / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        ref = ref / ref.norm(dim=1, keepdim=True)
    one, each, graph = m0.clone(), m0.clone(), m0.clone()
    ctx.llg_step(one, dt, alpha, 3, h_applied=happ)
    for _ in range(3):
        ctx.llg_step(each, dt, alpha, 1, h_applied=happ)
    ctx.llg_step_graph(graph, dt, alpha, 3, h_applied=happ)
    torch.cuda.synchronize()
    assert torch.equal(one, each) and torch.equal(one, graph)
    # a last-bit difference of a stage may round one FP32 input of the field
    # the other way: 2^-24 of a field that sums a few dozen of them
    assert float((one - ref).abs().max()) <= 3 * gamma0 * dt * hmax[0] * 2.0 ** -18
    batch = B.Batch(ctxs)
    packed, single = torch.cat(ms), torch.cat(ms)
    batch.llg_step(packed, dt, alpha, 3)
    for _ in range(3):
        batch.llg_step(single, dt, alpha, 1)
    torch.cuda.synchronize()
    assert torch.equal(packed, single)


@pytest.mark.parametrize("nx, ny, grid, terms, dt", [
    (4, 4, (16, 16, 4), 3, 1e-14),
    (9, 16, (16, 16, 4), 3, 3e-13),        # more basis vectors than one chunk of products
    (260, 256, (128, 128, 4), 1, 1e-13),   # more nodes than the workgroups take at once
])
def test_implicit_step_solves_its_equation(nx, ny, grid, terms, dt):
    """The step's residual, from the library's own field of the midpoint."""
    prob = mg.kuhn_box((nx, ny, 1), 1e-9, periodic=0b011, jitter=0.1, grid=grid)
    ctx = B.Context.from_problem(prob, device=0)
    _, _, nou, _ = ctx.query()
    m = torch.tensor(prob.m[nou], dtype=torch.float64, device="cuda")
    m = 0.05 * m + torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device="cuda")
    m = m / m.norm(dim=1, keepdim=True)
    x, alpha, tol = m.clone(), 0.3, 1e-5
    ctx.llg_implicit(x, dt, alpha, 1, terms=terms, tol=tol)
    mb = 0.5 * m + 0.5 * x
    h = torch.empty(m.shape, dtype=torch.float32, device="cuda")
    ctx.heff(mb.to(torch.float32), h, terms=terms)
    h = h.to(torch.float64)
    c = torch.linalg.cross(mb, h)
    c = c + alpha * torch.linalg.cross(mb, c)
    g = x - m + dt * 4e-7 * np.pi * 1.76086e11 / (1 + alpha ** 2) * c
    # Newton stops at tol; the FP64 roundings of this formula are 1e-14 of it
    assert float(g.pow(2).mean().sqrt()) <= tol * (1 + 1e-3)


@pytest.mark.parametrize("grid, nw", [((75, 75, 50), 2), ((75, 75, 75), 1)])
def test_scatter_of_the_largest_footprints(grid, nw):
    """Tiles of 15 boxes at p = 5, whose footprint leaves LDS for two copies
    or for one, against the gather by tiles."""
    prob = mg.kuhn_box((6, 7, 6), 1e-9, periodic=0b111, jitter=0.1, grid=grid)
    ctx = B.Context.from_problem(prob, device=0, order_p=5, near_boxes=1)
    fd = ctx.export("sc_plan")[6:9]
    padded = 4 * fd[2] * ((fd[0] * fd[1] - 16 + 31) // 32 * 32 + 16)
    assert fd[0] % 8 == 4 and min(4, 1 << int(np.log2((65536 - 12288) // padded))) == nw
    _, _, nou, _ = ctx.query()
    m = torch.tensor(prob.m[nou], dtype=torch.float32, device="cuda")
    h = []
    for v in (3, 1):
        ctx.set_variant("anterp", v)
        h.append(torch.empty_like(m))
        ctx.heff(m, h[-1], terms=B.TERM_MS)
    torch.cuda.synchronize()
    # as in the test of every order above
    assert float((h[0] - h[1]).norm() / h[1].norm()) < 1e-5


def convolution_error(ctx, seed):
    """Relative L2 error of the grid convolution against numpy in 64 bits, and
    the bound: about log2(M) roundings of 2^-24 per axis and direction, at most
    doubled."""
    info = ctx.export("grid_info")
    N, M = info[:3].astype(int), info[3:6].astype(int)
    q = np.random.default_rng(seed).standard_normal(N[::-1]).astype(np.float32)
    u = torch.empty(tuple(N[::-1]), dtype=torch.float32, device="cuda")
    ctx.grid_convolve(torch.tensor(q, device="cuda"), u)
    khat = ctx.export("khat").reshape(M[2], M[1], M[0] // 2 + 1).astype(np.float64)
    s = tuple(M[::-1])
    ref = np.fft.irfftn(np.fft.rfftn(q.astype(np.float64), s=s, axes=(0, 1, 2)) * khat, s=s,
                        axes=(0, 1, 2))[:N[2], :N[1], :N[0]] * np.prod(M)
    err = np.linalg.norm(u.cpu().numpy() - ref) / np.linalg.norm(ref)
    return err, 2 * 2 * np.log2(np.prod(M)) * 2.0 ** -24


@pytest.mark.parametrize("grid", [(48, 400, 4), (60, 324, 5), (125, 160, 4), (392, 50, 4),
                                  (400, 49, 4), (490, 40, 4)])
def test_planes_that_fit_in_lds_only_at_unpadded_strides(grid):
    ctx = B.Context.from_problem(mg.kuhn_box((4, 4, 2), 1e-9, periodic=0b011, grid=grid,
                                             m=[0.0, 0.0, 1.0]), device=0)
    ctx.set_variant("fft", 2)
    err, bound = convolution_error(ctx, grid[0])
    assert err < bound


@pytest.mark.parametrize("nx, ny", [
    (64, 65),      # 17 workgroups: a second share for one of the 16 lanes of a sum
    (256, 257),    # 257: a second batch of loads
    (516, 512),    # more nodes than 1024 workgroups take at once
])
def test_implicit_step_by_number_of_workgroups(nx, ny):
    """The sums over the workgroups' shares, as in the test above."""
    test_implicit_step_solves_its_equation(nx, ny, (128, 128, 4), 1, 1e-13)


@pytest.mark.parametrize("periodic, grid", [(0b011, (375, 16, 4)), (0b011, (16, 375, 4)),
                                            (0b111, (16, 14, 375))])
@pytest.mark.parametrize("fft", [1, 2])
def test_transforms_of_four_passes(periodic, grid, fft):
    """375 = 3 * 5 * 5 * 5 is the one extent that takes four passes, the most
    of any, along each axis in turn."""
    ctx = B.Context.from_problem(mg.kuhn_box((4, 4, 4), 1e-9, periodic=periodic, grid=grid,
                                             m=[0.0, 0.0, 1.0]), device=0)
    ctx.set_variant("fft", fft)
    err, bound = convolution_error(ctx, sum(grid))
    assert err < bound
