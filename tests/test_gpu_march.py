"""tau_g = 1 steps pass the sum of the populations from one to the next: as marches in
strips of 58 columns, or several in one launch on regions of 64 columns x 16 or 32 rows
where the lattice is small.  The state a call leaves and the order parameter it records
are bitwise those of single steps."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _populations(buf, nx, ny, storage):
    """The stored values of a saved state without the padding of its rows."""
    pitch = (nx + 31) // 32 * 32
    if storage == 0:
        return buf.view(torch.int32).view(ny, 9, pitch)[:, :, :nx].contiguous()
    rows = buf.view(ny, 20 * pitch)
    rest = rows[:, :4 * pitch].reshape(ny, pitch, 4)[:, :nx].reshape(ny, -1)
    moving = rows[:, 4 * pitch:].reshape(ny, 8, pitch, 2)[:, :, :nx].reshape(ny, -1)
    return torch.cat([rest, moving], 1)


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("nx,ny", [(5, 4), (40, 23), (58, 64), (61, 7), (117, 65), (256, 250), (250, 300),
                                   (300, 517), (701, 640)])
def test_many_steps_equal_single_steps(nx, ny, storage):
    import paper_1805_00007_amd as lbm
    rng = np.random.default_rng(nx * 1000 + ny)
    phi0 = np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1)
    tables = dict(ax=rng.uniform(-.04, .04, nx), ay=rng.uniform(-1, 1, ny),
                  bx=rng.uniform(-.04, .04, nx), by=rng.uniform(-1, 1, ny),
                  tf=np.cos(0.1 * np.arange(20)))
    field = (rng.uniform(-.04, .04, (ny, nx)), rng.uniform(-.04, .04, (ny, nx)))
    for model, vel in ((1, dict(velocity=tables)), (2, dict(velocity=tables)),
                       (1, dict(field=field)), (2, dict(field=field))):
        print(nx, ny, storage, model, list(vel), flush=True)
        one, many, rec = (lbm.Solver(nx, ny, phi0, storage=storage, **vel,
                                     **dict(workloads.PRESCRIBED, model=model))
                          for _ in range(3))
        phis = []
        for _ in range(13):
            phis.append(one.phi())
            one.step(1)
        many.step(2).step(4).step(7)
        traj = torch.empty((13, ny, nx), dtype=torch.float32, device="cuda")
        rec.record(6, traj).record(7, traj[6:])
        ref = _populations(one.save_state()[0], nx, ny, storage)
        assert torch.equal(_populations(many.save_state()[0], nx, ny, storage), ref)
        assert torch.equal(_populations(rec.save_state()[0], nx, ny, storage), ref)
        assert torch.equal(traj, torch.stack(phis))
        for s in (one, many, rec):
            s.close()


@pytest.mark.parametrize("storage", [0, 1])
def test_loaded_state_steps_as_the_saved_one(storage):
    """The sum field kept beside the populations follows a loaded state, also into a batch
    and back, whatever stepped before."""
    import paper_1805_00007_amd as lbm
    rng = np.random.default_rng(7)
    nx, ny = 130, 90
    phi0 = np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1)
    field = (rng.uniform(-.04, .04, (ny, nx)), rng.uniform(-.04, .04, (ny, nx)))
    s = lbm.Solver(nx, ny, phi0, field=field, storage=storage, **workloads.PRESCRIBED)
    s.step(5)
    saved = s.save_state()
    ref = s.step(9).phi()
    for n in (1, 2, 7):
        s.step(n)
        s.load_state(*saved)
        assert torch.equal(s.step(4).step(5).phi(), ref), n
    if storage == 0:
        s.load_state(*saved)
        b = lbm.Batch([s])
        b.step(2)
        s.step(3)
        b.step(1)
        s.step(3)
        b.close()
        assert torch.equal(s.phi(), ref)
    s.close()


@pytest.mark.parametrize("nx,ny", [(5, 4), (58, 11), (59, 64), (130, 37)])
def test_walled_marches_against_the_oracle(nx, ny):
    """tau_g = 1 between walls (marches with mirrored rows and bounce-back), single steps and
    calls of several, with the recorded order parameter: bitwise alike, and the oracle's phi
    after 13 steps to 13 steps of ~150 float32 roundings (6e-8 each, at most 1e-6 a step in
    phi of order 1)."""
    import oracle
    import paper_1805_00007_amd as lbm
    rng = np.random.default_rng(nx + ny)
    phi0 = np.float32(np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1))
    U, V = (np.float32(rng.uniform(-.04, .04, (ny, nx))) for _ in range(2))
    for model in (1, 2):
        phys = dict(workloads.PRESCRIBED, model=model)
        one, many = (lbm.Solver(nx, ny, phi0, field=(U, V), walls=1, **phys) for _ in range(2))
        phis = []
        for _ in range(13):
            phis.append(one.phi())
            one.step(1)
        traj = torch.empty((6, ny, nx), dtype=torch.float32, device="cuda")
        many.step(5).record(6, traj).step(2)
        assert torch.equal(traj, torch.stack(phis[5:11]))
        assert torch.equal(one.phi(), many.phi())
        p = oracle.Params(nx=nx, ny=ny, walls=1, **phys)
        ref = oracle.State(p, phi0.astype(np.float64), U.astype(np.float64),
                           V.astype(np.float64)).run(13).phi
        assert np.abs(one.phi().double().cpu().numpy() - ref).max() <= 1.3e-5
        one.close()
        many.close()


def test_batch_marches_equal_single_steps():
    """A batch call of several steps marches its tau_g = 1 lattices in launches of their own
    (here one per kernel variant, more than 64 lattices in one of them) and leaves bitwise
    the state of single steps, whatever the parity and with lattices at other tau_g beside."""
    import paper_1805_00007_amd as lbm
    rng = np.random.default_rng(3)
    pairs = []
    for i in range(74):
        nx, ny = int(rng.integers(20, 130)), int(rng.integers(4, 90))
        phi0 = np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1)
        field = (rng.uniform(-.04, .04, (ny, nx)), rng.uniform(-.04, .04, (ny, nx)))
        phys = dict(workloads.PRESCRIBED, model=1 if i % 25 == 3 else 2,
                    tau_g=0.9 if i % 25 == 7 else 1.0)
        pairs.append([lbm.Solver(nx, ny, phi0, field=field, **phys) for _ in range(2)])
    b = lbm.Batch([p[0] for p in pairs])
    for n, graph in ((3, False), (1, False), (4, True), (2, False), (5, True)):
        b.step(n, graph=graph)
        for _, one in pairs:
            for _ in range(n):
                one.step(1)
        for got, one in pairs:
            a, r = (_populations(s.save_state()[0], s.nx, s.ny, 0) for s in (got, one))
            assert torch.equal(a, r), (n, graph, got.nx, got.ny)
    b.close()
    for p in pairs:
        for s in p:
            s.close()


@pytest.mark.parametrize("storage,model", [(0, 1), (0, 2), (0, 3), (1, 1), (1, 2), (2, 2)])
@pytest.mark.parametrize("nx,ny", [(180, 170), (181, 197), (59, 700), (8000, 4)])
def test_population_march_equals_tiles(nx, ny, storage, model):
    """The population step at tau_g != 1 as a march in registers (the default at these
    sizes) leaves bitwise the state of the tiles, with and without walls, for separable
    and stored velocities."""
    import paper_1805_00007_amd as lbm
    rng = np.random.default_rng(nx + ny)
    phi0 = np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1)
    tables = dict(ax=rng.uniform(-.04, .04, nx), ay=rng.uniform(-1, 1, ny),
                  bx=rng.uniform(-.04, .04, nx), by=rng.uniform(-1, 1, ny),
                  tf=np.cos(0.1 * np.arange(20)))
    field = (rng.uniform(-.04, .04, (ny, nx)), rng.uniform(-.04, .04, (ny, nx)))
    for walls, vel, tau in ((0, dict(velocity=tables), 0.8), (1, dict(velocity=tables), 1.3),
                            (0, dict(field=field), 1.3), (1, dict(field=field), 0.8)):
        print(nx, ny, storage, model, walls, list(vel), flush=True)
        got = []
        for tiles in (None, (64, 8)):
            s = lbm.Solver(nx, ny, phi0, storage=storage, walls=walls, **vel,
                           **dict(workloads.PRESCRIBED, model=model, tau_g=tau))
            if tiles:
                s.set_tiles(*tiles)
            s.step(6)
            got.append(s.save_state()[0])
            s.close()
        size = ny * 20 * ((nx + 31) // 32 * 32) if storage else ny * 36 * ((nx + 31) // 32 * 32)
        a, b = (_populations(x[:size], nx, ny, storage) for x in got)
        assert torch.equal(a, b)
        assert torch.equal(got[0][size:], got[1][size:])  # model 3: its history
