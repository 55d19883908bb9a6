"""Every launch that serves a prescribed flow against another one that serves the same call:
tiles of every width and the register march at tau_g != 1, recording steps, the schedules
and tiles of a batch, and the populations that the launches at tau_g = 1 store beside the
sums that later calls read.  All bitwise."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lattice(nx, ny, seed=0):
    rng = np.random.default_rng(nx * 1000 + ny + seed)
    phi0 = np.clip(0.3 + 0.2 * rng.normal(size=(ny, nx)), -1, 1)
    tables = dict(ax=rng.uniform(-.04, .04, nx), ay=rng.uniform(-1, 1, ny),
                  bx=rng.uniform(-.04, .04, nx), by=rng.uniform(-1, 1, ny))
    field = (rng.uniform(-.04, .04, (ny, nx)), rng.uniform(-.04, .04, (ny, nx)))
    return phi0, (dict(velocity=tables), dict(field=field))


def _solver(nx, ny, phi0, vel, **phys):
    import paper_1805_00007_amd as lbm
    return lbm.Solver(nx, ny, phi0, **vel, **dict(workloads.PRESCRIBED, **phys))


def _state(s):
    """The saved state without the padding of its rows."""
    buf, _ = s.save_state()
    nx, ny, pitch = s.nx, s.ny, (s.nx + 31) // 32 * 32
    if s.params.storage == 0:
        n = ny * 36 * pitch
        parts = [buf[:n].view(ny, 9, pitch, 4)[:, :, :nx]]
    else:
        n = ny * 20 * pitch
        rows = buf[:n].view(ny, 20 * pitch)
        parts = [rows[:, :4 * pitch].reshape(ny, pitch, 4)[:, :nx],
                 rows[:, 4 * pitch:].reshape(ny, 8, pitch, 2)[:, :, :nx]]
    return torch.cat([p.reshape(-1) for p in parts] + [buf[n:]])


# by default all march; 1100 = 2 x 512 + 76
@pytest.mark.parametrize("nx,ny", [(5, 4), (61, 7), (131, 45), (181, 197), (1100, 37)])
@pytest.mark.parametrize("storage,model", [(0, 1), (0, 2), (0, 3), (1, 2), (2, 1)])
def test_tile_shapes_at_other_tau(nx, ny, storage, model):
    phi0, vels = _lattice(nx, ny)
    for walls, vel, tau in ((0, vels[0], 0.8), (1, vels[0], 1.3), (0, vels[1], 1.3), (1, vels[1], 0.8)):
        ref = None
        for tiles in (None, (64, 1), (64, 5), (128, 16), (256, 3), (256, 32), (512, 8), (512, 1)):
            s = _solver(nx, ny, phi0, vel, storage=storage, model=model, walls=walls, tau_g=tau)
            if tiles:
                s.set_tiles(*tiles)
            got = _state(s.step(6))
            s.close()
            ref = got if ref is None else ref
            assert torch.equal(got, ref), (walls, list(vel), tiles)


@pytest.mark.parametrize("nx,ny", [(131, 45), (181, 197), (1100, 37)])
@pytest.mark.parametrize("storage,model,walls", [(0, 1, 0), (0, 2, 0), (0, 3, 0), (0, 2, 1), (1, 2, 0)])
def test_record_at_other_tau(nx, ny, storage, model, walls):
    """Recorded steps leave the state of plain ones and the phi before each: the fused
    recording tiles of periodic float32 lattices with models 1 and 2, and the others."""
    phi0, vels = _lattice(nx, ny)
    for vel in vels:
        phys = dict(storage=storage, model=model, walls=walls, tau_g=0.8)
        one = _solver(nx, ny, phi0, vel, **phys)
        phis = []
        for _ in range(7):
            phis.append(one.phi())
            one.step(1)
        ref = _state(one)
        one.close()
        for tiles in (None, (64, 4), (128, 5), (256, 2), (512, 8)):
            s = _solver(nx, ny, phi0, vel, **phys)
            if tiles:
                s.set_tiles(*tiles)
            traj = torch.empty((7, ny, nx), dtype=torch.float32, device="cuda")
            s.record(3, traj).record(4, traj[3:])
            assert torch.equal(traj, torch.stack(phis)), (list(vel), tiles)
            assert torch.equal(_state(s), ref), (list(vel), tiles)
            s.close()


@pytest.mark.parametrize("tiles,graph,persistent", [
    ((0, 16), False, 0), ((0, 16), True, 1), ((64, 4), True, 0), ((64, 4), True, 1),
    ((256, 32), False, 1), ((128, 1), True, 0), ((128, 5), False, 1)])
def test_batch_at_other_tau(tiles, graph, persistent):
    """Tiles and schedules of a batch at tau_g != 1 against single steps of each lattice, which
    march."""
    import paper_1805_00007_amd as lbm
    sides = [(20, 9), (64, 64), (131, 45), (181, 197), (257, 130), (600, 51), (1100, 37)]
    pairs = []
    for i, (nx, ny) in enumerate(sides * 2):
        phi0, vels = _lattice(nx, ny, i)
        pairs.append([_solver(nx, ny, phi0, vels[i % 2], model=1 if i % 3 == 0 else 2,
                              tau_g=1.0 if i == 5 else 0.8) for _ in range(2)])
    b = lbm.Batch([p[0] for p in pairs]).set_tiles(*tiles).set_schedule(persistent)
    for n in (3, 2):
        b.step(n, graph=graph)
    for got, one in pairs:
        for _ in range(5):
            one.step(1)
        assert torch.equal(_state(got), _state(one)), (got.nx, got.ny)
    b.close()
    for p in pairs:
        for s in p:
            s.close()


def _stored_populations_hold_the_state(s, n):
    """After n steps: phi and a later step from the sums that the launches kept, and again
    from the sums of the populations that they stored (a loaded state is summed anew)."""
    s.step(n)
    phi = s.phi()
    saved = s.save_state()
    after = s.step(1).phi()
    s.load_state(*saved)
    assert torch.equal(s.phi(), phi), (s.nx, s.ny, n)
    assert torch.equal(s.step(1).phi(), after), (s.nx, s.ny, n)


# small: regions, 16 and 32 rows; the others march
@pytest.mark.parametrize("nx,ny", [(40, 23), (130, 90), (300, 260), (59, 1400), (701, 640)])
@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("walls", [0, 1])
def test_stored_populations_at_tau_one(nx, ny, storage, walls):
    phi0, vels = _lattice(nx, ny)
    for model, vel in ((1, vels[0]), (2, vels[0]), (2, vels[1])):
        s = _solver(nx, ny, phi0, vel, storage=storage, model=model, walls=walls)
        for n in (1, 2, 5):
            _stored_populations_hold_the_state(s, n)
        s.close()


@pytest.mark.parametrize("storage", [0, 1])
def test_stored_populations_at_the_largest_size(storage):
    """Population offsets near 2^31 bytes, written and read."""
    p = 80
    phi0, vels = _lattice(p, p)
    reps = (7760 // p, 7680 // p)
    field = tuple(torch.tensor(f, dtype=torch.float32, device="cuda").repeat(reps) for f in vels[1]["field"])
    s = _solver(7680, 7760, torch.tensor(phi0, dtype=torch.float32, device="cuda").repeat(reps),
                dict(field=field), storage=storage)
    _stored_populations_hold_the_state(s, 3)
    s.close()


@pytest.mark.parametrize("nx,ny", [(4, 5), (5, 4), (31, 9), (32, 8), (33, 40), (250, 7), (257, 129), (8, 600)])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_loaded_state_is_the_saved_one(nx, ny, storage):
    """A state loaded by the kernel that copies and sums, and from an odd address (a copy and
    a pass over it): every byte of the populations, padding included, and bitwise the phi
    and the steps of the state that was saved."""
    phi0, vels = _lattice(nx, ny)
    for walls in (0, 1):
        s = _solver(nx, ny, phi0, vels[0], storage=storage, walls=walls)
        buf, n = s.step(3).save_state()
        pad = torch.randint(0, 256, buf.shape, dtype=torch.uint8, device="cuda")
        body = torch.zeros_like(buf, dtype=torch.bool)
        pitch = (nx + 31) // 32 * 32
        if storage == 0:
            body.view(ny, 9, pitch, 4)[:, :, :nx] = True
        else:
            body.view(ny, 20 * pitch)[:, :4 * nx] = True
            body.view(ny, 20 * pitch)[:, 4 * pitch:].view(ny, 8, pitch, 2)[:, :, :nx] = True
        buf = torch.where(body, buf, pad)
        phi = s.phi()
        after = s.step(4).phi()
        odd = torch.empty(buf.numel() + 1, dtype=torch.uint8, device="cuda")[1:]
        odd.copy_(buf)
        for src in (buf, odd):
            s.load_state(src, n)
            assert torch.equal(s.save_state()[0], buf), walls
            assert torch.equal(s.phi(), phi), walls
            assert torch.equal(s.step(4).phi(), after), walls
        s.close()


@pytest.mark.parametrize("nx,ny", [(2048, 2048), (2111, 1999), (48 * 44, 2003), (4096, 4096), (4200, 4100)])
@pytest.mark.parametrize("walls", [0, 1])
def test_writing_march_of_large_lattices(nx, ny, walls):
    """Float32 lattices whose last march of a call stores the populations past the caches, in
    strips of 48 columns (up to 2^24 nodes), and one size beyond: the state stored, the phi
    recorded, and the sums kept are those of launches in 58-column strips (the same steps as
    the first of a longer call) and of the populations."""
    phi0, vels = _lattice(nx, ny)
    for model, vel in ((2, vels[0]), (1, vels[1])):
        s = _solver(nx, ny, phi0, vel, model=model, walls=walls)
        _stored_populations_hold_the_state(s, 1)
        saved = s.save_state()
        traj = torch.empty((3, ny, nx), dtype=torch.float32, device="cuda")
        s.record(3, traj)  # 58-column strips for the first two
        end = s.phi()
        s.load_state(*saved)
        for k in range(3):
            one = torch.empty((1, ny, nx), dtype=torch.float32, device="cuda")
            s.record(1, one)
            assert torch.equal(one[0], traj[k]), (model, k)
        assert torch.equal(s.phi(), end), model
        s.close()


@pytest.mark.parametrize("storage", [0, 1])
def test_load_and_steps_under_capture(storage):
    """A captured load and an even number of steps replay from the loaded state, whatever ran
    before."""
    phi0, vels = _lattice(257, 129)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = _solver(257, 129, phi0, vels[0], storage=storage)
        buf, n = s.step(2).save_state()
        want = s.step(4).phi()
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        s.load_state(buf, n).step(4)
    for k in (2, 6, 4):
        with torch.cuda.stream(st):
            graph.replay()
            assert torch.equal(s.phi(), want), k
            s.step(k)
    s.close()


# at most 256 tiles of 64 x 16, and too large for marches of 3 rows
@pytest.mark.parametrize("nx,ny", [(505, 509), (64, 4096), (65, 2035), (4090, 63), (449, 430), (100, 2000)])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_single_step_tiles(nx, ny, storage):
    """The last step of a call in tiles: phi recorded, sums kept and populations stored are
    bitwise those of marches (the same steps as the first of a longer call)."""
    rng = np.random.default_rng(nx)
    phi0, vels = _lattice(nx, ny)
    vels[0]["velocity"]["tf"] = rng.uniform(0.5, 1, 9)
    for model, vel in ((1, vels[0]), (2, vels[0]), (1, vels[1]), (2, vels[1])):
        s = _solver(nx, ny, phi0, vel, storage=storage, model=model)
        saved = s.save_state()
        traj = torch.empty((5, ny, nx), dtype=torch.float32, device="cuda")
        s.record(5, traj)  # marches but for the last
        end, state = s.phi(), _state(s)
        s.load_state(*saved)
        one = torch.empty((5, ny, nx), dtype=torch.float32, device="cuda")
        for k in range(5):
            s.record(1, one[k:k + 1])
        assert torch.equal(one, traj), (model, list(vel))
        assert torch.equal(s.phi(), end) and torch.equal(_state(s), state), (model, list(vel))
        _stored_populations_hold_the_state(s, 1)
        s.close()
