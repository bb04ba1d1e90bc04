"""Launch shapes of the kernels with more than one plane, bit for bit: the arithmetic of a cell does not depend on the
tile, so every shape, and every batch, gives the same state in every storage form."""
import numpy as np
import pytest

from paper_1508_03452_amd import workloads as W

from .parity_util import run_gpu

pytestmark = pytest.mark.gpu
STORAGES = ["f64", "f32", "f16"]
PER, OPEN = ("periodic", "periodic"), ("open", "open")
# the tuner's shared walks (px, zb, zg), one that divides neither the planes nor the tile's two, and plain walks;
# 67 planes: every zg stays as given, the last chunk and (FP64, FP32) the last tile are ragged
SHAPES = [(32, 8, 2), (32, 8, 4), (32, 8, 8), (64, 4, 2), (64, 4, 4), (64, 8, 2), (64, 16, 4), (64, 3, 2), (16, 5, 3),
          (64, 1, 1), (32, 1, 1), (64, 67, 1)]


def _torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _state(s):
    return s.get_state().cpu().numpy()


def _box(shape=(70, 13, 67), **kw):
    return W.random_state(shape=shape, seed=6, vmax=0.1, Bmag=0.2, Emag=0.02, sigma=3.0, bc=(OPEN, PER, OPEN), **kw)


@pytest.mark.parametrize("storage", STORAGES)
def test_shared_walks_give_identical_states(storage):
    _torch_cuda()
    w = _box()
    ref = run_gpu(w, 3, storage=storage)
    want = _state(ref)
    assert np.isfinite(want).all()
    s = run_gpu(w, 0, storage=storage)
    for shape in SHAPES:
        print(f"[tiles] {storage} {shape}", flush=True)
        s.init_fields(w.fields)
        s.set_tuning(*shape)
        s.step(3)
        assert np.array_equal(want, _state(s)), shape


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("kw", [dict(collision=1), dict(flux=1), dict(collision=1, flux=1), dict(b_prev=1)])
def test_shared_walks_of_the_other_readings(storage, kw):
    _torch_cuda()
    print(f"[tiles] {storage} {kw}", flush=True)
    w = _box((70, 13, 19), **kw)
    want = _state(run_gpu(w, 3, storage=storage))
    assert np.isfinite(want).all()
    s = run_gpu(w, 0, storage=storage)
    for shape in [(64, 4, 2), (64, 3, 2), (64, 1, 1), (64, 19, 1)]:
        s.init_fields(w.fields)
        s.set_tuning(*shape)
        s.step(3)
        assert np.array_equal(want, _state(s)), shape


@pytest.mark.parametrize("storage", STORAGES)
def test_shared_walks_with_the_learned_guess(storage):
    """The network on a box with an odd number of planes: every lane stays, those without a cell compute a copy of the
    edge cell.  The shapes agree bit for bit, and with the plain recovery within the forms' parity bounds (1e-12, 5e-5
    and 5e-3 of each state array's scale): the root is the same."""
    _torch_cuda()
    w = W.random_state(shape=(70, 13, 17), seed=31, vmax=0.8, modes=1, Bmag=0.1, Emag=0.01, sigma=10.0, tau=3.0)
    s = run_gpu(w, 0, storage=storage)
    s.train_guess(W.mlp_init(11), n_samples=8192, iters=200)
    s.set_guess(True)
    states = []
    for shape in [(64, 4, 1), (64, 4, 2), (64, 3, 2), (64, 1, 1)]:
        print(f"[tiles] guess {storage} {shape}", flush=True)
        s.init_fields(w.fields)
        s.set_tuning(*shape)
        s.step(3)
        states.append(_state(s))
        assert np.array_equal(states[0], states[-1]), shape
    assert s.moments(fields=())["diag"]["guess_steps"] == 3
    plain = _state(run_gpu(w, 3, storage=storage))
    scale = np.maximum(np.abs(plain).reshape(plain.shape[0], -1).max(axis=1), 1e-2)
    gap = (np.abs(states[0] - plain).reshape(plain.shape[0], -1).max(axis=1) / scale).max()
    assert gap <= {"f64": 1e-12, "f32": 5e-5, "f16": 5e-3}[storage], gap


def _batch(ws, storage, stream):
    from paper_1508_03452_amd.rmhdlb import Batch
    b = Batch([(w.shape, w.bc, w.params) for w in ws], storage=storage, stream=stream)
    for w, s in zip(ws, b.instances):
        s.init_fields(w.fields)
    return b


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("kinds", ["slabs", "boxes", "mixed"])
def test_batches_match_instances_stepped_alone(storage, kinds):
    """Slabs whose fields have every component, boxes, and both: a slab beside a box takes the general kernels, alone
    those for a single plane, and its state is the same."""
    torch = _torch_cuda()
    print(f"[tiles] batch {kinds} {storage}", flush=True)
    ws = []
    if kinds != "boxes":
        ws += [_box((130, 9, 1)), W.random_state(shape=(63, 14, 1), seed=9, vmax=0.3, Bmag=0.2, Emag=0.05, sigma=3.0,
                                                 bc=(PER, OPEN, PER))]
    if kinds != "slabs":
        ws += [_box((70, 13, 9)), W.random_state(shape=(33, 20, 6), seed=8, vmax=0.2, Bmag=0.2, Emag=0.02, sigma=3.0)]
    want = [_state(run_gpu(w, 6, storage=storage)) for w in ws]
    for px, yw in ((64, 1), (32, 2)):
        b = _batch(ws, storage, torch.cuda.Stream())
        b.set_tuning(px, yw, 2)
        b.step(6)
        torch.cuda.synchronize()
        for w, s, r in zip(ws, b.instances, want):
            assert np.array_equal(_state(s), r), (w.shape, px, yw)
        b.close()


@pytest.mark.parametrize("storage", STORAGES)
def test_walks_of_one_plane_and_of_an_odd_number(storage):
    """One-plane walks, stacked groups and odd walks of the two-plane tiles, on boxes of 7 planes and on a single plane
    above a driven face (the general kernels with one plane)."""
    _torch_cuda()
    driven = W.flare(nx=70, ny=24, nz=1, Lz=6.0, sigma=1e3)
    for w in (_box((70, 29, 7)), driven):
        ref = run_gpu(w, 0, storage=storage)
        ref.set_tuning(64, 2, 1, 1)
        ref.step(3)
        want = _state(ref)
        assert np.isfinite(want).all()
        for shape in [(64, 1, 1, 4), (32, 1, 1, 4), (16, 1, 4, 2), (32, 3, 2, 1), (64, 7, 1, 8), (32, 5, 1, 2)]:
            print(f"[tiles] {storage} {w.shape} {shape}", flush=True)
            s = run_gpu(w, 0, storage=storage)
            s.set_tuning(*shape)
            s.step(3)
            assert np.array_equal(want, _state(s)), (w.shape, shape)


@pytest.mark.parametrize("storage,px", [("f32", 64), ("f64", 32)])
def test_walks_of_one_plane_leave_no_half_block_idle(storage, px):
    """With four groups stacked, a step of one-plane walks takes about as long as one of four-plane walks: with two
    planes to the tile there as well, half of every block found no rows and the step took 1.3 times as long (FP32 and
    FP64)."""
    torch = _torch_cuda()
    s = run_gpu(_box((128, 128, 128)), 2, storage=storage)
    ms = {}
    for zb, yw in ((1, 4), (4, 1)) * 2:
        s.set_tuning(px, zb, 1, yw)
        s.step(3)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(s.stream)
        s.step(20)
        b.record(s.stream)
        torch.cuda.synchronize()
        ms[zb] = min(ms.get(zb, 1e9), a.elapsed_time(b) / 20)
    print(f"[tiles] {storage} px {px}: one plane {ms[1]:.4f} ms, four {ms[4]:.4f}", flush=True)
    assert ms[1] <= 1.25 * ms[4], ms


def test_batch_tuner_times_each_kernel_family():
    """Slabs of the same sizes with and without a driven face run different kernels (general ones, and those for a
    single plane): each kind is timed, not given the other's cached shape.  A trial writes the buffer that the state is
    not in, so a batch that was timed has a changed workspace, and a cached one has not."""
    torch = _torch_cuda()
    slab = lambda: _box((67, 45, 1))
    driven = lambda: W.flare(nx=67, ny=45, nz=1, Lz=6.0, sigma=1e3)

    def timed(ws):
        b = _batch(ws, "f32", torch.cuda.Stream())
        torch.cuda.synchronize()
        before = [t.clone() for t in b.workspaces]
        b.autotune()
        torch.cuda.synchronize()
        changed = any(not torch.equal(x, t) for x, t in zip(before, b.workspaces))
        b.close()
        return changed

    assert timed([slab(), slab()])
    assert not timed([slab(), slab()])
    assert timed([driven(), driven()])
    assert timed([slab(), driven()])       # a slab beside a driven one takes the general kernels as well


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nz", [7, 8, 9])
def test_one_plane_walks_on_both_sides_of_the_line(storage, nz):
    """Around 256 blocks a walk of one plane takes tiles of one plane or of two: the state is the same on both sides
    (64-wide FP32 tiles of 64 x 4 cells: 32 per plane of 64 x 128; 32-wide FP64 ones likewise), in a batch as alone."""
    torch = _torch_cuda()
    w = _box((64, 128, nz))
    px = 64 if storage == "f32" else 32
    want = run_gpu(w, 0, storage=storage)
    want.set_tuning(64, 2, 1, 1)
    want.step(3)
    want = _state(want)
    s = run_gpu(w, 0, storage=storage)
    s.set_tuning(px, 1)
    s.step(3)
    assert np.array_equal(want, _state(s))
    b = _batch([w, w], storage, torch.cuda.Stream())
    b.set_tuning(px, 1, 2)
    for i in b.instances:
        i.set_tuning(px, 1)
    b.step(3)
    torch.cuda.synchronize()
    for i in b.instances:
        assert np.array_equal(want, _state(i))
    b.close()


@pytest.mark.parametrize("storage", STORAGES)
def test_persistent_batch_of_boxes_matches_graph_replays(storage):
    """Boxes in the persistent launch, whose wavefronts are not kept in step, against graph replays: the tile's planes
    come from the batch's table there as well.  The device is idle before the cooperative launch."""
    torch = _torch_cuda()
    print(f"[tiles] persistent boxes {storage}", flush=True)
    ws = [W.random_state(shape=sh, seed=8, vmax=0.1, Bmag=0.2, Emag=0.02, sigma=3.0)
          for sh in ((70, 13, 9), (33, 20, 6), (64, 48, 31))]
    states = []
    for persistent in (False, True):
        b = _batch(ws, storage, torch.cuda.Stream())
        b.set_persistent(persistent)
        torch.cuda.synchronize()
        b.step(5)
        torch.cuda.synchronize()
        states.append([_state(s) for s in b.instances])
        b.close()
    for g, p in zip(*states):
        assert np.array_equal(g, p)
