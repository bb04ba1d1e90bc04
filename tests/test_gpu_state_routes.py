"""Export and import of the raw state: a thread per record on small grids, a thread per cell from 65536 cells on.  Sizes
on both sides of the line, and of the smallest grids; values that every storage form holds exactly (multiples of 1/8
below 256: at most 11 bits), so the state comes back equal, in every array and in each layout's order."""
import numpy as np
import pytest

from paper_1508_03452_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("b_prev", [0, 1])
@pytest.mark.parametrize("shape", [(1, 1, 1), (65, 1, 1), (17, 5, 3), (257, 255, 1), (256, 256, 1), (33, 2, 1000)])
def test_state_comes_back_as_it_went_in(storage, b_prev, shape):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_03452_amd.rmhdlb import Solver
    print(f"[routes] {storage} {shape} b_prev {b_prev}", flush=True)
    for bc in (W.PERIODIC3, (("periodic",) * 2, ("periodic",) * 2, ("driven", "open"))):   # without and with ghost planes
        s = Solver(shape, bc, storage=storage, b_prev=b_prev)
        n = shape[0] * shape[1] * shape[2]
        arrays = s.state_len() // n
        assert arrays == (69 if b_prev else 66)
        rng = np.random.default_rng(3)
        raw = rng.integers(-2047, 2048, size=(arrays,) + shape[::-1]).astype(np.float64) / 8.0
        s.set_state(torch.from_numpy(raw).cuda())
        assert np.array_equal(s.get_state().cpu().numpy(), raw)
