"""GPU parity of the rank 1, 2 and 4 kernels where their dispatch and their row ends change: row
lengths on both sides of every class (lanes per row, one or several waves, one or several column
blocks), lengths that are not a multiple of four, buckets whose tensors start off the 16-byte grid,
and rows longer than 5120 columns, whose P-step leaves the residual implied in the error arena."""

import numpy as np
import pytest
import torch

import synthgrad as sg
from paper_2306_08881_amd import _lib as L
from tests import parity_util as PU
from tests.test_gpu_powersgd import run_psgd_parity

pytestmark = pytest.mark.gpu

# columns: 63-66 (16 lanes per row or 32), 127-130, 255-258, 511-514 (narrow or not), 767-769 (three
# waves), 1023-1025, 3072-3073 and 4095-4097 (eight waves), 5119-5121 (one block or several), then
# up to 17 column blocks; rows around the 8-row rounds, the 64-row tiles and the 256-row chunks
COLS = [(9, 63), (70, 66), (33, 127), (130, 130), (41, 255), (257, 257), (65, 511), (66, 513), (5, 3), (63, 767),
        (20, 769), (7,), (300, 1023), (40, 1025), (17, 3072), (13, 3073), (12, 4095), (11, 4097), (3,), (10, 5119),
        (9, 5120), (67, 5121), (1,), (520, 5123), (8, 8192), (16, 17001)]


@pytest.mark.parametrize("rank", [1, 2, 4])
@pytest.mark.parametrize("ef", [True, False])
def test_row_classes(rank, ef):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    params = [sg.Param(f"t{i}", s) for i, s in enumerate(COLS)]
    wl = sg.Workload("cols", params, rank, 5, lambda p: 0.05, seed=5, cap_bytes=1 << 20)
    for grouped in (False, True):
        rep = PU.run_parity(wl, "fresh", 5, range(1, 6), list(range(len(COLS))), ef=ef, free=3, grouped=grouped)
        assert not rep.failures, "\n".join(rep.failures[:20])


# the same classes with whole 16-byte words only, whose launches take the kernels without the ragged form
ALIGNED = [(9, 64), (70, 68), (33, 128), (41, 256), (65, 512), (66, 516), (5, 4), (63, 768), (20, 772), (8,),
           (300, 1024), (40, 1028), (40, 2052), (17, 3072), (13, 3076), (12, 4096), (11, 4100), (9, 5120), (67, 5124),
           (4,), (520, 5128), (16, 17004)]


@pytest.mark.parametrize("rank", [1, 2, 4])
@pytest.mark.parametrize("ef", [True, False])
def test_aligned_row_classes(rank, ef):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    params = [sg.Param(f"t{i}", s) for i, s in enumerate(ALIGNED)]
    wl = sg.Workload("cols", params, rank, 7, lambda p: 0.05, seed=5, cap_bytes=1 << 20)
    for grouped in (False, True):
        rep = PU.run_parity(wl, "fresh", 5, range(1, 6), list(range(len(ALIGNED))), ef=ef, free=3, grouped=grouped)
        assert not rep.failures, "\n".join(rep.failures[:20])


@pytest.mark.parametrize("rank", [1, 4])
def test_long_rows_resume_after_a_p_step(rank):
    """A state saved after an odd step (the long rows' arena holds X), and the same state with the
    error written out (as a library without that form saves it), both continue like the run."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    shapes = [(70, 6001), (33,), (40, 300)]
    rng = np.random.default_rng(3)
    a = PU.Runner(shapes, rank)
    sets = [{i: (0.05 * rng.standard_normal(s)).astype(np.float32) for i, s in enumerate(shapes)} for _ in range(5)]
    for t in (1, 2, 3):
        a.step(t, a.pack(sets[t - 1]))
    blob = bytearray(a.acp.get_state())
    a.acp.error(0, a.ebuf[0])
    torch.cuda.synchronize()
    version = slice(8, 16)  # after the magic number
    assert blob[version] == np.int64(2).tobytes()  # a library without the form has to refuse it
    explicit = bytearray(blob)
    explicit[version] = np.int64(1).tobytes()
    head = 96 + 8  # the record of the only bucket: step, then the arena's form
    assert np.frombuffer(blob, np.int64, 2, 96).tolist() == [3, 2]
    explicit[head:head + 8] = np.int64(0).tobytes()
    e = a.ebuf[0].cpu().numpy()
    n = shapes[2][0] * shapes[2][1]  # backward order: the third tensor first, then the vector
    for off, k in ((0, n), (n + 33, 70 * 6001)):
        at = 96 + 16 + 4 * off
        explicit[at:at + 4 * k] = e[off:off + k].tobytes()
    b, c = PU.Runner(shapes, rank), PU.Runner(shapes, rank)
    unknown = bytearray(blob)
    unknown[version] = np.int64(3).tobytes()
    with pytest.raises(L.AcpError):
        b.acp.set_state(bytes(unknown))
    b.acp.set_state(bytes(blob))
    c.acp.set_state(bytes(explicit))
    for t in (4, 5):
        g = a.pack(sets[t - 1])
        for run in (a, b, c):
            run.step(t, g)
        torch.cuda.synchronize()
        assert torch.equal(a.fbuf[0], b.fbuf[0]) and torch.equal(a.out[0], b.out[0]), t
        # the residual's term is rounded once more when it is written out: a few fp32 roundings
        assert PU.rel_err(c.out[0].cpu().numpy(), a.out[0].cpu().numpy()) < 1e-5, t
        if t == 4:  # after an even step every matrix has the form version 1 knows
            assert bytes(a.acp.get_state())[version] == np.int64(1).tobytes()


@pytest.mark.parametrize("rank", [1, 2, 4, 8])
@pytest.mark.parametrize("ef", [True, False])
def test_powersgd_row_classes(rank, ef):
    """Power-SGD's first half runs in the P-step kernels: P = M' Q with Q as it is, M' kept."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    shapes = [s for s in COLS if len(s) == 1 or min(s) > rank]
    params = [sg.Param(f"t{i}", s) for i, s in enumerate(shapes)]
    wl = sg.Workload("cols", params, rank, 4, lambda p: 0.05, seed=6, cap_bytes=1 << 20)
    rep = run_psgd_parity(wl, 4, list(range(len(shapes))), ef=ef, free=2)
    assert not rep.failures, "\n".join(rep.failures[:20])
