"""GPU parity of the alternative pre-encoder signals (Table 5's low-res frame
difference and dHash, in the readings of the oracle) through the C ABI: the
signal rows bit-identical to the oracle's on ragged, unaligned, gray and
workload-sized frames, and the whole keep rule on them (calibrated
thresholds, scores, masks, kept counts) bit-identical to the oracle's
selection over the oracle's rows."""
import numpy as np
import pytest

import oracle
from paper_2609_03675_amd import binding as B
from paper_2609_03675_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import require_gpu, to_dev  # noqa: E402

KINDS = {"framediff": (B.FRAMEDIFF, oracle.FRAMEDIFF), "dhash": (B.DHASH, oracle.DHASH)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()
    B.lib()


def gpu_rows(frames_d, kind, G):
    n, H, W = frames_d.shape[:3]
    C = frames_d.shape[3] if frames_d.dim() == 4 else 1
    nsig = B.cofie_ngff_nbins(kind, G)
    out = torch.empty((n, nsig), dtype=torch.int32, device="cuda")
    B.cofie_ngff_histogram(frames_d, G, kind, out=out)
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("name", ["framediff", "dhash"])
@pytest.mark.parametrize("shape,G", [((5, 33, 47, 3), 4),      # W not a multiple of 4: byte loads
                                     ((3, 64, 64, 1), 16),     # gray frames
                                     ((2, 90, 160, 3), 32),
                                     ((3, 37, 29, 3), 2),
                                     ((2, 64, 64, 3), 64),     # one pixel per cell
                                     ((4, 448, 448, 3), 32),   # the workloads' frames
                                     ((2, 1080, 1920, 3), 32)])
def test_signal_rows_bit_exact(name, shape, G):
    kind, okind = KINDS[name]
    rng = np.random.default_rng([2609, 3675, 64, shape[1], G])
    f = rng.integers(0, 256, size=shape, dtype=np.uint8)
    print(f"signal {name} shape={shape} G={G}", flush=True)
    got = gpu_rows(to_dev(f), kind, G)
    assert np.array_equal(got, oracle.signature(f, okind, G))


@pytest.mark.parametrize("name,shape,G", [("framediff", (2, 9, 2, 3), 2),       # rows of fewer than 4 pixels
                                          ("framediff", (3, 5, 3, 1), 2),
                                          ("framediff", (2, 16, 4, 3), 4),      # one column group
                                          ("framediff", (2, 35, 5, 1), 4),      # a group that overlaps the one before
                                          ("framediff", (2, 530, 67, 3), 32),   # 17 rows a grid row: two slices, 9 and 8
                                          ("dhash", (1, 1031, 131, 3), 8),      # 9 slices a grid row, one frame
                                          ("framediff", (1100, 12, 18, 3), 4),  # more frames than four per CU
                                          ("dhash", (3, 8, 9, 3), 8)])          # one pixel per cell
@pytest.mark.parametrize("offset", [0, 3])
def test_signal_rows_task_edges(name, shape, G, offset):
    """The signature kernel's tasks at their edges: short rows, the row's last
    column group, row slices, workgroup splits, rows at any byte."""
    kind, okind = KINDS[name]
    rng = np.random.default_rng([2609, 3675, 66, shape[1], shape[2]])
    f = rng.integers(0, 256, size=shape, dtype=np.uint8)
    buf = torch.empty(f.nbytes + offset, dtype=torch.uint8, device="cuda")
    view = buf[offset:].view(shape)
    view.copy_(torch.from_numpy(f))
    print(f"signal {name} shape={shape} G={G} offset={offset}", flush=True)
    assert np.array_equal(gpu_rows(view, kind, G), oracle.signature(f, okind, G))


@pytest.mark.parametrize("name", ["framediff", "dhash"])
def test_signal_rows_unaligned_frames(name):
    """Frames starting at an odd byte address."""
    kind, okind = KINDS[name]
    rng = np.random.default_rng([2609, 3675, 65])
    f = rng.integers(0, 256, size=(3, 40, 48, 3), dtype=np.uint8)
    buf = torch.empty(f.nbytes + 1, dtype=torch.uint8, device="cuda")
    view = buf[1:].view(3, 40, 48, 3)
    view.copy_(torch.from_numpy(f))
    print(f"signal {name} unaligned", flush=True)
    assert np.array_equal(gpu_rows(view, kind, 8), oracle.signature(f, okind, 8))


@pytest.mark.parametrize("name", ["framediff", "dhash"])
@pytest.mark.parametrize("seg", [0, 100])
def test_keep_rule_on_signals(name, seg):
    """The 1 fps stream's first 200 frames (and two segments of 100): the
    thresholds calibrated for 40 % retention, then the filter, all equal to
    the oracle's selection over the oracle's signal rows."""
    kind, okind = KINDS[name]
    G = 32
    wl = synth.WORKLOADS[2]
    f = synth.frames(2, count=200)
    n = f.shape[0]
    rows = oracle.signature(f, okind, G)
    mass = oracle.signal_two_m(okind, G) // 2
    target = 40 if seg else 80
    theta, tau_o = oracle.ngff_calibrate(rows, mass, target, 30, 4, seg)
    fd = to_dev(f)
    rule0 = B.keep_rule(kind, 0.3, 30, 4, seg)
    print(f"keep rule {name} seg={seg}: oracle theta {theta.tolist()}", flush=True)
    tau_g = B.cofie_ngff_calibrate(fd, G, rule0, target)
    assert np.array_equal(tau_g.cpu().numpy().view(np.uint32), tau_o.view(np.uint32))
    nseg = 2 if seg else 1
    count = torch.empty(nseg, dtype=torch.int32, device="cuda")
    hist = torch.empty((n, B.cofie_ngff_nbins(kind, G)), dtype=torch.int32, device="cuda")
    rule = B.keep_rule(kind, 0.3, 30, 4, seg, tau_per_segment=tau_g, out_hist=hist, out_count=count)
    s, m = B.cofie_ngff_filter(fd, G, rule)
    torch.cuda.synchronize()
    so, mo, ko = oracle.ngff_select(rows, mass, tau_o, 30, 4, seg)
    assert np.array_equal(hist.cpu().numpy().view(np.uint32), rows)
    assert np.array_equal(m.cpu().numpy(), mo)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), so.view(np.uint32))
    assert np.array_equal(count.cpu().numpy(), ko.astype(np.int32))
    print(f"  kept {ko.tolist()}", flush=True)
