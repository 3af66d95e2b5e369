"""GPU parity of NGFF (Sec. 3.2) against the CPU oracle through the C ABI:
histogram counts, keep masks, scores, kept counts and calibrated thresholds
must be bit-identical."""
import zlib

import numpy as np
import pytest

import oracle
from paper_2609_03675_amd import binding as B
from paper_2609_03675_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import hist_np, require_gpu, to_dev  # noqa: E402

MODES = {"gray": oracle.GRAY, "per_channel": oracle.PER_CHANNEL, "joint3d": oracle.JOINT3D}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()
    B.lib()


def gpu_hist(frames, bins, mode):
    h = B.cofie_ngff_histogram(to_dev(frames), bins, mode)
    torch.cuda.synchronize()
    return hist_np(h)


# ---------------------------------------------------------------- histogram --

@pytest.mark.parametrize("shape", [(3, 64, 64, 3),     # whole 768-byte units only
                                   (2, 40, 40, 3),     # units + pixel tail
                                   (3, 37, 53, 3),     # frame bytes not a multiple of 4
                                   (5, 448, 448, 3),   # several workgroups per frame
                                   (1, 1, 1, 3)])
@pytest.mark.parametrize("mode,bins", [("per_channel", 32), ("per_channel", 16), ("per_channel", 64),
                                       ("per_channel", 2), ("joint3d", 8), ("joint3d", 4),
                                       ("joint3d", 16), ("gray", 32), ("gray", 256)])
def test_histogram_bit_exact(shape, mode, bins):
    print(f"hist shape={shape} mode={mode} bins={bins}", flush=True)
    f = synth.random_frames(zlib.crc32(repr((shape, mode, bins)).encode()) % 1000, *shape)
    assert np.array_equal(gpu_hist(f, bins, mode), oracle.histogram(f, bins, MODES[mode]))


@pytest.mark.parametrize("shape", [(4, 64, 64), (3, 37, 53), (2, 448, 448)])
@pytest.mark.parametrize("bins", [32, 256, 8])
def test_histogram_gray_single_channel(shape, bins):
    f = synth.random_frames(7, *shape, C=1)[..., 0]
    assert np.array_equal(gpu_hist(f, bins, "gray"), oracle.histogram(f, bins, oracle.GRAY))


@pytest.mark.parametrize("H,W", [(17, 53),    # just past one unit (a head of 3 pixels leaves one)
                                 (16, 16),    # one unit exactly: none when the frame may start at any byte
                                 (121, 135)])  # several batches of units, every alignment among the frames
@pytest.mark.parametrize("mode,bins", [("per_channel", 32), ("joint3d", 8), ("gray", 32), ("gray1", 32)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_histogram_frames_at_any_byte(H, W, mode, bins, offset):
    """Frames whose addresses take every remainder mod 4: the pixels before the
    first aligned one, the vector units and the tail together count each pixel
    once."""
    C = 1 if mode == "gray1" else 3
    mode = "gray" if mode == "gray1" else mode
    n = 5
    f = synth.random_frames(11 + offset, n, H, W, C=C)
    buf = torch.zeros(f.size + 8, dtype=torch.uint8, device="cuda")
    view = buf[offset:offset + f.size].view(f.shape)
    view.copy_(to_dev(f))
    got = hist_np(B.cofie_ngff_histogram(view if C == 3 else view[..., 0], bins, mode))
    assert np.array_equal(got, oracle.histogram(f if C == 3 else f[..., 0], bins, MODES[mode]))


def test_histogram_split_frames_past_one_per_cu():
    """A few more large frames than CUs with counters of 128 KiB: frames are
    split between workgroups, whose counts meet in zeroed rows."""
    f = synth.random_frames(5, 262, 479, 641)
    got = gpu_hist(f, 8, "joint3d")
    assert np.array_equal(got, oracle.histogram(f, 8, oracle.JOINT3D))


def test_histogram_extreme_values():
    """All-0 and all-255 frames, and every byte value, land in the edge bins."""
    f = np.zeros((3, 16, 48, 3), dtype=np.uint8)
    f[1] = 255
    f[2] = np.arange(16 * 48 * 3).reshape(16, 48, 3) % 256
    for mode, bins in [("per_channel", 32), ("joint3d", 8), ("gray", 32)]:
        assert np.array_equal(gpu_hist(f, bins, mode), oracle.histogram(f, bins, MODES[mode]))


@pytest.mark.parametrize("cfg", [1, 2])
def test_histogram_workloads(cfg):
    wl = synth.WORKLOADS[cfg]
    f = synth.frames(cfg)
    assert np.array_equal(gpu_hist(f, wl.bins, wl.hist_mode),
                          oracle.histogram(f, wl.bins, MODES[wl.hist_mode]))


def test_histogram_empty_batch():
    out = torch.zeros((1, 96), dtype=torch.int32, device="cuda")
    B.cofie_ngff_histogram(torch.zeros((0, 8, 8, 3), dtype=torch.uint8, device="cuda"), 32,
                           "per_channel", out=out)
    torch.cuda.synchronize()
    assert int(out.abs().sum()) == 0


def test_histogram_deterministic():
    f = to_dev(synth.frames(2, 0, 0, 16))
    a = hist_np(B.cofie_ngff_histogram(f, 32, "per_channel"))
    b = hist_np(B.cofie_ngff_histogram(f, 32, "per_channel"))
    assert np.array_equal(a, b)


# ------------------------------------------------------------------ filter --

def run_filter(frames, bins, mode, tau, L_max=30, M_min=4, seg_len=0, tau_per_segment=None):
    n = frames.shape[0]
    nseg = 1 if seg_len <= 0 else (n + seg_len - 1) // seg_len
    fd = to_dev(frames)
    nb = B.cofie_ngff_nbins(mode, bins)
    hist = torch.empty((n, nb), dtype=torch.int32, device="cuda")
    count = torch.empty(nseg, dtype=torch.int32, device="cuda")
    tps = to_dev(np.asarray(tau_per_segment, dtype=np.float32)) if tau_per_segment is not None else None
    rule = B.keep_rule(mode, tau, L_max, M_min, seg_len, tau_per_segment=tps, out_hist=hist,
                       out_count=count)
    s, m = B.cofie_ngff_filter(fd, bins, rule)
    torch.cuda.synchronize()
    return s.cpu().numpy(), m.cpu().numpy(), hist_np(hist), count.cpu().numpy()


def oracle_filter(frames, bins, mode, tau, L_max=30, M_min=4, seg_len=0):
    h = oracle.histogram(frames, bins, MODES[mode])
    H, W = frames.shape[1:3]
    M = oracle.mass(MODES[mode], H, W)
    s, m, k = oracle.ngff_select(h, M, tau, L_max, M_min, seg_len)
    return s, m, h, k


def assert_filter_equal(g, o):
    s, m, h, c = g
    so, mo, ho, ko = o
    assert np.array_equal(h, ho), "histograms differ"
    assert np.array_equal(m, mo), f"masks differ at {np.flatnonzero(m != mo)[:10]}"
    assert np.array_equal(s.view(np.uint32), so.view(np.uint32)), \
        f"scores differ at {np.flatnonzero(s != so)[:10]}"
    assert np.array_equal(c, ko.astype(np.int32))


@pytest.mark.parametrize("cfg", [1, 2])
def test_filter_workload_calibrated(cfg):
    """Workload streams with the retention threshold the oracle calibrates."""
    wl = synth.WORKLOADS[cfg]
    f = synth.frames(cfg)
    h = oracle.histogram(f, wl.bins, MODES[wl.hist_mode])
    M = oracle.mass(MODES[wl.hist_mode], wl.H, wl.W)
    theta, tau = oracle.ngff_calibrate(h, M, wl.target, 30, 4)
    g = run_filter(f, wl.bins, wl.hist_mode, float(tau[0]))
    o = oracle_filter(f, wl.bins, wl.hist_mode, tau[0])
    assert_filter_equal(g, o)
    assert g[3][0] <= wl.target


@pytest.mark.parametrize("tau", [0.0, 0.05, 0.3, 0.9, 1.5, -1.0])
@pytest.mark.parametrize("L_max,M_min", [(30, 4), (1, 4), (7, 0), (0, 4), (0, 0), (200, 50)])
def test_filter_rule_edges(tau, L_max, M_min):
    f = synth.random_frames(21, 70, 12, 16, scenes=9)
    assert_filter_equal(run_filter(f, 16, "per_channel", tau, L_max, M_min),
                        oracle_filter(f, 16, "per_channel", np.float32(tau), L_max, M_min))


@pytest.mark.parametrize("T", [1, 2, 3])
def test_filter_short_streams(T):
    f = synth.random_frames(22, T, 8, 8)
    assert_filter_equal(run_filter(f, 32, "per_channel", 0.3),
                        oracle_filter(f, 32, "per_channel", np.float32(0.3)))


def test_filter_static_and_alternating():
    static = np.full((100, 8, 8, 3), 77, dtype=np.uint8)
    g = run_filter(static, 32, "gray", 0.3)
    assert np.flatnonzero(g[1]).tolist() == [0, 30, 60, 90, 99]
    assert_filter_equal(g, oracle_filter(static, 32, "gray", np.float32(0.3)))
    alt = np.zeros((20, 8, 8, 3), dtype=np.uint8)
    alt[1::2] = 255
    g = run_filter(alt, 32, "per_channel", 1.0)
    assert g[1].all()


@pytest.mark.parametrize("seg_len,n", [(40, 160), (40, 150), (512, 1100)])
def test_filter_segments_per_stream_tau(seg_len, n):
    f = synth.random_frames(23, n, 6, 10, scenes=12)
    nseg = (n + seg_len - 1) // seg_len
    taus = np.linspace(0.05, 0.6, nseg).astype(np.float32)
    g = run_filter(f, 16, "per_channel", 0.3, L_max=9, M_min=3, seg_len=seg_len, tau_per_segment=taus)
    o = oracle_filter(f, 16, "per_channel", taus, L_max=9, M_min=3, seg_len=seg_len)
    assert_filter_equal(g, o)


@pytest.mark.parametrize("mode,bins", [("joint3d", 8), ("gray", 32), ("per_channel", 32)])
def test_filter_modes(mode, bins):
    f = synth.random_frames(24, 50, 30, 20, scenes=7)
    assert_filter_equal(run_filter(f, bins, mode, 0.2, L_max=12),
                        oracle_filter(f, bins, mode, np.float32(0.2), L_max=12))


def test_filter_long_segment_global_scratch_path():
    """A stream too long for the select kernel's LDS copy (next[] in global memory)."""
    f = synth.random_frames(25, 24000, 2, 2, scenes=60)
    assert_filter_equal(run_filter(f, 8, "per_channel", 0.4, L_max=5),
                        oracle_filter(f, 8, "per_channel", np.float32(0.4), L_max=5))


@pytest.mark.parametrize("n,seg_len,L_max,mode,bins", [
    (2100, 1, 30, "per_channel", 16),   # several one-frame streams per workgroup
    (2100, 3, 9, "per_channel", 16),    # streams straddling workgroups
    (2100, 7, 30, "gray", 32),
    (9000, 0, 31, "per_channel", 8),    # three selection chunks, the widest keep word
    (3000, 0, 45, "per_channel", 8),    # L_max > 31: separate kernels
    (600, 0, 33, "per_channel", 16),
    (300, 0, 16, "joint3d", 4),
    (300, 0, 30, "joint3d", 16),        # 4096 bins: rows too wide to stage, separate kernels
])
def test_filter_band_keep_geometry(n, seg_len, L_max, mode, bins):
    """The band/keep-word kernel and the selection across their launch shapes:
    several frames and several streams per workgroup, selection chunks, and
    the separate-kernel path for L_max > 31 or histograms too wide for LDS."""
    f = synth.random_frames(26, n, 6, 10, scenes=n // 9)
    print(f"filter n={n} seg_len={seg_len} L_max={L_max} {mode} {bins}", flush=True)
    assert_filter_equal(run_filter(f, bins, mode, 0.25, L_max=L_max, M_min=4, seg_len=seg_len),
                        oracle_filter(f, bins, mode, np.float32(0.25), L_max=L_max, M_min=4,
                                      seg_len=seg_len))


@pytest.mark.parametrize("n,seg_len,L_max,mode,bins", [
    (1, 0, 30, "gray", 256),       # one frame: no lag inside the stream
    (41, 0, 31, "gray", 256),      # 256 bins, the longest keep word, a grid past the frames
    (67, 20, 1, "gray", 256),      # one lag, segments
    (90, 33, 4, "joint3d", 8),     # 512 bins, one lag a wave
    (64, 0, 17, "joint3d", 16),    # 4096 bins: several passes over a row
    (50, 7, 30, "joint3d", 16)])   # streams shorter than L_max
def test_filter_wide_rows(n, seg_len, L_max, mode, bins):
    """Rows of whole 1 KiB loads take the keep kernel without LDS staging."""
    f = synth.random_frames(n + L_max, n, 24, 40, scenes=9)
    for tau in (0.05, 0.4):
        s, m, h, k = run_filter(f, bins, mode, tau, L_max, 4, seg_len)
        so, mo, ho, ko = oracle_filter(f, bins, mode, tau, L_max, 4, seg_len)
        assert np.array_equal(h, ho) and np.array_equal(m, mo) and np.array_equal(k, ko)
        assert np.array_equal(s.view(np.uint32), so.view(np.uint32))


@pytest.mark.parametrize("seg_len,L_max", [(0, 30), (100, 9), (0, 45), (0, 0)])
def test_filter_from_histograms(seg_len, L_max):
    """cofie_ngff_filter_hist on cofie_ngff_histogram's counts, run on another
    stream, equals cofie_ngff_filter bit for bit (and the oracle)."""
    f = synth.random_frames(28, 700, 12, 16, scenes=60)
    fd = to_dev(f)
    nseg = 1 if seg_len == 0 else (700 + seg_len - 1) // seg_len
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        h = B.cofie_ngff_histogram(fd, 16, "per_channel")
        count = torch.empty(nseg, dtype=torch.int32, device="cuda")
        s2, m2 = B.cofie_ngff_filter_hist(h, 12, 16, 3, 16, B.keep_rule("per_channel", 0.25, L_max, 4, seg_len,
                                                                       out_count=count))
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = (s2.cpu().numpy(), m2.cpu().numpy(), hist_np(h), count.cpu().numpy())
    assert_filter_equal(g, oracle_filter(f, 16, "per_channel", np.float32(0.25), L_max, 4, seg_len))
    s1, m1 = B.cofie_ngff_filter(fd, 16, B.keep_rule("per_channel", 0.25, L_max, 4, seg_len))
    torch.cuda.synchronize()
    assert torch.equal(s1, s2) and torch.equal(m1, m2)


def test_filter_poisoned_workspace():
    """Tables in a reused workspace start from whatever the previous call (or
    nothing) left there: fill it with 0xFF, then call twice."""
    f = synth.random_frames(27, 700, 6, 10, scenes=60)
    fd = to_dev(f)
    nb = B.cofie_ngff_nbins("per_channel", 16)
    for seg_len in (0, 100):
        rule = B.keep_rule("per_channel", 0.3, 30, 4, seg_len)
        ws = torch.full((B.ngff_workspace_bytes(700, 6, 10, 3, 16, rule),), 255, dtype=torch.uint8,
                        device="cuda")
        nseg = 1 if seg_len == 0 else 7
        o = oracle_filter(f, 16, "per_channel", np.float32(0.3), seg_len=seg_len)
        for _ in range(2):
            hist = torch.empty((700, nb), dtype=torch.int32, device="cuda")
            count = torch.empty(nseg, dtype=torch.int32, device="cuda")
            r = B.keep_rule("per_channel", 0.3, 30, 4, seg_len, out_hist=hist, out_count=count,
                            workspace=ws)
            s, m = B.cofie_ngff_filter(fd, 16, r)
            torch.cuda.synchronize()
            assert_filter_equal((s.cpu().numpy(), m.cpu().numpy(), hist_np(hist), count.cpu().numpy()), o)


def test_filter_deterministic_and_workspace():
    f = synth.frames(2, 0, 0, 64)
    fd = to_dev(f)
    rule = B.keep_rule("per_channel", 0.2, 30, 4)
    nbytes = B.ngff_workspace_bytes(64, 448, 448, 3, 32, rule)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    rule2 = B.keep_rule("per_channel", 0.2, 30, 4, workspace=ws)
    s1, m1 = B.cofie_ngff_filter(fd, 32, rule)
    s2, m2 = B.cofie_ngff_filter(fd, 32, rule2)
    torch.cuda.synchronize()
    assert torch.equal(s1, s2) and torch.equal(m1, m2)
    small = torch.empty(max(nbytes // 2, 1), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.CofieError) as e:
        B.cofie_ngff_filter(fd, 32, B.keep_rule("per_channel", 0.2, 30, 4, workspace=small))
    assert e.value.code == B.COFIE_ENOMEM


# ------------------------------------------------------------- calibration --

@pytest.mark.parametrize("case", ["tiny", "random", "segments", "1fps"])
def test_calibration_matches_oracle(case):
    if case == "tiny":
        wl = synth.WORKLOADS[1]
        f, bins, mode, target, seg, L = synth.frames(1), wl.bins, wl.hist_mode, wl.target, 0, 30
    elif case == "1fps":
        wl = synth.WORKLOADS[2]
        f, bins, mode, target, seg, L = synth.frames(2), wl.bins, wl.hist_mode, wl.target, 0, 30
    elif case == "random":
        f, bins, mode, target, seg, L = synth.random_frames(31, 90, 6, 6, scenes=20), 8, "per_channel", 30, 0, 6
    else:
        f, bins, mode, target, seg, L = synth.random_frames(32, 200, 6, 6, scenes=40), 16, "joint3d", 12, 50, 8
    n, H, W = f.shape[:3]
    h = oracle.histogram(f, bins, MODES[mode])
    M = oracle.mass(MODES[mode], H, W)
    theta, tau_o = oracle.ngff_calibrate(h, M, target, L, 4, seg)
    rule = B.keep_rule(mode, 0.3, L, 4, seg)
    tau_g = B.cofie_ngff_calibrate(to_dev(f), bins, rule, target).cpu().numpy()
    assert np.array_equal(tau_g.view(np.uint32), tau_o.view(np.uint32))


@pytest.mark.parametrize("H,W,mode,bins", [(2160, 3840, "per_channel", 32),   # 4K: 2M = 4.98e7
                                           (1464, 1920, "per_channel", 16),   # 2M just above 2^24
                                           (2160, 3840, "gray", 32)])         # 2M just below 2^24
def test_filter_frames_beyond_2_24(H, W, mode, bins):
    """Frames whose 2M reaches past 2^24 (Eq. 2 with the score the correctly
    rounded D / 2M): histograms, a threshold calibrated for 50 % retention
    (the binary-search threshold path), scores, masks and counts equal to the
    oracle's, bit for bit."""
    f = synth.random_frames(4242 + H, 24, H, W, 3, scenes=6)
    print(f"4K-class frames {f.shape} {mode} {bins}: 2M = {2 * oracle.mass(MODES[mode], H, W)}", flush=True)
    h = oracle.histogram(f, bins, MODES[mode])
    M = oracle.mass(MODES[mode], H, W)
    theta, tau = oracle.ngff_calibrate(h, M, 12, 30, 4)
    fd = to_dev(f)
    tau_g = B.cofie_ngff_calibrate(fd, bins, B.keep_rule(mode, 0.3, 30, 4), 12)
    torch.cuda.synchronize()
    assert np.array_equal(tau_g.cpu().numpy().view(np.uint32), tau.view(np.uint32))
    for t in (float(tau[0]), 0.011, 0.3):
        g = run_filter(f, bins, mode, t)
        o = oracle_filter(f, bins, mode, t)
        assert_filter_equal(g, o)
