"""Two time steps per launch (FP64 and FP32 cases and batches, marching strips
or in tiles, by size) against one step per launch: the same operations on every
node, so the same bits."""
import numpy as np
import pytest

from paper_1810_09299_amd import inputs

pytestmark = pytest.mark.gpu


def _spec(nr, nz, zper, collision):
    s = inputs.static_droplet(nr=nr, nz=nz, R=max(2.0, 0.3 * min(nr, nz)), W=4.0, ratio=10.0, sigma=1e-3,
                              z_periodic=zper)
    s.collision = "mrt" if collision == "general" else collision
    s.g_z, s.g_ramp = -1e-5, 6.0                      # each of the two steps has its own acceleration
    if collision in ("general", "nmrt"):
        s.s_g = (1.0, 1.1, 1.2, 1.1, 1.1, 0.9, 0.9, 1.0, 1.0)
        s.free_s1 = True
    return s


def _single_steps(spec, precision, n):
    """State after n steps taken one by one."""
    from paper_1810_09299_amd.case import AxiCase
    c = AxiCase(spec, precision=precision)
    for _ in range(n):
        c.step(1)
    st = c.get_state()
    c.close()
    return st


# widths at the edges of one and two wavefronts, of a strip's own columns, and
# of a whole period of lanes (64, 128, 512); fewest rows, short runs of rows
GRIDS = [(4, 4), (5, 7), (9, 54), (16, 55), (7, 64), (12, 65), (20, 118), (33, 119), (40, 128), (24, 182), (11, 247),
         (10, 502), (13, 503), (48, 512), (6, 513)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("collision", ["mrt", "general", "srt", "nmrt"])
@pytest.mark.parametrize("beside", [None, (101, 331), (301, 501), (1201, 1001)])
def test_batch_pairs_equal_single_steps(precision, collision, beside):
    """Small and odd grids, periodic and walled; the case beside them decides
    how the batch goes: the three smallest alone (8 x 4 tiles), in larger tiles,
    or marching.  7 steps: three pairs and an odd step."""
    from paper_1810_09299_amd.batch import Batch
    specs = [_spec(nr, nz, zper, collision) for nr, nz in (GRIDS if beside else GRIDS[:3]) for zper in (True, False)]
    more = [_spec(*beside, True, collision)] if beside else []
    b = Batch(pool_bytes=Batch.pool_for(specs + more, precision), max_cases=len(specs) + len(more),
              precision=precision)
    slots = [b.admit(s, 7) for s in specs]
    for s in more:
        b.admit(s, 8)
    b.run(7)
    for s, slot in zip(specs, slots):
        f, g, aux, t = b.get_state(slot)
        fs, gs, xs, ts = _single_steps(s, precision, 7)
        assert t == ts == 7
        assert np.isfinite(f).all() and np.isfinite(g).all()
        assert np.array_equal(f, fs) and np.array_equal(g, gs) and np.array_equal(aux, xs), (s.nr, s.nz, s.z_periodic)
    b.close()


# in tiles of each shape (one and several to a compute unit), singly where that
# is ahead (69 x 1717, 133 x 920), and marching
CASES = [("fp64", 133, 920, True),
         ("fp32", 52, 1073, True), ("fp64", 52, 1073, False), ("fp32", 69, 1717, False), ("fp32", 300, 600, True),
         ("fp32", 64, 128, False), ("fp64", 33, 65, True), ("fp64", 61, 286, True), ("fp32", 149, 301, False),
         ("fp32", 255, 509, True), ("fp64", 250, 511, False), ("fp64", 131, 2040, True), ("fp64", 405, 2003, True),
         ("fp64", 1605, 500, False), ("fp32", 601, 2003, False), ("fp32", 2370, 512, True), ("fp32", 9600, 128, False)]


@pytest.mark.parametrize("precision,nr,nz,zper", CASES)
def test_case_pairs_equal_single_steps(precision, nr, nz, zper):
    """One case: any split of the steps into calls gives the same state, and
    reading it back (whose fields use the other population buffer) or loading a
    state between pairs leaves the next steps right."""
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(nr, nz, zper, "mrt")
    ref = _single_steps(spec, precision, 8)
    c = AxiCase(spec, precision=precision)
    c.step(5)
    fields, _, _ = c.moments()
    st = c.get_state()
    assert np.array_equal(c.moments()[0]["p"], fields["p"])
    c.step(3)
    got = c.get_state()
    assert got[3] == 8
    for x, y in zip(ref[:3], got[:3]):
        assert np.array_equal(x, y)
    c.set_state(*st)
    c.step(3)
    for x, y in zip(ref[:3], c.get_state()[:3]):
        assert np.array_equal(x, y)
    c.close()


@pytest.mark.parametrize("nr,nz", [(64, 128), (601, 2003)])
def test_recorded_steps_replay_from_their_own_result(nr, nz):
    """Steps recorded into a graph go one by one: an even number of them ends in
    the buffer they started from, so replays continue each other."""
    import torch
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(nr, nz, True, "mrt")
    spec.g_ramp = 0.0                                 # a recording holds the acceleration of its own steps
    ref = _single_steps(spec, "fp32", 6)
    stream = torch.cuda.Stream()
    c = AxiCase(spec, precision="fp32", stream=stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        c.step(2)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    for x, y in zip(ref[:3], c.get_state()[:3]):
        assert np.array_equal(x, y)
    c.close()


FIELDS = ("phi", "rho", "uz", "ur", "p")


@pytest.mark.parametrize("precision,nr,nz", [("fp64", 64, 128), ("fp32", 64, 128), ("fp16", 64, 128),
                                             ("fp64", 601, 2003), ("fp32", 601, 2003)])
def test_live_steps_between_replays(precision, nr, nz):
    """A replay starts from the buffer that was current when its steps, or its
    read-back, were recorded: live steps, in tiles and marching, leave the state
    there after any even number of them."""
    import torch
    from paper_1810_09299_amd import abi
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(nr, nz, True, "mrt")
    spec.g_ramp = 0.0
    stream = torch.cuda.Stream()
    c = AxiCase(spec, precision=precision, stream=stream)
    ref = AxiCase(spec, precision=precision)
    c.step(6)                                         # before the recording: three pairs, buffer 1
    out = [torch.empty((nr, nz), dtype=torch.float64, device="cuda") for _ in FIELDS]
    diag = torch.empty(64, dtype=torch.float64, device="cuda")
    steps, read = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(read, stream=stream):
        abi.lbm_axi_moments_noalloc(c.handle, *(o.data_ptr() for o in out), diag.data_ptr())
    with torch.cuda.graph(steps, stream=stream):
        c.step(2)
    done = 6

    def replay(graph):                                # on the case's stream, after its live steps
        with torch.cuda.stream(stream):
            graph.replay()

    for live in ((2,), (6,), (50,), (3, 5), (0,), (7, 1, 2)):
        replay(steps)
        for n in live:
            c.step(n)
        done += 2 + sum(live)
        while ref.t < done:
            ref.step(1)
        want = ref.moments()[0]
        replay(read)
        torch.cuda.synchronize()
        got = c.moments()[0]
        for o, k in zip(out, FIELDS):
            assert np.array_equal(o.cpu().numpy(), want[k]), (live, k)
            assert np.array_equal(got[k], want[k]), (live, k)
    for x, y in zip(ref.get_state()[:3], c.get_state()[:3]):
        assert np.array_equal(x, y)
    c.close()
    ref.close()


def test_recorded_batch_steps_replay_from_their_own_result():
    """Steps of a batch that a caller records (launched one by one: a gravity
    ramp), replayed between live ones, against a case in the same sequence."""
    import torch
    from paper_1810_09299_amd.batch import Batch
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(33, 130, True, "mrt")
    spec.g_ramp = 1000.0
    streams = [torch.cuda.Stream() for _ in range(2)]
    b = Batch(pool_bytes=Batch.pool_for([spec], "fp32"), max_cases=1, precision="fp32", stream=streams[0])
    slot = b.admit(spec, 10 ** 6)
    c = AxiCase(spec, precision="fp32", stream=streams[1])
    b.run(4)
    for _ in range(4):
        c.step(1)
    b.sync()
    graphs = []
    for step, stream in ((b.run, streams[0]), (c.step, streams[1])):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            step(2)
        graphs.append(g)
    for live in ((2,), (6,), (1, 3), (50,)):
        for g in graphs:
            for _ in range(2):
                g.replay()
                torch.cuda.synchronize()
        for n in live:
            b.run(n)
            for _ in range(n):
                c.step(1)
        for x, y in zip(b.get_state(slot)[:3], c.get_state()[:3]):
            assert np.array_equal(x, y), live
    b.close()
    c.close()


def test_steps_on_the_null_stream_while_another_stream_records():
    """A program records a graph of its own on a blocking stream; a case on the
    null stream goes on stepping, in pairs and singly."""
    import ctypes

    import torch
    from paper_1810_09299_amd.case import AxiCase
    hip = ctypes.CDLL("libamdhip64.so")
    spec = _spec(64, 128, True, "mrt")
    c = AxiCase(spec, precision="fp32", stream=torch.cuda.default_stream())
    assert c.stream.cuda_stream == 0
    s, g = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(s)) == 0
    assert hip.hipStreamBeginCapture(s, 2) == 0       # hipStreamCaptureModeRelaxed
    try:
        for n in (2, 1, 4):
            c.step(n)
    finally:
        assert hip.hipStreamEndCapture(s, ctypes.byref(g)) == 0
    if g.value:
        assert hip.hipGraphDestroy(g) == 0
    assert hip.hipStreamDestroy(s) == 0
    for x, y in zip(_single_steps(spec, "fp32", 7)[:3], c.get_state()[:3]):
        assert np.array_equal(x, y)
    c.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_read_back_between_replays_of_single_steps(precision):
    """Two graphs of one step each, one per buffer, replayed in turn: a live
    read-back in between (of the other buffer, in which the first graph began)
    leaves the state that the second begins with."""
    import torch
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(33, 130, True, "mrt")
    spec.g_ramp = 0.0
    stream = torch.cuda.Stream()
    c = AxiCase(spec, precision=precision, stream=stream)
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
    for g in graphs:
        with torch.cuda.graph(g, stream=stream):
            c.step(1)
    for _ in range(3):
        for g in graphs:
            g.replay()
            torch.cuda.synchronize()
            last = c.moments()[0]
            c.diagnostics()
    ref = AxiCase(spec, precision=precision)
    for _ in range(6):
        ref.step(1)
    want = ref.moments()[0]
    for k in FIELDS:
        assert np.array_equal(last[k], want[k]), k
    for x, y in zip(ref.get_state()[:3], c.get_state()[:3]):
        assert np.array_equal(x, y)
    c.close()
    ref.close()
