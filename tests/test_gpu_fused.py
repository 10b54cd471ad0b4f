"""Fused D2Q9 steps: several steps in one launch equal the same steps taken
one call at a time (the two-kernel path) bit for bit, in every form, for
tiles of every shape the plan chooses and lattices smaller than their halo."""
import numpy as np
import pytest

import paper_2605_22214_amd as nf

pytestmark = pytest.mark.gpu

FIELDS = ("C", "V", "P", "F", "MU")
PLAIN, DIFF, POT = 0, nf.FLAG_NO_HYDRO, nf.FLAG_POTENTIAL_FORCE


def _config(shape, N, precision, flags=0, omega=0.0, force=(0.0, 0.0, 0.0)):
    return dict(lattice="D2Q9", shape=shape + (1,), sigma=0.01 * (np.ones((N, N)) - np.eye(N)), tau=np.ones(N),
                m=0.05, precision=precision, flags=flags, omega_stab=omega, body_force=force)


def _noise(shape, N, seed):
    C = 1.0 / N + np.random.default_rng(seed).uniform(-0.1, 0.1, size=(N, 1, shape[1], shape[0]))
    return C / C.sum(axis=0)


def _same(a, b):
    for name in FIELDS:
        assert np.array_equal(a.get_field(name), b.get_field(name)), name
    assert np.array_equal(a.get_state(), b.get_state())


CASES = [
    ((64, 64), 3, "fp64", PLAIN, 0.0, (0.0, 0.0, 0.0)),        # small tiles, four steps a launch
    ((5, 3), 2, "fp32", PLAIN, 0.0, (0.0, 0.0, 1e-6)),         # smaller than the halo
    ((1, 1), 3, "fp32", PLAIN, 0.0, (0.0, 0.0, 0.0)),
    ((161, 150), 4, "fp32", PLAIN, 0.05, (1e-5, 0.0, 0.0)),    # 20 x 8 tiles
    ((250, 253), 4, "fp16s", PLAIN, 0.0, (0.0, 1e-6, 0.0)),    # 24 x 8
    ((515, 389), 3, "fp32", POT, 0.0, (0.0, 0.0, 0.0)),        # 24 x 24, 1024 threads
    ((419, 470), 5, "fp16s", POT, 0.05, (0.0, 0.0, 0.0)),      # 24 x 24, 512 threads
    ((301, 250), 6, "fp64", PLAIN, 0.05, (0.0, 0.0, 0.0)),     # 24 x 16, 768 threads
    ((333, 299), 5, "fp64", POT, 0.0, (1e-6, 0.0, 0.0)),
    ((301, 150), 7, "fp64", PLAIN, 0.05, (0.0, 0.0, 0.0)),     # 24 x 16, 512 threads
    ((170, 333), 8, "fp64", PLAIN, 0.0, (0.0, 0.0, 0.0)),      # the largest records
    ((90, 33), 7, "fp32", PLAIN, 0.0, (0.0, 0.0, 0.0)),
    ((700, 433), 4, "fp32", DIFF, 0.05, (0.0, 0.0, 0.0)),      # 56 x 24
    ((90, 33), 3, "fp64", DIFF, 0.0, (0.0, 0.0, 0.0)),
    ((433, 250), 5, "fp16s", DIFF, 0.0, (0.0, 0.0, 0.0)),
    ((3, 70), 8, "fp64", DIFF, 0.05, (0.0, 0.0, 0.0)),
]


@pytest.mark.parametrize("shape,N,precision,flags,omega,force", CASES)
def test_fused_equals_single_steps(shape, N, precision, flags, omega, force):
    cfg = _config(shape, N, precision, flags, omega, force)
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    C = _noise(shape, N, 1)
    a.set_fields(C)
    b.set_fields(C)
    for _ in range(15):
        a.step(1)
    b.step(1)
    b.step(2)
    b.step(3)
    b.step(9)
    _same(a, b)


@pytest.mark.parametrize("precision,flags", [("fp32", PLAIN), ("fp64", PLAIN), ("fp32", DIFF)])
def test_fused_batch_equals_single_steps(precision, flags):
    shapes = [(64, 41), (130, 97), (7, 200), (33, 33)]
    cfgs = [_config(s, 3, precision, flags, 0.05 * (i & 1)) for i, s in enumerate(shapes)]
    batch = nf.Batch(cfgs)
    sims = [nf.Simulation(**c) for c in cfgs]
    for i, s in enumerate(shapes):
        batch.set_fields(i, _noise(s, 3, i))
        sims[i].set_fields(_noise(s, 3, i))
    for n in (1, 7, 1, 12):
        batch.step(n)
        for s in sims:
            for _ in range(n):
                s.step(1)
    for m, s in zip(batch.members, sims):
        _same(m, s)


def test_fused_steps_report_nan():
    cfg = _config((70, 50), 3, "fp32")
    s = nf.Simulation(**cfg)
    C = _noise((70, 50), 3, 2)
    C[0, 0, 20, 30] = np.nan
    s.set_fields(C)
    s.set_nan_check(5)
    s.step(3)
    s.synchronize()          # no checked step yet
    s.step(4)                # the fifth is
    with pytest.raises(nf.NflbmError):
        s.synchronize()


MOB_CASES = [
    ((90, 70), 4, "fp32", 0.0),
    ((5, 3), 3, "fp64", 0.05),       # smaller than the halo
    ((1, 1), 2, "fp32", 0.0),
    ((45, 131), 4, "fp16s", 0.05),
    ((67, 50), 8, "fp64", 0.0),      # the largest LDS records: one step a launch
    ((60, 47), 6, "fp32", 0.05),
]


@pytest.mark.parametrize("shape,N,precision,omega", MOB_CASES)
def test_fused_mobility_equals_single_steps(shape, N, precision, omega):
    cfg = _config(shape, N, precision, nf.FLAG_NO_HYDRO | nf.FLAG_C2C2_MOBILITY, omega)
    cfg["m"] = 10.0
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    C = _noise(shape, N, 3)
    a.set_fields(C)
    b.set_fields(C)
    for _ in range(14):
        a.step(1)
    b.step(2)
    b.step(3)
    b.step(9)
    if shape != (1, 1):              # a single node stays as it is
        assert np.abs(a.get_field("C") - C).max() > 1e-6
    assert np.array_equal(a.get_field("C"), b.get_field("C"))
    assert np.array_equal(a.get_field("G_RAW"), b.get_field("G_RAW"))


def test_fused_mobility_steps_report_nan():
    cfg = _config((70, 50), 4, "fp32", nf.FLAG_NO_HYDRO | nf.FLAG_C2C2_MOBILITY)
    s = nf.Simulation(**cfg)
    C = _noise((70, 50), 4, 2)
    C[0, 0, 20, 30] = np.nan
    s.set_fields(C)
    s.step(16)
    with pytest.raises(nf.NflbmError):
        s.synchronize()


@pytest.mark.parametrize("flags,N", [(PLAIN, 3), (nf.FLAG_NO_HYDRO | nf.FLAG_C2C2_MOBILITY, 4)])
def test_captured_fused_steps_replay(flags, N):
    """An even number of steps captured into a graph advances the state by as
    many on every replay, read-backs between them included."""
    torch = pytest.importorskip("torch")
    cfg = _config((70, 50), N, "fp32", flags)
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    C = _noise((70, 50), N, 4)
    stream = torch.cuda.Stream()
    b.set_stream(stream.cuda_stream)
    for s in (a, b):
        s.set_fields(C)
        s.set_nan_check(0)
    a.step(1)
    b.step(1)
    a.step(2)
    b.step(2)                   # the fused steps' memory is there
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        b.step(6)
    for _ in range(3):
        for _ in range(6):
            a.step(1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(a.get_field("C"), b.get_field("C"))


@pytest.mark.parametrize("batch", [False, True])
def test_restored_velocities_advect_one_step(batch):
    """A state of a run with flow, restored where the flow is not evolved:
    its velocities act on the first step, as they do in single steps."""
    shape, N = (70, 50), 3
    cfg = _config(shape, N, "fp32", DIFF)
    with nf.Simulation(**_config(shape, N, "fp32", nf.FLAG_F_POPULATIONS)) as flow:
        v = np.zeros((3, 1, shape[1], shape[0]))
        v[0] = 0.02 * np.random.default_rng(5).uniform(-1.0, 1.0, size=v.shape[1:])
        flow.set_fields(_noise(shape, N, 5), v)
        flow.step(3)
        raw = flow.get_state()
    a = nf.Simulation(**cfg)
    b = nf.Batch([cfg]) if batch else nf.Simulation(**cfg)
    s = b.members[0] if batch else b
    for warm in (a, s):
        warm.set_fields(_noise(shape, N, 6))
    a.step(2)
    b.step(2)
    a.set_state(raw)
    s.set_state(raw)
    for _ in range(7):
        a.step(1)
    b.step(7)
    _same(a, s)


def test_captured_step_replays_after_odd_calls():
    """A captured pair of single steps advances the state after calls of any
    lengths that add up to an even number."""
    torch = pytest.importorskip("torch")
    cfg = _config((70, 50), 3, "fp32")
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    stream = torch.cuda.Stream()
    b.set_stream(stream.cuda_stream)
    for s in (a, b):
        s.set_fields(_noise((70, 50), 3, 4))
        s.set_nan_check(0)
        s.step(1)
        s.step(1)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        b.step(1)
        b.step(1)
    total = 0
    for n in (3, 5, 7):
        b.step(n)
        b.step(1)
        with torch.cuda.stream(stream):
            g.replay()
        total += n + 3
    for _ in range(total):
        a.step(1)
    assert np.array_equal(a.get_field("C"), b.get_field("C"))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("N", range(2, 9))
def test_resting_state_keeps_its_bytes(N, precision):
    """At rest -3/2 v.v is a zero, whose sign binary16 records hold as the
    two kernels store it: the checkpoint's bytes do not depend on the split."""
    for flags, omega in ((PLAIN, 0.0), (PLAIN, 0.05), (POT, 0.0), (POT, 0.05), (DIFF, 0.0)):
        cfg = _config((40, 33), N, precision, flags, omega)
        _resting_bytes(cfg, N, (flags, omega))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("N", range(2, 9))
def test_resting_mobility_state_keeps_its_bytes(N, precision):
    """The same where the source terms are zeros of either sign."""
    for omega in (0.0, 0.05):
        cfg = _config((40, 33), N, precision, DIFF | nf.FLAG_C2C2_MOBILITY, omega)
        cfg["m"] = 10.0
        _resting_bytes(cfg, N, omega)


def _resting_bytes(cfg, N, case):
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    for s in (a, b):
        s.set_fields(np.full((N, 1, 33, 40), 1.0 / N))
    for _ in range(9):
        a.step(1)
    b.step(9)
    assert np.array_equal(a.get_state(), b.get_state()), case


@pytest.mark.parametrize("shape,N,precision,flags,omega", [
    ((701, 643), 5, "fp32", PLAIN, 0.0),      # 24 x 20, two workgroups a CU
    ((611, 470), 5, "fp16s", PLAIN, 0.0),
    ((601, 580), 6, "fp32", POT, 0.05),       # 24 x 16
    ((563, 541), 7, "fp32", PLAIN, 0.0),      # 24 x 12
    ((371, 370), 8, "fp16s", PLAIN, 0.0),     # one round of the tallest tile
    ((561, 540), 5, "fp64", PLAIN, 0.0),      # 24 x 20, 768 threads
    ((333, 299), 6, "fp64", PLAIN, 0.05),     # 24 x 16, 512 threads
    ((431, 419), 7, "fp64", PLAIN, 0.0),      # 24 x 12
    ((431, 419), 8, "fp64", POT, 0.05),
    ((1001, 523), 8, "fp32", PLAIN, 0.05),    # the two kernels
])
def test_shapes_beyond_one_round(shape, N, precision, flags, omega):
    cfg = _config(shape, N, precision, flags, omega, (1e-6, 0.0, 0.0))
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    C = _noise(shape, N, 7)
    for s in (a, b):
        s.set_fields(C)
    for _ in range(8):
        a.step(1)
    b.step(3)
    b.step(5)
    _same(a, b)


def test_fused_mobility_tall_tiles():
    shape, N = (311, 290), 8                # 28 x 12, one step a launch
    cfg = _config(shape, N, "fp64", nf.FLAG_NO_HYDRO | nf.FLAG_C2C2_MOBILITY, 0.05)
    cfg["m"] = 10.0
    a, b = nf.Simulation(**cfg), nf.Simulation(**cfg)
    C = _noise(shape, N, 8)
    for s in (a, b):
        s.set_fields(C)
    for _ in range(5):
        a.step(1)
    b.step(2)
    b.step(3)
    assert np.array_equal(a.get_state(), b.get_state())


@pytest.mark.parametrize("N,precision", [(3, "fp32"), (6, "fp64"), (4, "fp16s")])
def test_batch_member_gains_and_loses_solid_nodes(N, precision):
    """A batch leaves the fused steps while a member has solid nodes and takes
    them again afterwards, at the state its members have by then."""
    shapes = [(64, 41), (90, 57)]
    cfgs = [_config(s, N, precision) for s in shapes]
    batch = nf.Batch(cfgs)
    sims = [nf.Simulation(**c) for c in cfgs]
    solid = np.zeros((1, 57, 90), dtype=bool)
    solid[0, 20:30, 10:25] = True
    for i, s in enumerate(shapes):
        batch.set_fields(i, _noise(s, N, i))
        sims[i].set_fields(_noise(s, N, i))

    def advance(n):
        batch.step(n)
        for s in sims:
            for _ in range(n):
                s.step(1)

    advance(6)
    for mask in (solid, None, solid, None):
        batch.members[1].set_solid(mask)
        sims[1].set_solid(mask)
        advance(5)
        batch.members[0].step(3)         # one member on its own in between
        for _ in range(3):
            sims[0].step(1)
        advance(4)
    for m, s in zip(batch.members, sims):
        _same(m, s)
