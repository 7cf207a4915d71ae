"""Parity fuzzing of the kernel generators: random groups (elementwise ops on full and per-row
values, reductions over the last dim, broadcasts back, optional column sums) are planned, run
on the GPU and compared with the CPU oracle, through every template that takes them."""
import random
import sys

import pytest
import torch

from oracle import interp
from paper_1911_11576_amd import FsError, FusedProgram, Plan, binding
from workloads import TOLERANCE, graphs, inputs

from gpu_util import alloc_outputs, assert_close, check_against_oracle, to_device

pytestmark = pytest.mark.gpu


def announce(msg):
    sys.__stderr__.write(f"[gpu-case] {msg}\n")
    sys.__stderr__.flush()


@pytest.fixture(autouse=True)
def _need_gpu(device):
    yield


SHAPES = [(37, 128), (5, 768), (3, 7, 64), (2, 3, 5, 32), (300, 8), (33, 100), (65, 30), (7, 770), (4, 4096), (129, 16)]


@pytest.mark.parametrize("seed", range(24))
def test_random_row_groups(seed):
    rng = random.Random(4242 + seed)
    shape = SHAPES[seed % len(SHAPES)]
    dtype = ["f32", "f32", "bf16", "f16"][seed % 4]
    ops, pshapes = graphs.random_row_group(rng, shape, dtype, n_ops=rng.randint(6, 16))
    ins = inputs.normal_tensors(pshapes, dtype, seed_offset=100 + seed)
    announce(f"random row group seed {seed} shape {shape} {dtype}: {len(ops)} ops")
    with Plan(ops) as p:
        schedule = p.info()["schedule"]
        assert schedule in ("row", "elementwise")
        streamed = "streamed" in p.describe()
    check_against_oracle(ops, ins, what=f"random group {seed}")
    if schedule == "row":
        if not streamed:
            check_against_oracle(ops, ins, what=f"random group {seed} streamed", grid=3)
        try:
            check_against_oracle(ops, ins, what=f"random group {seed} persistent", grid=2, rows_per_wave=1)
        except FsError as e:
            assert e.status == binding.FS_ERR_UNSUPPORTED      # rows too long for one wavefront's registers


@pytest.mark.parametrize("seed", range(15))
def test_random_groups_with_column_sums(seed):
    rng = random.Random(777 + seed)
    # (rank above 2: the sum over the rows is a chain of sums over the leading dim)
    shape = [(37, 128), (300, 8), (33, 100), (517, 1024), (65, 30), (5, 2048), (1000, 64), (129, 16),
             (40, 4096), (33, 3000), (9, 8192), (3, 7, 64), (2, 3, 5, 32), (2, 9, 4096), (4, 50, 100)][seed]
    ops, pshapes = graphs.random_row_group(rng, shape, "f32", n_ops=rng.randint(5, 12), column_sums=True)
    ins = inputs.normal_tensors(pshapes, "f32", seed_offset=200 + seed)
    announce(f"random group with column sum seed {seed} shape {shape}: {len(ops)} ops")
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row_col" and p.info()["n_kernels"] == 2
    check_against_oracle(ops, ins, what=f"random column group {seed}")
    check_against_oracle(ops, ins, what=f"random column group {seed} grid 3", grid=3, wg_size=128)


@pytest.mark.parametrize("seed", range(12))
def test_random_groups_with_column_sums_per_run_of_rows(seed):
    """Random row groups whose extra outputs are sums over the innermost row dims ([B, S, H] over S;
    [B, N, S, H] over S, or over S and N): runs of 1 to 600 rows, one or several workgroups per run,
    rows of one wavefront and of a team."""
    rng = random.Random(4242 + seed)
    shape = [(37, 5, 128), (300, 7, 8), (3, 600, 100), (2, 3, 5, 32), (65, 2, 30), (5, 9, 2048), (1, 64, 64), (4, 1, 96),
             (6, 20, 4096), (2, 4, 50, 100), (700, 3, 64), (2, 2, 2, 2)][seed]
    dtype = ["f32", "bf16", "f16"][seed % 3]
    ops, pshapes = graphs.random_row_group(rng, shape, dtype, n_ops=rng.randint(4, 12), column_sums="runs")
    ins = inputs.normal_tensors(pshapes, dtype, seed_offset=400 + seed)
    announce(f"random group with column sums per run seed {seed} shape {shape} {dtype}: {len(ops)} ops")
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row_col" and "per run of" in p.describe()
    check_against_oracle(ops, ins, what=f"random run-sum group {seed}")
    check_against_oracle(ops, ins, what=f"random run-sum group {seed} wg 128", wg_size=128)


@pytest.mark.parametrize("shape,dtype", [((300, 96), "f32"), ((7, 5, 33), "f32"), ((64, 2048), "bf16"), ((1000, 4), "f16")])
def test_per_row_arithmetic_without_a_reduction(shape, dtype):
    ops = graphs.gated_rows(shape, dtype)
    ins = inputs.normal_tensors([shape, shape[:-1], shape[-1:]], dtype, seed_offset=31)
    announce(f"gated rows {shape} {dtype}")
    check_against_oracle(ops, ins, what=f"gated rows {shape}")
    check_against_oracle(ops, ins, what=f"gated rows {shape} streamed", grid=5)


POOL = [(37, 128), (5, 768), (3, 7, 64), (2, 3, 5, 32), (300, 8), (33, 100), (65, 30), (7, 770), (4, 4096), (129, 16),
        (6, 40000), (50, 2), (9, 1), (3, 2, 2, 2), (17, 6000)]


@pytest.mark.parametrize("seed", range(45))
def test_random_groups_wide_pool(seed):
    """More shapes (rows of 1 or 2 elements, rows for the streamed template, rows for wavefront
    teams), all three dtypes, 3 to 24 ops, a column sum on every fourth rank-2 case."""
    rng = random.Random(9000 + seed)
    shape = POOL[seed % len(POOL)]
    dtype = ["f32", "bf16", "f16"][seed % 3]
    col = seed % 4 == 3 and len(shape) == 2
    ops, pshapes = graphs.random_row_group(rng, shape, dtype, n_ops=rng.randint(3, 24), column_sums=col)
    ins = inputs.normal_tensors(pshapes, dtype, seed_offset=300 + seed)
    announce(f"random group (wide pool) seed {seed} shape {shape} {dtype} column sum {col}: {len(ops)} ops")
    try:
        check_against_oracle(ops, ins, what=f"random group {seed}")
    except FsError as e:
        # the one documented limit this pool reaches
        assert e.status == binding.FS_ERR_UNSUPPORTED and "column reductions over rows longer" in e.message


@pytest.mark.parametrize("seed", range(20))
def test_random_packed_elementwise_parts(seed):
    """Independent elementwise computations of different shapes and dtypes in one op list: one kernel,
    each part on its own run of workgroups."""
    import numpy as np
    rng = random.Random(5000 + seed)
    ops, pshapes, pdtypes = graphs.random_elementwise_parts(rng)
    r = np.random.default_rng(seed)
    ins = [inputs.round_to(r.normal(0.0, 1.0, s), dt) for s, dt in zip(pshapes, pdtypes)]
    announce(f"random packed parts seed {seed}: {len(ops)} ops, shapes {pshapes[::3]}")
    with Plan(ops) as p:
        assert p.info()["schedule"] == "elementwise" and p.info()["n_kernels"] == 1
    check_against_oracle(ops, ins, what=f"random packed parts {seed}")


DOT_SHAPES = [(3, 64, 64, 64, 64), (2, 37, 52, 40, 32), (4, 16, 128, 32, 128), (2, 100, 36, 72, 64), (5, 1, 8, 16, 32),
              (2, 128, 128, 128, 64), (3, 50, 20, 24, 32), (2, 33, 100, 64, 128)]


@pytest.mark.parametrize("seed", range(32))
def test_random_groups_around_two_dots(seed):
    """dot -> random middle section -> dot -> random epilogue (elementwise ops and row reductions on the second
    dot's result), the first dot's second operand stored either way, f16 and bf16: all through the generated
    block-composed kernel (the hand-written attention kernel is not asked), one kernel each."""
    import numpy as np
    rng = random.Random(12000 + seed)
    B, M, N, Kc, D = DOT_SHAPES[seed % len(DOT_SHAPES)]
    dtype = ["f16", "bf16"][seed % 2]
    ops, params = graphs.random_dot_group(rng, B, M, N, Kc, D, dtype)
    r = np.random.Generator(np.random.PCG64(inputs.BASE_SEED + 400 + seed))
    ins = [inputs.round_to(r.normal(0.0, 1.0, shape), dt) for shape, dt in params]
    announce(f"random group around two dots, seed {seed} {B}x{M}x{N} K={Kc} D={D} {dtype}: {len(ops)} ops")
    with Plan(ops, "generated") as plan:
        assert plan.info()["schedule"] == "block_dot" and plan.info()["n_kernels"] == 1
    check_against_oracle(ops, ins, "generated", what=f"random dot group {seed}")


def random_whole_tensor_group(rng):
    """Tensors of several shapes and dtypes, sums and maxima over whole ones, ops on those scalars, and ops on the tensors that read them."""
    g = graphs.Graph()

    def f32(v):
        return v if g.dtype(v) == "f32" else g.convert(v, "f32")

    def mixed(a, b):
        return rng.choice([g.add, g.subtract, g.multiply, g.maximum])(a, b)

    def bounded(v):
        return rng.choice([lambda: v, lambda: g.tanh(v), lambda: g.negate(v), lambda: g.multiply(v, g.constant(0.5)), lambda: g.multiply(v, v), lambda: g.logistic(v)])()

    tensors, pshapes, dtypes = [], [], []
    for k in range(rng.randint(1, 5)):
        shape = rng.choice([(1,), (3,), (7,), (33, 100), (4095,), (3, 5, 7), (1030,), (257, 129), (2, 3, 4, 5), (64, 64), (9001,)])
        dt = rng.choice(["f32", "f32", "bf16", "f16"])
        ps = [g.parameter(f"x{k}_{j}", dt if j == 0 else rng.choice([dt, "f32"]), shape) for j in range(rng.choice([1, 1, 2, 3]))]
        pshapes += [shape] * len(ps)
        dtypes += [g.dtype(p) for p in ps]
        v = bounded(f32(ps[0]))
        for p in ps[1:]:
            v = mixed(v, bounded(f32(p)))
        tensors.append((v, ps, dt))
    n_inputs = rng.randint(0, 2)
    scalars = [g.parameter(f"s{k}", "f32", ()) for k in range(n_inputs)]
    for v, ps, _ in tensors:
        for _ in range(rng.choice([0, 1, 1, 2]) if v != tensors[0][0] else 1):
            s, size, total = rng.choice([v, f32(ps[0]), f32(ps[-1])]), 1, rng.random() < 0.6
            if rng.random() < 0.5:
                s = bounded(s)
            for e in g.shape(s):
                size *= e
            while len(g.shape(s)) > 0:
                s = (g.reduce_sum if total else g.reduce_max)(s, rng.choice([0, len(g.shape(s)) - 1]))
            scalars.append(g.multiply(s, g.constant(1.0 / size)) if total else s)
    for _ in range(rng.randint(0, 4)):
        a = mixed(rng.choice(scalars), rng.choice(scalars + [g.constant(0.75)]))
        scalars.append(rng.choice([lambda: g.tanh(a), lambda: g.sqrt(g.add(g.multiply(a, a), g.constant(1.0))), lambda: g.divide(a, g.sqrt(g.add(g.multiply(a, a), g.constant(0.5))))])())
    reads = False
    for v, ps, dt in tensors:
        y = rng.choice([v, f32(ps[0])])
        for _ in range(rng.choice([0, 1, 1, 2]) if reads else 1):
            y = mixed(y, g.broadcast(rng.choice(scalars[n_inputs:]), g.shape(y), 0))
            reads = True
        y = g.add(bounded(y), g.constant(0.25))
        g.output(y if dt == "f32" else g.convert(y, dt))
        if rng.random() < 0.2:
            g.output(g.multiply(y, g.constant(2.0)))
    for s in rng.sample(scalars[n_inputs:], rng.choice([0, 0, 1])):
        g.output(g.add(s, g.constant(0.5)))
    # (what no output reads is left out, the inputs apart)
    read = set()
    for i in range(len(g.ops) - 1, -1, -1):
        if g.ops[i].kind in ("output", "parameter") or i in read:
            read |= {i, *g.ops[i].operands}
    number = {old: new for new, old in enumerate(sorted(read))}
    ops = [g.ops[i]._replace(operands=tuple(number[o] for o in g.ops[i].operands)) for i in sorted(read)]
    return ops, pshapes + [()] * n_inputs, dtypes + ["f32"] * n_inputs


@pytest.mark.parametrize("seed", range(24))
def test_random_whole_tensor_groups(seed):
    """As one two-step plan where that takes the group, and as a program, whose plan may or may not be one."""
    rng = random.Random(90210 + seed)
    ops, pshapes, dtypes = random_whole_tensor_group(rng)
    announce(f"random whole-tensor group seed {seed}: {len(ops)} ops over {pshapes}")
    ins = [inputs.normal_tensors([s or (1,)], d, seed_offset=300 + 10 * seed + k)[0].reshape(s) for k, (s, d) in enumerate(zip(pshapes, dtypes))]
    want = interp.run(ops, ins)
    dev_in = to_device(ops, ins)
    results = []
    try:
        plan, extra = Plan.two_step(ops)
        with plan:
            outs = alloc_outputs(ops)
            plan.launch(dev_in, outs + [torch.empty(extra, dtype=torch.uint8, device="cuda:0")])
            torch.cuda.synchronize()
            results.append(outs)
    except FsError as e:
        assert e.status == binding.FS_ERR_UNSUPPORTED
    with FusedProgram(ops) as prog:
        results.append(prog.run(dev_in))
        torch.cuda.synchronize()
    tol = TOLERANCE["f32" if set(dtypes) == {"f32"} else "bf16"]      # (16-bit groups take the short forms of tanh and exp)
    for outs in results:
        for k, (a, b) in enumerate(zip(outs, want)):
            assert_close(a.double().cpu().numpy(), b, tol, f"random whole-tensor group {seed} output {k}")
