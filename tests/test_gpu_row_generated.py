"""GPU parity of the generated row schedule (elementwise ops and reductions over the last
dim emitted as one kernel) against the CPU oracle: the benchmark's row groups in generated
form, and op mixes that no hand-written kernel matches."""
import sys

import numpy as np
import pytest
import torch

from oracle import interp
from paper_1911_11576_amd import FsError, Plan, binding
from workloads import BY_NAME, TOLERANCE, graphs, inputs

from gpu_util import alloc_outputs, assert_close, check_against_oracle, product_with_column_sums, run_gpu, to_device

pytestmark = pytest.mark.gpu


def announce(msg):
    sys.__stderr__.write(f"[gpu-case] {msg}\n")
    sys.__stderr__.flush()


@pytest.fixture(autouse=True)
def _need_gpu(device):
    yield


@pytest.mark.parametrize("name", ["layernorm_fwd", "scaled_masked_softmax", "bias_gelu_residual_layernorm"])
def test_benchmark_row_groups_in_generated_form(name):
    announce(f"generated row {name}")
    ops, ins = BY_NAME[name].build("small")
    with Plan(ops, "generated") as p:
        assert p.info()["schedule"] == "row" and "generated kernel" in p.describe()
    check_against_oracle(ops, ins, "generated", what=f"{name} generated")


def test_key_padding_mask_in_generated_form():
    announce("generated row key padding")
    shape = (2, 3, 16, 128)
    ops = graphs.scaled_masked_softmax(shape, 0.125, "key_padding")
    ins = inputs.scaled_masked_softmax(shape, "key_padding")
    check_against_oracle(ops, ins, "generated", what="key padding generated")


SHAPES = [(37, 128), (5, 768), (3, 7, 64), (2, 3, 5, 32), (300, 8), (129, 16), (33, 100), (9, 1000), (65, 30), (7, 770), (11, 5), (4, 2048), (1, 4)]


@pytest.mark.parametrize("shape", SHAPES)
def test_log_softmax(shape):
    announce(f"log_softmax {shape}")
    ops = graphs.log_softmax(shape)
    with Plan(ops) as p:                       # no hand-written kernel matches: generated by default
        assert p.info()["schedule"] == "row" and "generated kernel" in p.describe()
    check_against_oracle(ops, inputs.normal_tensors([shape], scale=3.0), what=f"log_softmax {shape}")


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(37, 128), (5, 768), (3, 7, 64), (33, 100), (65, 30), (300, 8), (19, 2048)])
def test_rmsnorm(shape, dtype):
    announce(f"rmsnorm {shape} {dtype}")
    ops = graphs.rmsnorm(shape, dtype)
    check_against_oracle(ops, inputs.normal_tensors([shape, shape[-1:]], dtype), what=f"rmsnorm {shape} {dtype}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(37, 128), (3, 7, 64), (2, 3, 5, 32), (33, 100), (11, 5)])
def test_l2_normalize_with_row_operand_and_row_output(shape, dtype):
    announce(f"l2 normalize {shape} {dtype}")
    ops = graphs.l2_normalize_scaled(shape, dtype)
    check_against_oracle(ops, inputs.normal_tensors([shape, shape[:-1]], dtype), what=f"l2norm {shape} {dtype}")


@pytest.mark.parametrize("rows,cols,dtype", [(37, 768, "f32"), (203, 1024, "bf16"), (5, 12, "f32"), (64, 100, "f16")])
def test_layernorm_forward_returning_its_statistics(rows, cols, dtype):
    announce(f"layernorm with stats {rows}x{cols} {dtype}")
    ops = graphs.layernorm_fwd_with_stats(rows, cols, dtype)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row" and p.info()["n_kernels"] == 1
    check_against_oracle(ops, inputs.layernorm_fwd(rows, cols, dtype), what="layernorm with stats")


@pytest.mark.parametrize("shape", [(37, 128), (2, 3, 5, 32), (300, 8), (33, 100)])
def test_softmax_with_log_sum_exp(shape):
    announce(f"softmax+lse {shape}")
    ops = graphs.softmax_with_lse(shape)
    got, want = check_against_oracle(ops, inputs.normal_tensors([shape], scale=2.0), what=f"softmax+lse {shape}")
    assert_close(got[0].sum(-1), np.ones(shape[:-1]), 1e-5, "rows sum to one")


@pytest.mark.parametrize("shape", [(37, 128), (1000, 4), (65, 30), (3, 1024)])
def test_lone_row_reduction(shape):
    announce(f"row sum of squares {shape}")
    ops = graphs.row_sum_of_squares(shape)
    check_against_oracle(ops, inputs.normal_tensors([shape]), what=f"sum of squares {shape}")


def test_tiny_rows_use_the_thread_template_and_long_rows_the_wavefront():
    announce("templates")
    with Plan(graphs.log_softmax((300, 5))) as p:
        assert "THREAD]" in p.describe()           # one thread per row, sequential reduction
    with Plan(graphs.log_softmax((300, 8)), rows_per_wave=64) as p:
        assert "THREAD]" in p.describe()           # ... on request for any short row
    with Plan(graphs.log_softmax((300, 768))) as p:
        assert "WARP]" in p.describe()
    # every lanes-per-row template computes the same thing
    shape = (301, 32)
    ops, ins = graphs.softmax_with_lse(shape), inputs.normal_tensors([shape], scale=2.0)
    want = interp.run(ops, ins)
    for rpw in (1, 2, 4, 8, 16, 32, 64):
        got = run_gpu(ops, ins, rows_per_wave=rpw)
        for a, b in zip(got, want):
            assert_close(a, b, 1e-5, f"rows_per_wave={rpw}")
    with pytest.raises(FsError) as e:              # 2048 columns on one lane: too many registers
        Plan(graphs.log_softmax((4, 2048)), rows_per_wave=64)
    assert e.value.status == binding.FS_ERR_UNSUPPORTED
    with pytest.raises(FsError) as e:
        Plan(graphs.log_softmax((4, 64)), rows_per_wave=3)
    assert e.value.status == binding.FS_ERR_INVALID


def test_generated_matches_hand_written_and_options():
    announce("generated vs hand-written")
    ops, ins = BY_NAME["layernorm_fwd"].build("small")
    a = run_gpu(ops, ins, "stitched")
    b = run_gpu(ops, ins, "generated")
    assert_close(a[0], b[0], 1e-5, "hand-written vs generated")
    for wg in (64, 128):
        c = run_gpu(ops, ins, "generated", wg_size=wg)
        assert np.array_equal(b[0], c[0])
    with pytest.raises(FsError) as e:
        Plan(graphs.log_softmax((8, 64)), wg_size=100)
    assert e.value.status == binding.FS_ERR_INVALID


def test_tuner_times_generated_against_hand_written():
    announce("tune generated vs hand-written")
    ops, ins = BY_NAME["scaled_masked_softmax"].build("small")
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with Plan.tune(ops, dev_in, dev_out, trials=5) as plan:
        assert plan.info()["schedule"] == "row"
    torch.cuda.synchronize()
    (want,) = interp.run(ops, ins)
    assert_close(dev_out[0].to(torch.float64).cpu().numpy(), want, 1e-5, "tuned softmax")
    ops = graphs.log_softmax((257, 256))
    ins = inputs.normal_tensors([(257, 256)])
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with Plan.tune(ops, dev_in, dev_out, trials=5) as plan:
        assert "generated kernel" in plan.describe()
    torch.cuda.synchronize()
    (want,) = interp.run(ops, ins)
    assert_close(dev_out[0].to(torch.float64).cpu().numpy(), want, 1e-5, "tuned log_softmax")


def test_empty_and_unsupported_row_groups():
    announce("generated row edge cases")
    ops = graphs.log_softmax((0, 64))
    assert run_gpu(ops, inputs.normal_tensors([(0, 64)]))[0].size == 0
    with pytest.raises(FsError) as e:           # a reduction over an outer dim that keeps the dims between is not a row group
        g = graphs.Graph()
        x = g.parameter("x", "f32", (4, 8, 6, 64))
        g.output(g.reduce_sum(g.exp(x), 1))
        Plan(g.ops)
    assert e.value.status == binding.FS_ERR_UNSUPPORTED


@pytest.mark.parametrize("shape,dtype", [((4, 8192), "f32"), ((3, 4096), "f32"), ((2, 32768), "f32"), ((5, 5000), "f32"),
                                         ((3, 16384), "bf16"), ((7, 2052), "f16"), ((2, 3, 4100), "f32")])
def test_long_rows_go_to_a_team_of_wavefronts(shape, dtype):
    announce(f"generated team rows {shape} {dtype}")
    ops = graphs.rmsnorm(shape, dtype)
    with Plan(ops) as p:
        assert "CTA-S" in p.describe() and p.info()["lds_bytes"] > 0
    check_against_oracle(ops, inputs.normal_tensors([shape, shape[-1:]], dtype), what=f"rmsnorm team {shape} {dtype}")
    if dtype == "f32":
        ops = graphs.softmax_with_lse(shape)
        check_against_oracle(ops, inputs.normal_tensors([shape], scale=2.0), what=f"softmax+lse team {shape}")


@pytest.mark.parametrize("batch,m,n,k", [(7, 94, 94, 1), (3, 94, 94, 3), (5, 16, 64, 2), (4, 5, 10, 1), (2, 33, 128, 8), (1, 1, 94, 1)])
def test_dot_elementwise_reduce_dot_pattern(batch, m, n, k):
    """The motivating pattern: a tiny batched dot expands two small tensors into a tile, a
    softmax-like chain runs on it, a second dot contracts it again; four outputs."""
    announce(f"multi-interest pattern B={batch} m={m} n={n} k={k}")
    ops = graphs.multi_interest_pattern(batch, m, n, k)
    ins = inputs.multi_interest_pattern(batch, m, n, k)
    with Plan(ops) as p:
        info = p.info()
        assert info["schedule"] == "row" and info["n_kernels"] == 1 and "reduce x3" in p.describe()
    got, want = check_against_oracle(ops, ins, what="multi-interest pattern")
    assert [g.shape for g in got] == [(batch, m, n), (batch, m, n), (batch, m), (batch, m, 1)]
    per_op = run_gpu(ops, ins, "per_op")
    for a, b in zip(got, per_op):
        assert_close(a, b, 1e-5, "stitched vs per_op")


def test_dot_forms_the_generator_does_not_take():
    announce("dot limits")
    g = graphs.Graph()                               # contraction of 16: needs the matrix unit
    x = g.parameter("x", "f32", (4, 32, 16))
    y = g.parameter("y", "f32", (4, 16, 64))
    d = g.dot(x, y)
    g.output(g.subtract(d, g.row_broadcast(g.reduce_max(d, -1), d)))
    with pytest.raises(FsError) as e:
        Plan(g.ops)
    assert e.value.status == binding.FS_ERR_UNSUPPORTED and "contraction" in str(e.value)


# ---------------------------------------------------------------- streamed block template

STREAM_CASES = [
    ("log_softmax", (37, 128), "f32"), ("log_softmax", (33, 100), "f32"), ("log_softmax", (65, 30), "f32"), ("log_softmax", (7, 770), "f32"),
    ("rmsnorm", (37, 128), "bf16"), ("rmsnorm", (5, 768), "f16"), ("rmsnorm", (9, 1000), "f32"),
    ("ln_stats", (37, 768), "f32"), ("ln_stats", (64, 100), "f16"),
    ("softmax_lse", (2, 3, 5, 32), "f32"), ("softmax_lse", (33, 100), "f32"),
    ("l2", (3, 7, 64), "bf16"), ("sumsq", (65, 30), "f32"),
]


def _stream_group(kind, shape, dtype):
    if kind == "log_softmax":
        return graphs.log_softmax(shape, dtype), inputs.normal_tensors([shape], dtype, scale=3.0)
    if kind == "rmsnorm":
        return graphs.rmsnorm(shape, dtype), inputs.normal_tensors([shape, shape[-1:]], dtype)
    if kind == "ln_stats":
        return graphs.layernorm_fwd_with_stats(shape[0], shape[1], dtype), inputs.layernorm_fwd(shape[0], shape[1], dtype)
    if kind == "softmax_lse":
        return graphs.softmax_with_lse(shape), inputs.normal_tensors([shape], scale=2.0)
    if kind == "l2":
        return graphs.l2_normalize_scaled(shape, dtype), inputs.normal_tensors([shape, shape[:-1]], dtype)
    return graphs.row_sum_of_squares(shape), inputs.normal_tensors([shape])


@pytest.mark.parametrize("kind,shape,dtype", STREAM_CASES)
def test_streamed_template_on_small_rows(kind, shape, dtype):
    """A fixed grid selects the template that walks each row in passes (values kept in LDS row
    buffers laid out by Algorithm 4); forced here on rows that would fit registers."""
    announce(f"streamed {kind} {shape} {dtype}")
    ops, ins = _stream_group(kind, shape, dtype)
    with Plan(ops, grid=5) as p:
        assert "streamed in" in p.describe() and "cta_num=5" in p.describe()
    check_against_oracle(ops, ins, what=f"streamed {kind} {shape} {dtype}", grid=5)
    for wg in (64, 1024):
        check_against_oracle(ops, ins, what=f"streamed {kind} wg {wg}", grid=3, wg_size=wg)


def test_streamed_template_runs_the_motivating_pattern_and_benchmark_groups():
    announce("streamed pattern and configs")
    ops, ins = graphs.multi_interest_pattern(5), inputs.multi_interest_pattern(5)
    check_against_oracle(ops, ins, what="streamed pattern", grid=7)
    ops, ins = graphs.multi_interest_pattern(3, 16, 64, 3), inputs.multi_interest_pattern(3, 16, 64, 3)
    check_against_oracle(ops, ins, what="streamed pattern k=3", grid=2)
    for name in ("layernorm_fwd", "scaled_masked_softmax", "bias_gelu_residual_layernorm"):
        ops, ins = BY_NAME[name].build("small")
        check_against_oracle(ops, ins, "generated", what=f"streamed {name}", grid=16)


@pytest.mark.parametrize("kind,shape,dtype,expect", [
    ("log_softmax", (3, 40000), "f32", "1 taken over"),           # one 160 KB buffer: exp's argument takes over the input's
    ("log_softmax", (2, 131072), "f32", "re-read per pass"),     # vocabulary-sized rows: nothing fits, three passes over HBM
    ("softmax_lse", (3, 33000), "f32", "re-read per pass"),
    ("ln_stats", (3, 36000), "f32", "1 row buffers"),            # the centred row is kept, the input is read twice
    ("rmsnorm", (3, 40000), "bf16", "1 row buffers"),
    ("rmsnorm", (2, 70000), "f32", "re-read per pass"),
])
def test_rows_beyond_the_register_templates(kind, shape, dtype, expect):
    announce(f"long rows {kind} {shape} {dtype}")
    ops, ins = _stream_group(kind, shape, dtype)
    with Plan(ops) as p:
        assert "streamed in" in p.describe() and expect in p.describe(), p.describe()
        assert p.info()["lds_bytes"] <= 160 * 1024
    check_against_oracle(ops, ins, what=f"long rows {kind} {shape}")


def test_tuner_on_long_rows_times_the_streamed_template():
    announce("tune long rows")
    shape = (64, 8192)
    ops, ins = graphs.log_softmax(shape), inputs.normal_tensors([shape], scale=3.0)
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with Plan.tune(ops, dev_in, dev_out, trials=3) as plan:
        assert plan.info()["schedule"] == "row" and plan.tuned["us"] > 0
    torch.cuda.synchronize()
    (want,) = interp.run(ops, ins)
    assert_close(dev_out[0].to(torch.float64).cpu().numpy(), want, 1e-5, "tuned long rows")


# ---------------------------------------------------------------- column reductions packed with the row work

@pytest.mark.parametrize("rows,cols", [(517, 1024), (33, 768), (100, 2048), (7, 64), (1000, 100), (65, 30), (1, 256)])
def test_layernorm_backward_generated(rows, cols):
    """Config 5's group through the generator: row reductions, dx, and the two column
    reductions packed over the same register-resident rows (one partial row per workgroup,
    then the combine kernel)."""
    announce(f"generated LN backward {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops, "generated") as p:
        info = p.info()
        assert info["schedule"] == "row_col" and info["n_kernels"] == 2 and info["workspace_bytes"] > 0
        assert "column reduce x2" in p.describe()
    got, want = check_against_oracle(ops, ins, "generated", what=f"generated LN backward {rows}x{cols}")
    again = run_gpu(ops, ins, "generated", launches=3)          # partial rows are rewritten, not accumulated
    for a, b in zip(got, again):
        assert_close(a, b, 1e-6, "relaunch")
    for opts in (dict(wg_size=256, grid=7), dict(wg_size=1024, grid=3), dict(grid=1)):
        check_against_oracle(ops, ins, "generated", what=f"generated LN backward {opts}", **opts)


@pytest.mark.parametrize("rows,cols", [(517, 1024), (1, 256), (2, 64), (5, 768), (13, 2048), (1000, 100)])
def test_rows_requested_two_steps_ahead(rows, cols, monkeypatch):
    """The generated persistent kernels with three row buffers that take turns (FS_ROW_PREFETCH=2, the form the
    hand-written LayerNorm-backward kernel uses): trips of three steps, a partial last trip, fewer rows than
    buffers; plain row groups in the persistent form too."""
    announce(f"two rows ahead {rows}x{cols}")
    monkeypatch.setenv("FS_ROW_PREFETCH", "2")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    for opts in (dict(), dict(grid=1), dict(wg_size=64, grid=3)):
        check_against_oracle(ops, ins, "generated", what=f"two rows ahead, LN backward {opts}", **opts)
    ops, ins = graphs.encoder_tail_bwd(rows, cols), inputs.encoder_tail_bwd(rows, cols)
    check_against_oracle(ops, ins, "generated", what="two rows ahead, backward tail", grid=2)
    if cols <= 1024:
        ops, ins = graphs.rmsnorm((rows, cols), "bf16"), inputs.normal_tensors([(rows, cols), (cols,)], "bf16")
        check_against_oracle(ops, ins, what="two rows ahead, persistent row form", grid=2, rows_per_wave=1)


def test_layernorm_backward_beyond_the_hand_written_kernel_and_a_lone_column_sum():
    announce("generated LN backward 2048 cols, lone column sum")
    ops, ins = graphs.layernorm_bwd(64, 2048), inputs.layernorm_bwd(64, 2048)
    with Plan(ops) as p:                          # default mode: the hand-written kernel stops at 1024 columns
        assert "generated kernel" in p.describe()
    check_against_oracle(ops, ins, what="LN backward 2048")
    g = graphs.Graph()
    x = g.parameter("x", "f32", (301, 256))
    b = g.parameter("b", "f32", (256,))
    g.output(g.reduce_sum(g.exp(g.multiply(x, g.col_broadcast(b, x))), 0))
    xs = inputs.normal_tensors([(301, 256), (256,)], scale=0.5)
    check_against_oracle(g.ops, xs, what="lone column sum")
    for mode in ("stitched", "generated", "per_op"):        # sums over zero rows are zero
        out = run_gpu(graphs.layernorm_bwd(0, 64), inputs.layernorm_bwd(0, 64), mode)
        assert out[1].tolist() == [0.0] * 64 and out[2].tolist() == [0.0] * 64, mode


@pytest.mark.parametrize("rows,cols", [(130, 4096), (37, 3000), (20, 8192), (70, 2304), (3, 2052)])
def test_layernorm_backward_on_rows_of_several_wavefronts(rows, cols):
    """Rows beyond one wavefront's registers: a workgroup per row (team of wavefronts) loops over the
    rows, each lane keeps the running column sums of its own columns, one partial row per workgroup."""
    announce(f"LN backward, wavefront teams, {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row_col" and "CTA-S" in p.describe()
    got, want = check_against_oracle(ops, ins, what=f"team LN backward {rows}x{cols}")
    again = run_gpu(ops, ins, launches=3)
    for a, b in zip(got, again):
        assert np.array_equal(np.asarray(a), np.asarray(b)), "relaunch is bit-identical"
    for opts in (dict(grid=7), dict(grid=1), dict(grid=1000)):
        check_against_oracle(ops, ins, what=f"team LN backward {opts}", **opts)


@pytest.mark.parametrize("rows,cols,dtype", [(300, 96, "f32"), (40, 4096, "f32"), (33, 3000, "bf16"), (517, 1024, "bf16"), (2, 16384, "f32")])
def test_elementwise_chain_with_a_column_sum_and_no_row_reduction(rows, cols, dtype):
    announce(f"bias+GELU backward {rows}x{cols} {dtype}")
    ops = graphs.bias_gelu_bwd(rows, cols, dtype)
    ins = inputs.normal_tensors([(rows, cols), (rows, cols), (cols,)], dtype, seed_offset=77)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row_col" and p.info()["n_kernels"] == 2
    check_against_oracle(ops, ins, what=f"bias+GELU backward {rows}x{cols}")
    check_against_oracle(ops, ins, what=f"bias+GELU backward {rows}x{cols} grid 2", grid=2)


# rows whose length no vector width divides: two chunks and a bit, the edges of the lanes-per-row templates, of a wavefront and of
# a team; row counts that leave the last workgroup partly empty
@pytest.mark.parametrize("rows,cols", [(70, 9), (131, 17), (67, 33), (1000, 65), (301, 197), (41, 511), (41, 513), (29, 999), (9, 1025), (37, 2047), (3, 2049), (33, 3001),
                                       (5, 5001), (2, 32767)])
def test_ragged_rows_generated(rows, cols):
    announce(f"generated ragged rows {rows}x{cols}")
    for dtype in ("f32", "bf16"):
        check_against_oracle(graphs.log_softmax((rows, cols), dtype), inputs.normal_tensors([(rows, cols)], dtype, scale=3.0), what="log_softmax")
        check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype), inputs.bias_gelu_residual_layernorm(rows, cols, dtype), what="cfg4")
        check_against_oracle(graphs.bias_gelu_bwd(rows, cols, dtype), inputs.normal_tensors([(rows, cols), (rows, cols), (cols,)], dtype), what="bias+GELU backward")
        if cols <= 4096:
            check_against_oracle(graphs.sequence_pool((3, rows, cols), dtype=dtype, pool="both"), inputs.normal_tensors([(3, rows, cols)], dtype), what="pooled")
    if cols <= 5001:                      # (longer rows: their running sums fit no template)
        check_against_oracle(graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols), "generated", what="LN backward")
    if cols <= 1025:
        check_against_oracle(graphs.sequence_pool((300, 7, cols), with_row_work=True), inputs.normal_tensors([(300, 7, cols)]), what="pooled rows")
    # in the input's own buffer: a chunk that overlaps its neighbour must not read what the neighbour has already stored
    for ops, ins in [(graphs.log_softmax((rows, cols)), inputs.normal_tensors([(rows, cols)], scale=3.0)),
                     (graphs.gated_rows((rows, cols)), inputs.normal_tensors([(rows, cols), (rows,), (cols,)]))]:
        bufs, outs = to_device(ops, ins), alloc_outputs(ops)
        outs[0] = bufs[0]
        with Plan(ops) as p:
            p.launch(bufs, outs)
            torch.cuda.synchronize()
        for got, want in zip(outs, interp.run(ops, ins)):
            assert_close(got.to(torch.float64).cpu().numpy(), want, 1e-5, "in place")


@pytest.mark.parametrize("rows,cols", [(2047, 999), (2048, 999), (2050, 513), (2049, 2047), (2300, 1025)])
def test_column_reductions_over_many_ragged_rows(rows, cols):
    """Both sides of the line from which rows of no vector width take 16-byte chunks beside column sums, and the edges of the lane tiles beyond it."""
    announce(f"column reductions over ragged rows {rows}x{cols}")
    check_against_oracle(graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols), "generated", what="LN backward")
    for dtype in ("f32", "bf16"):
        ops, ins = graphs.bias_gelu_bwd(rows, cols, dtype), inputs.normal_tensors([(rows, cols), (rows, cols), (cols,)], dtype)
        got, want = run_gpu(ops, ins), interp.run(ops, ins)
        assert_close(got[0], want[0], TOLERANCE[dtype], f"bias+GELU backward {dtype}, full output")
        # a term of a column's sum is an fp32 chain of some ten roundings beside dy, 2^-22 of |dy| on average at most
        assert_close(got[1], want[1], TOLERANCE[dtype], f"bias+GELU backward {dtype}, column sums", slack=2.0 ** -22 * np.abs(ins[0]).sum(axis=0))
    for shape in ((23, rows // 23, cols), (91, 91, 513)):                                    # ... and per run of rows, both sides of its line
        check_against_oracle(graphs.sequence_pool(shape, pool="both"), inputs.normal_tensors([shape]), what="pooled")


# a team per row: sixteen rows to a workgroup below 256, down to four from there on within the bound on partial rows, sixteen
# again where there are rows enough; ordinary loads, and nontemporal ones beyond 128 MB (3 x 2300 x 5000 fp32)
@pytest.mark.parametrize("rows,cols,grid", [(255, 4096, 16), (256, 4096, 64), (257, 3001, 65), (300, 4096, 75), (1024, 2304, 227), (1030, 4096, 128), (2300, 5000, 144)])
def test_column_reductions_over_team_rows(rows, cols, grid):
    announce(f"column reductions over team rows {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops, "generated") as p:
        assert p.info()["workspace_bytes"] == 2 * grid * cols * 8, p.describe()
    check_against_oracle(ops, ins, "generated", what="LN backward")
    if rows <= 300:
        check_against_oracle(graphs.bias_gelu_bwd(rows, cols, "bf16"), inputs.normal_tensors([(rows, cols), (rows, cols), (cols,)], "bf16"), what="bias+GELU backward")


# rows beyond the register templates: register-resident in a full workgroup (up to 88 live elements per thread), or streamed; of any length
@pytest.mark.parametrize("rows,cols", [(5, 32769), (4, 36865), (9, 40001), (6, 45056), (5, 50257), (4, 65536), (7, 65537), (4, 90112), (4, 90113), (4, 100001),
                                       (3, 40001), (2, 131071)])
def test_long_rows_of_any_length(rows, cols):
    announce(f"generated long rows {rows}x{cols}")
    for dtype in ("f32", "bf16"):
        check_against_oracle(graphs.log_softmax((rows, cols), dtype), inputs.normal_tensors([(rows, cols)], dtype, scale=3.0), what="log_softmax")
        check_against_oracle(graphs.rmsnorm((rows, cols), dtype), inputs.normal_tensors([(rows, cols), (cols,)], dtype), what="rmsnorm")
        check_against_oracle(graphs.layernorm_fwd_with_stats(rows, cols, dtype), inputs.layernorm_fwd(rows, cols, dtype), what="layernorm with stats")
    check_against_oracle(graphs.softmax_with_lse((rows, cols)), inputs.normal_tensors([(rows, cols)], scale=2.0), what="softmax + lse")
    if cols <= 50257:
        check_against_oracle(graphs.bias_gelu_bwd(rows, cols), inputs.normal_tensors([(rows, cols), (rows, cols), (cols,)]), what="bias+GELU backward")
    # masked entries at -inf, and a row that holds nothing else but one value
    x = inputs.normal_tensors([(rows, cols)], scale=3.0)
    x[0][0, ::3] = -np.inf
    x[0][-1, 1:] = -np.inf
    with np.errstate(divide="ignore", invalid="ignore"):
        (want,) = interp.run(graphs.log_softmax((rows, cols)), x)
    got = run_gpu(graphs.log_softmax((rows, cols)), x)[0]
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    assert_close(np.where(np.isfinite(got), got, 0.0), np.where(np.isfinite(want), want, 0.0), 1e-5, "log_softmax with -inf")


@pytest.mark.parametrize("rows,cols,dtype", [(5, 90113, "f32"), (4, 94208, "f32"), (6, 114689, "f32"), (4, 118784, "f32"), (7, 118785, "f32"), (3, 131071, "f32"), (300, 122884, "f32"),
                                             (4, 151552, "f32"), (4, 57352, "bf16"), (5, 65537, "f16"), (270, 81928, "bf16"), (4, 131072, "f16"), (4, 163848, "bf16"), (4, 237569, "f16"),
                                             (4, 303104, "bf16")])
def test_rows_held_in_registers_and_lds(rows, cols, dtype):
    """Log-softmax of rows that are read once: edges of the chunks in registers, in LDS and read again, last chunks that are whole, begun or one
    element, more rows than workgroups at a time; infinities; bit-reproducible; no update in place, as in the streamed form."""
    announce(f"held rows {rows}x{cols} {dtype}")
    ops, ins = graphs.log_softmax((rows, cols), dtype), inputs.normal_tensors([(rows, cols)], dtype, scale=3.0)
    with Plan(ops) as p:
        assert "held in registers and LDS" in p.describe() and p.info()["lds_bytes"] <= 160 * 1024 and p.info()["n_kernels"] == 1
        dev = to_device(ops, ins)
        with pytest.raises(FsError):
            p.launch(dev, dev)
    got, _ = check_against_oracle(ops, ins, what="log_softmax held")
    assert np.array_equal(got[0], run_gpu(ops, ins, launches=2)[0])
    if rows <= 7:
        x = [np.array(a) for a in ins]
        x[0][0, ::3] = -np.inf
        x[0][-1, :-1] = -np.inf
        x[0][1, -1] = np.inf
        with np.errstate(divide="ignore", invalid="ignore"):
            (want,) = interp.run(ops, x)
        got = run_gpu(ops, x)[0]
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got == -np.inf, want == -np.inf)
        fine = np.isfinite(want)
        assert_close(np.where(fine, got, 0.0), np.where(fine, want, 0.0), TOLERANCE[dtype], "log_softmax with infinities")


def _held(shape, dtype, outputs, of=None):
    """Log-softmax "y", the row's maximum "max" and log-sum-exp "lse", those named; of: the input's shape, with dims of one for those it is repeated over."""
    g = graphs.Graph()
    x = g.parameter("x", dtype, of or shape)
    if dtype != "f32":
        x = g.convert(x, "f32")
    if of:
        x = g.broadcast(x, shape, 0)
    m = g.reduce_max(x, -1)
    c = g.subtract(x, g.row_broadcast(m, x))
    log_sum = g.log(g.reduce_sum(g.exp(c), -1))
    for name in outputs:
        if name == "y":
            y = g.subtract(c, g.row_broadcast(log_sum, c))
            g.output(y if dtype == "f32" else g.convert(y, dtype), "y")
        else:
            g.output(m if name == "max" else g.add(log_sum, m), name)
    return g.ops


@pytest.mark.parametrize("outputs", [("lse",), ("max", "lse"), ("y", "lse"), ("y", "max", "lse")], ids="+".join)
@pytest.mark.parametrize("rows,cols,dtype", [(5, 90113, "f32"), (4, 118784, "f32"), (7, 118785, "f32"), (4, 151552, "f32"), (4, 57352, "bf16"), (5, 65537, "f16"), (4, 237569, "bf16")])
def test_held_rows_with_row_outputs(rows, cols, dtype, outputs):
    """Log-sum-exp and maximum of held rows, alone and beside log-softmax: chunks in registers, in LDS and read again, whole and ragged; infinities."""
    announce(f"held rows {rows}x{cols} {dtype} {outputs}")
    ops, (x,) = _held((rows, cols), dtype, outputs), inputs.normal_tensors([(rows, cols)], dtype, scale=3.0)
    with Plan(ops) as p:
        assert "held in registers and LDS" in p.describe() and p.info()["n_kernels"] == 1
    check_against_oracle(ops, [x], what="held rows")
    x = np.array(x)
    x[0, ::3] = -np.inf
    x[1, -1] = np.inf
    x[2, :] = -np.inf
    x[-1, :-1] = -np.inf
    with np.errstate(divide="ignore", invalid="ignore"):
        want = interp.run(ops, [x])
    for name, a, b in zip(outputs, run_gpu(ops, [x]), want):
        fine = np.isfinite(b)
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~fine & ~np.isnan(b)], b[~fine & ~np.isnan(b)]), name
        assert_close(np.where(fine, a, 0.0), np.where(fine, b, 0.0), TOLERANCE[dtype], f"held rows with infinities, {name}")


@pytest.mark.parametrize("shape,of,dtype", [((4, 5, 100000), (4, 1, 100000), "f32"), ((2, 3, 2, 65537), (2, 1, 2, 65537), "bf16"), ((3, 2, 118785), (1, 2, 118785), "f32")])
def test_held_rows_of_a_repeated_input(shape, of, dtype):
    """Rows found by their coordinates: one row of the input is several of the group."""
    announce(f"held rows {shape} of {of} {dtype}")
    ops = _held(shape, dtype, ("y", "lse"), of)
    with Plan(ops) as p:
        assert "held in registers and LDS" in p.describe()
    check_against_oracle(ops, inputs.normal_tensors([of], dtype, scale=3.0), what="held rows of a repeated input")


def test_layernorm_backward_generated_at_full_size():
    announce("generated LN backward full size")
    ops, ins = BY_NAME["layernorm_bwd"].build("full")
    check_against_oracle(ops, ins, "generated", what="generated LN backward 32768x1024")


def test_persistent_register_form_of_plain_row_groups():
    """A fixed grid together with explicit lanes per row: the register templates loop over the rows
    and request the next row while the current one is worked on."""
    announce("persistent row form")
    for ops, ins, rpw in [(graphs.log_softmax((1030, 128)), inputs.normal_tensors([(1030, 128)], scale=3.0), 4),
                          (graphs.rmsnorm((203, 1024), "bf16"), inputs.normal_tensors([(203, 1024), (1024,)], "bf16"), 1),
                          (graphs.layernorm_fwd_with_stats(37, 100), inputs.layernorm_fwd(37, 100), 2)]:
        with Plan(ops, grid=5, rows_per_wave=rpw) as p:
            assert "persistent" in p.describe() and "cta_num=5" in p.describe()
        check_against_oracle(ops, ins, what="persistent row form", grid=5, rows_per_wave=rpw)
        check_against_oracle(ops, ins, what="persistent row form", grid=1000, rows_per_wave=rpw, wg_size=64)


@pytest.mark.parametrize("shape,dtype", [((2, 3, 64, 64), "f32"), ((5, 16, 16), "bf16"), ((33, 33), "f32"), ((2, 128, 128), "f16"), ((3, 100, 100), "f32")])
def test_causal_mask_inside_generated_kernels(shape, dtype):
    """causal_mask is an elementwise op that depends on the element's own indices: the row
    generator (softmax of causally masked scores) and the elementwise generator both take it."""
    announce(f"causal mask {shape} {dtype}")
    ops = graphs.causal_softmax(shape, dtype=dtype)
    got, _ = check_against_oracle(ops, inputs.normal_tensors([shape], dtype, scale=2.0), what=f"causal softmax {shape}")
    assert np.all(np.triu(got[0].reshape(-1, shape[-2], shape[-1])[0], 1) == 0.0)      # nothing right of the diagonal
    check_against_oracle(ops, inputs.normal_tensors([shape], dtype, scale=2.0), what="causal softmax streamed", grid=3)
    ops = graphs.causal_fill(shape, dtype=dtype)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "elementwise"
    check_against_oracle(ops, inputs.normal_tensors([shape], dtype), what=f"causal fill {shape}")


# ---------------------------------------------------------------- per-column values computed inside the group

@pytest.mark.parametrize("shape,dtype", [((300, 1024), "bf16"), ((4, 7, 96), "f32"), ((5, 40000), "f32"), ((3, 4096), "f16"), ((1000, 12), "f32")])
def test_scale_vector_computed_in_the_group(shape, dtype):
    """y = x * rsqrt(mean(x^2) + eps) * (1 + w): the [C]-shaped add is part of the group (done per row
    on the lanes' own columns), not a kernel of its own."""
    announce(f"rmsnorm with 1 + w, {shape} {dtype}")
    ops = graphs.rmsnorm_one_plus_weight(shape, dtype)
    ins = inputs.normal_tensors([shape, shape[-1:]], dtype, seed_offset=51)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row" and p.info()["n_kernels"] == 1
    check_against_oracle(ops, ins, what=f"rmsnorm 1+w {shape}")
    check_against_oracle(ops, ins, what=f"rmsnorm 1+w {shape} streamed", grid=3)
    if shape[-1] <= 2048:
        check_against_oracle(ops, ins, what=f"rmsnorm 1+w {shape} persistent", grid=2, rows_per_wave=1)


def test_per_column_arithmetic_without_any_reduction_and_its_limits():
    g = graphs.Graph()
    x = g.parameter("x", "f32", (257, 320))
    w = g.parameter("w", "f32", (320,))
    b = g.parameter("b", "f32", (320,))
    scale = g.multiply(g.add(g.tanh(w), g.constant(1.0)), b)             # [320], two ops deep
    g.output(g.add(g.multiply(x, g.col_broadcast(scale, x)), g.col_broadcast(b, x)))
    ins = inputs.normal_tensors([(257, 320), (320,), (320,)], seed_offset=52)
    announce("per-column arithmetic, no reduction")
    with Plan(g.ops) as p:
        assert p.info()["n_kernels"] == 1
    check_against_oracle(g.ops, ins, what="per-column arithmetic")
    # the per-column value as a group output is not one kernel's work here
    g.output(scale, "scale")
    with pytest.raises(FsError) as e:
        Plan(g.ops)
    assert e.value.status == binding.FS_ERR_UNSUPPORTED


@pytest.mark.parametrize("dtype,rows,cols", [("bf16", 203, 1024), ("f32", 37, 768), ("f16", 5, 4096)])
def test_exact_gelu_in_a_row_group(dtype, rows, cols):
    """Config 4's group with the erf form of GELU: no hand-written kernel matches, the generator takes it."""
    announce(f"bias + erf-GELU + residual + LayerNorm {dtype} {rows}x{cols}")
    ops = graphs.bias_gelu_erf_residual_layernorm(rows, cols, dtype)
    ins = inputs.bias_gelu_residual_layernorm(rows, cols, dtype)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row" and "generated kernel" in p.describe()
    check_against_oracle(ops, ins, what=f"erf-gelu ln {dtype} {rows}x{cols}")
    check_against_oracle(ops, ins, "per_op", what=f"erf-gelu ln per-op {dtype} {rows}x{cols}")


@pytest.mark.parametrize("shape,n_trailing,dtype", [((32, 8, 96), 2, "f32"), ((6, 4, 5, 32), 3, "bf16"), ((5, 7, 3, 50), 2, "f32"),
                                                    ((3, 64, 130), 2, "f16"), ((2, 40, 1000), 2, "f32")])
def test_normalisation_over_trailing_dims_spelled_as_reduction_chains(shape, n_trailing, dtype):
    """Statistics over the last two or three dims jointly, each a chain of reductions over one dim:
    the chains are merged into reductions over one merged dim and the group is one row kernel
    (rows of 768 to 40 000 elements: wavefront, team and streamed templates)."""
    announce(f"trailing-dim reduction chains {shape} {n_trailing} {dtype}")
    ops = graphs.norm_over_trailing_dims(shape, n_trailing, dtype)
    ins = inputs.normal_tensors([shape], dtype, seed_offset=51, scale=2.0)
    with Plan(ops) as p:
        assert p.info()["n_kernels"] == 1
    check_against_oracle(ops, ins, what=f"norm over trailing dims {shape}")


@pytest.mark.parametrize("shape,n_trailing,dtype", [((64, 3, 50), 2, "f32"), ((6, 4, 5, 32), 3, "f16"), ((300, 2, 2), 2, "bf16")])
def test_max_abs_over_trailing_dims(shape, n_trailing, dtype):
    announce(f"trailing-dim max chains {shape} {n_trailing} {dtype}")
    ops = graphs.max_abs_over_trailing_dims(shape, n_trailing, dtype)
    ins = inputs.normal_tensors([shape], dtype, seed_offset=52)
    check_against_oracle(ops, ins, what=f"max abs over trailing dims {shape}")


@pytest.mark.parametrize("shape,levels,dtype,with_row_work", [
    ((64, 50, 128), 1, "f32", False),        # one workgroup per run of 50 rows, results stored by the kernel
    ((300, 7, 96), 1, "f32", True),          # runs shorter than a workgroup's round of rows; a row reduction packed with it
    ((4, 3, 7, 96), 2, "f32", False),        # two reduction links: runs of 21 rows
    ((8, 600, 1024), 1, "f32", True),        # few long runs: several workgroups per run, partial rows, combine kernel
    ((3, 5000, 64), 1, "bf16", False),       # the same with 16-bit input
    ((37, 20, 4096), 1, "f32", False),       # rows of several wavefronts (a team per row), partial rows
    ((520, 5, 4096), 1, "f32", True),        # a team per row, one workgroup per run: results stored from registers
    ((2, 33, 2052), 1, "f32", True),
    ((1, 9, 40), 1, "f16", True),
    ((2101, 7, 96), 1, "f32", False),        # many short runs, nothing full-size written: a run per wavefront
    ((4099, 3, 128), 1, "bf16", False),      # (the last workgroup has idle wavefronts)
    ((2048, 50, 40), 1, "f16", False),
    ((2050, 5, 1024), 1, "f32", False),      # a row per wavefront
    ((2101, 7, 96), 1, "f32", True),         # the same runs with a full-size output: a run per workgroup
    ((70, 30, 13, 64), 2, "f32", False),     # 70 runs of 390 rows
])
def test_sums_over_the_innermost_row_dims(shape, levels, dtype, with_row_work):
    """[.., S, H] summed over S (sequence pooling): column sums per run of S consecutive rows, packed
    with the row work over the same register-resident rows."""
    announce(f"column sums per run of rows {shape} {levels} {dtype} {with_row_work}")
    ops = graphs.sequence_pool(shape, levels, dtype, with_row_work)
    ins = inputs.normal_tensors([shape], dtype, seed_offset=53)
    with Plan(ops) as p:
        assert p.info()["schedule"] == "row_col"
        if shape[0] > 2000 and not with_row_work:
            assert "one wavefront per run" in p.describe()
    check_against_oracle(ops, ins, what=f"sequence pool {shape}")


@pytest.mark.parametrize("shape,levels,dtype,with_row_work,pool", [
    ((64, 50, 128), 1, "f32", False, "max"), ((300, 7, 96), 1, "bf16", True, "both"), ((8, 600, 1024), 1, "f32", False, "both"),
    ((2101, 7, 96), 1, "f32", False, "max"), ((37, 20, 4096), 1, "f32", False, "max"), ((4, 3, 7, 96), 2, "f16", True, "both"),
])
def test_max_pooling_over_the_innermost_row_dims(shape, levels, dtype, with_row_work, pool):
    announce(f"column maxima per run of rows {shape} {levels} {dtype} {with_row_work} {pool}")
    ops = graphs.sequence_pool(shape, levels, dtype, with_row_work, pool)
    ins = inputs.normal_tensors([shape], dtype, seed_offset=54)
    check_against_oracle(ops, ins, what=f"max pool {shape}")


@pytest.mark.parametrize("shape,dtype", [((517, 1024), "f32"), ((33, 100), "bf16"), ((3, 7, 64), "f32"), ((20, 8192), "f32"), ((1, 40), "f16")])
def test_maximum_over_all_rows_beside_a_sum(shape, dtype):
    """Column maximum and column sum of the same value, packed: partial rows and the combine kernel
    carry each reduction's own operator."""
    announce(f"column max and sum {shape} {dtype}")
    g = graphs.Graph()
    x = g.parameter("x", dtype, shape)
    t = g.tanh(x if dtype == "f32" else g.convert(x, "f32"))
    mx, sm = t, t
    for _ in range(len(shape) - 1):
        mx, sm = g.reduce_max(mx, 0), g.reduce_sum(sm, 0)
    g.output(mx)
    g.output(sm)
    ins = inputs.normal_tensors([shape], dtype, seed_offset=55)
    with Plan(g.ops) as p:
        assert p.info()["schedule"] == "row_col" and p.info()["n_kernels"] == 2
    check_against_oracle(g.ops, ins, what=f"column max and sum {shape}")


# ---- column reductions beyond the register templates, and over a leading dim that keeps the inner dims
# (Section 4.2: column reductions have parallelisation needs of their own)

@pytest.mark.parametrize("rows,cols", [(37, 16384), (9, 20000), (130, 12288), (5, 24576)])
def test_layernorm_backward_on_streamed_rows(rows, cols):
    """Rows too long for the register templates: the streamed template walks a row in passes and keeps the
    column sums as double-precision running values per thread; partial rows, then the combine kernel."""
    announce(f"layernorm_bwd streamed {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops) as plan:
        assert plan.info()["schedule"] == "row_col" and "streamed" in plan.describe() and plan.info()["n_kernels"] == 2
    check_against_oracle(ops, ins, what=f"lnbwd streamed {rows}x{cols}")


@pytest.mark.parametrize("rows,cols,dtype,grid,two", [(50, 40000, "f32", 0, False), (33, 24000, "bf16", 7, True), (3, 50000, "f32", 0, False), (600, 18000, "f32", 0, True)])
def test_softmax_with_a_column_sum_and_a_column_maximum_on_streamed_rows(rows, cols, dtype, grid, two):
    announce(f"softmax + column sum/max streamed {rows}x{cols} {dtype} grid={grid}")
    g = graphs.Graph()
    x = g.parameter("x", dtype, (rows, cols))
    xf = g.convert(x, "f32") if dtype != "f32" else x
    zmax = g.reduce_max(xf, -1)
    e = g.exp(g.subtract(xf, g.row_broadcast(zmax, xf)))
    p = g.divide(e, g.row_broadcast(g.reduce_sum(e, -1), e))
    g.output(g.convert(p, dtype) if dtype != "f32" else p)
    g.output(g.reduce_sum(p, 0))           # how much of the probability mass each column gets
    if two:
        g.output(g.reduce_max(xf, 0))
    ins = inputs.normal_tensors([(rows, cols)], dtype, scale=2.0)
    with Plan(g.ops, grid=grid) as plan:
        assert "streamed" in plan.describe() and f"column reduce x{2 if two else 1}" in plan.describe()
    check_against_oracle(g.ops, ins, what="softmax + column reductions, streamed", grid=grid)


@pytest.mark.parametrize("shape,dtype", [((32, 50, 128), "f32"), ((7, 3, 5, 64), "bf16"), ((300, 2, 100), "f32"), ((4, 129, 130), "f32"), ((2, 8, 2052), "f16")])
def test_reduction_over_the_leading_dim_keeping_the_inner_dims(shape, dtype):
    """[B, S, H] -> [S, H]: the same memory read as [B, S*H] is a sum (and a maximum) over the rows of a matrix."""
    announce(f"leading-dim reduction {shape} {dtype}")
    g = graphs.Graph()
    x = g.parameter("x", dtype, shape)
    b = g.parameter("b", dtype, shape[1:])
    xf, bf = (g.convert(t, "f32") for t in (x, b)) if dtype != "f32" else (x, b)
    y = g.tanh(g.add(xf, g.broadcast(bf, shape, 1)))
    g.output(g.convert(y, dtype) if dtype != "f32" else y)
    g.output(g.reduce_sum(y, 0))
    g.output(g.reduce_max(xf, 0))
    ins = inputs.normal_tensors([shape, shape[1:]], dtype)
    with Plan(g.ops) as plan:
        assert plan.info()["schedule"] == "row_col"
    check_against_oracle(g.ops, ins, what=f"leading-dim reduction {shape}")


@pytest.mark.parametrize("rows,cols", [(256, 1284), (300, 1801), (257, 2048), (1030, 1535), (259, 30), (1025, 139), (260, 1023)])
@pytest.mark.parametrize("group", ["layernorm_bwd", "encoder_tail_bwd"])
def test_column_sums_meet_in_lds_and_in_teams(rows, cols, group):
    """The hand-over of running sums between the wavefronts of a workgroup (lanes per row of every width, whole and ragged chunks), and rows
    of more than twenty elements a lane: a team from 256 rows on; both against the oracle, and the same twice."""
    announce(f"column sums {group} {rows}x{cols}")
    ops, ins = getattr(graphs, group)(rows, cols), getattr(inputs, group)(rows, cols)
    with Plan(ops, "generated") as p:
        assert ("CTA-S" in p.describe()) == (cols > 1280)
    got, _ = check_against_oracle(ops, ins, "generated", what=f"{group} {rows}x{cols}")
    for a, b in zip(got, run_gpu(ops, ins, "generated", launches=2)):
        assert np.array_equal(a, b)
    for opts in (dict(wg_size=512), dict(wg_size=128, grid=5), dict(wg_size=64, grid=300)):      # a wavefront per row with other numbers of wavefronts
        check_against_oracle(ops, ins, "generated", what=f"{group} {rows}x{cols} {opts}", **opts)


@pytest.mark.parametrize("dtype,n", [("f32", 3), ("f32", 5), ("f32", 7), ("bf16", 2), ("bf16", 3), ("bf16", 4), ("f16", 7)])
@pytest.mark.parametrize("rows,cols", [(255, 1536), (256, 1284), (300, 1801), (259, 2048), (1030, 1540), (2051, 1035)])
def test_many_column_sums_over_rows_of_registers(rows, cols, dtype, n):
    """Two to seven sums beside a row reduction and a full output, as a wavefront's rows and as a team's: against the oracle, the same twice, and the same in
    place of the first input and from the static scratch memory."""
    announce(f"{n} column sums {rows}x{cols} {dtype}")
    ops, ins = product_with_column_sums(rows, cols, dtype, n), inputs.normal_tensors([(rows, cols)] * 2, dtype, scale=0.5)
    got, _ = check_against_oracle(ops, ins, what=f"{n} column sums {rows}x{cols} {dtype}")
    dev_in, outs = to_device(ops, ins), alloc_outputs(ops)
    with Plan(ops) as p:
        p.launch(dev_in, outs)
        launches = [p.launch] + ([p.launch_static] if p.info()["workspace_bytes"] <= 8 * 2**20 else [])
        for launch in launches:
            dev_in = to_device(ops, ins)
            outs = [dev_in[0]] + alloc_outputs(ops)[1:]
            launch(dev_in, outs)
            torch.cuda.synchronize()
            for a, b in zip(got, outs):
                assert np.array_equal(a, b.double().cpu().numpy())


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("cols", [2052, 4099, 9001, 16385, 32768, 32769, 45056, 50257, 53248, 57001, 90000])
def test_maximum_and_sum_of_exponentials_in_one_go(cols, dtype):
    """Log-softmax of rows for a team: rows of ordinary values, of values far apart in rising and falling order (every chunk has a new maximum, or
    none), with elements of -inf, of the type's lowest value, and with what makes the row NaN."""
    announce(f"log-softmax in one go {cols} {dtype}")
    rows = 9
    ops = graphs.log_softmax((rows, cols), dtype)
    x = inputs.normal_tensors([(rows, cols)], dtype, scale=3.0)[0]
    lowest = {"f32": -3.4028234663852886e38, "bf16": -3.3895313892515355e38, "f16": -65504.0}[dtype]
    x[1] = np.linspace(-200.0, 90.0, cols)
    x[2] = x[1][::-1]
    x[3, : cols // 2] = -np.inf                      # whole chunks of nothing
    x[4, ::3] = lowest
    x[5] = lowest                                    # a row of equal values: -log(cols)
    x[6, cols - 1] = 80.0                            # the maximum in the last, moved chunk
    x = inputs.round_to(x, dtype)
    with np.errstate(invalid="ignore"):
        want = interp.run(ops, [x])[0]
    got = run_gpu(ops, [x])[0]
    same = np.isinf(want)
    assert np.array_equal(same, np.isinf(got)) and np.array_equal(np.sign(want[same]), np.sign(got[same]))
    assert_close(np.where(same, 0.0, got), np.where(same, 0.0, want), TOLERANCE[dtype], f"log-softmax {cols} {dtype}")
    for bad in (np.full(cols, -np.inf), np.where(np.arange(cols) == cols // 3, np.inf, 0.0), np.where(np.arange(cols) == 5, np.nan, 0.0)):
        x[7] = bad
        out = run_gpu(ops, [inputs.round_to(x, dtype)])[0]
        assert np.isnan(out[7]).all() and np.array_equal(out[:7], got[:7])


@pytest.mark.parametrize("cols", [2052, 40001, 45056])
def test_maximum_and_sum_in_one_go_beside_other_outputs(cols):
    """The maximum, the sum and the difference as outputs too, an elementwise prologue, and a group that also reads the exponentials (apart)."""
    announce(f"log-sum-exp forms {cols}")
    for reads_exponentials in (False, True):
        g = graphs.Graph()
        x = g.parameter("x", "f32", (6, cols))
        b = g.parameter("b", "f32", (cols,))
        z = g.add(g.multiply(x, g.constant(0.5)), g.col_broadcast(b, x))
        m = g.reduce_max(z, 1)
        d = g.subtract(z, g.row_broadcast(m, z))
        e = g.exp(d)
        s = g.reduce_sum(e, 1)
        g.output(g.add(m, g.log(s)), "lse")
        g.output(m, "max")
        g.output(s, "sum")
        if reads_exponentials:
            g.output(g.divide(e, g.row_broadcast(s, e)), "softmax")
        ins = inputs.normal_tensors([(6, cols), (cols,)], scale=2.0)
        check_against_oracle(g.ops, ins, what=f"log-sum-exp {cols} {reads_exponentials}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cols", [64, 2048, 2052, 20000, 40001, 45056, 100001])
def test_sums_of_exponentials_of_infinite_rows(cols, dtype):
    """The maximum, the sum of exponentials and its logarithm of rows of -inf alone, with one finite element, with +inf and with NaN: the same in every form."""
    announce(f"log-sum-exp of infinite rows {cols} {dtype}")
    g = graphs.Graph()
    x = g.parameter("x", dtype, (6, cols))
    z = x if dtype == "f32" else g.convert(x, "f32")
    m = g.reduce_max(z, 1)
    s = g.reduce_sum(g.exp(g.subtract(z, g.row_broadcast(m, z))), 1)
    g.output(g.add(m, g.log(s)), "lse")
    g.output(m, "max")
    g.output(s, "sum")
    a = inputs.normal_tensors([(6, cols)], dtype)[0]
    a[0] = a[1] = -np.inf
    a[1, cols - 1] = 1.5
    a[2, cols // 2] = np.inf
    a[3, 1] = np.nan
    with np.errstate(invalid="ignore"):
        want = interp.run(g.ops, [a])
    lse, top, total = run_gpu(g.ops, [a])
    assert top[0] == -np.inf and top[1] == lse[1] == 1.5 and total[1] == 1.0 and top[2] == np.inf
    for v in (lse, total):
        assert np.isnan(v[[0, 2, 3]]).all(), v
        assert_close(v[4:], want[0 if v is lse else 2][4:], TOLERANCE[dtype], f"log-sum-exp {cols} {dtype}")


def test_maximum_and_sum_in_one_go_in_a_packed_launch():
    announce("log-softmax teams in a packed launch")
    shapes = [((30, 5000), "f32"), ((20, 3001), "f32"), ((7, 4099), "bf16")]
    lists = [graphs.log_softmax(s, d) for s, d in shapes]
    ins = [inputs.normal_tensors([s], d, scale=3.0) for s, d in shapes]
    plan, taken = Plan.packed([binding.marshal_ops(ops) for ops in lists])
    outs = [o for ops in lists for o in alloc_outputs(ops)]
    with plan:
        assert taken == [0, 1, 2]
        plan.launch([t for ops, x in zip(lists, ins) for t in to_device(ops, x)], outs)
        torch.cuda.synchronize()
    for got, ops, x, (_, d) in zip(outs, lists, ins, shapes):
        assert_close(got.double().cpu().numpy(), interp.run(ops, x)[0], TOLERANCE[d], "packed log-softmax")
