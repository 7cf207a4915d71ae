"""GPU parity: the stitched kernels (and the per-op baseline), called through the C ABI,
against the CPU oracle, element by element on the same seeded inputs.

Bar: |gpu - oracle| <= tol + tol*|oracle| with tol = 1e-5 for fp32 groups and 2e-2 for
fp16/bf16 groups (the oracle is fp64 and unrounded)."""
import sys

import numpy as np
import pytest
import torch

from oracle import interp
from paper_1911_11576_amd import FsError, Plan
from paper_1911_11576_amd import binding
from workloads import BY_NAME, CONFIGS, TOLERANCE, graphs, inputs

from gpu_util import (alloc_outputs, assert_close, check_against_oracle, run_gpu,
                      to_device, with_outputs)

pytestmark = pytest.mark.gpu


def announce(msg):
    # names the case on the real stderr before any GPU work, so that it survives a dead box
    sys.__stderr__.write(f"[gpu-case] {msg}\n")
    sys.__stderr__.flush()


@pytest.fixture(autouse=True)
def _need_gpu(device):
    yield


# ---------------------------------------------------------------- the five configs, small

@pytest.mark.parametrize("cfg", CONFIGS, ids=lambda c: c.name)
def test_config_small_stitched(cfg):
    announce(f"small stitched {cfg.name}")
    ops, ins = cfg.build("small")
    check_against_oracle(ops, ins, "stitched", what=cfg.name)


@pytest.mark.parametrize("cfg", CONFIGS, ids=lambda c: c.name)
def test_config_small_per_op_baseline(cfg):
    """The unfused baseline rounds every intermediate to its declared dtype, as the oracle's
    storage-rounding mode does; it is held to the group tolerance except for the fp32
    column sums over many rows, whose per-op rounding alone exceeds 1e-5 absolute."""
    announce(f"small per_op {cfg.name}")
    ops, ins = cfg.build("small")
    want = interp.run(ops, ins)
    got = run_gpu(ops, ins, "per_op")
    tol = TOLERANCE[cfg.dtype]
    for i, (a, b) in enumerate(zip(got, want)):
        t = 1e-3 if (cfg.name == "layernorm_bwd" and b.ndim == 1) else tol
        assert_close(a, b, t, f"{cfg.name} per_op output {i}")


@pytest.mark.parametrize("cfg", CONFIGS, ids=lambda c: c.name)
def test_stitched_equals_per_op_on_gpu(cfg):
    announce(f"stitched vs per_op {cfg.name}")
    ops, ins = cfg.build("small")
    a = run_gpu(ops, ins, "stitched")
    b = run_gpu(ops, ins, "per_op")
    tol = TOLERANCE[cfg.dtype]
    for i, (x, y) in enumerate(zip(a, b)):
        t = 1e-3 if (cfg.name == "layernorm_bwd" and x.ndim == 1) else 2 * tol
        assert_close(x, y, t, f"{cfg.name} stitched vs per_op output {i}")


# ---------------------------------------------------------------- row schedule: shapes

@pytest.mark.parametrize("rows,cols", [(1, 4), (3, 8), (5, 24), (37, 100), (9, 256), (64, 768), (37, 1000),
                                       (11, 1536), (6, 2048), (130, 32)])
def test_layernorm_shapes_f32(rows, cols):
    announce(f"layernorm f32 {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols), inputs.layernorm_fwd(rows, cols), what=f"ln {rows}x{cols}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("rows,cols", [(1, 8), (7, 40), (33, 512), (19, 1024), (5, 2048)])
def test_layernorm_shapes_16bit(rows, cols, dtype):
    announce(f"layernorm {dtype} {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols, dtype), inputs.layernorm_fwd(rows, cols, dtype),
                         what=f"ln {dtype} {rows}x{cols}")


# The group with the GELU prologue has two stitched forms: the default is the generated kernel
# (mode "stitched"), the hand-written kernels serve mode "prebuilt"
GELU_LN_MODES = ["stitched", "prebuilt"]


@pytest.mark.parametrize("mode", GELU_LN_MODES)
@pytest.mark.parametrize("dtype,rows,cols", [("bf16", 203, 1024), ("f16", 33, 768), ("f32", 65, 1024),
                                             ("bf16", 4, 2048), ("f32", 3, 8)])
def test_bias_gelu_residual_layernorm_shapes(dtype, rows, cols, mode):
    announce(f"bias+gelu+res+ln {dtype} {rows}x{cols} {mode}")
    check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype),
                         inputs.bias_gelu_residual_layernorm(rows, cols, dtype), mode, what=f"cfg4 {dtype} {rows}x{cols}")


@pytest.mark.parametrize("shape", [(1, 4), (3, 12), (1030, 128), (77, 64), (5, 1000), (9, 2048), (130, 32), (33, 16)])
@pytest.mark.parametrize("mask", ["full", "none"])
def test_softmax_shapes_f32(shape, mask):
    announce(f"softmax f32 {shape} mask={mask}")
    check_against_oracle(graphs.scaled_masked_softmax(shape, 0.125, mask),
                         inputs.scaled_masked_softmax(shape, mask), what=f"softmax {shape} {mask}")


@pytest.mark.parametrize("shape", [(3, 4, 16, 16), (2, 3, 5, 128), (4, 2, 7, 64)])
def test_softmax_key_padding_mask(shape):
    announce(f"softmax key_padding {shape}")
    check_against_oracle(graphs.scaled_masked_softmax(shape, 0.125, "key_padding"),
                         inputs.scaled_masked_softmax(shape, "key_padding"), what=f"softmax kp {shape}")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_softmax_16bit(dtype):
    announce(f"softmax {dtype}")
    shape = (67, 128)
    # a mask of -1e4 is not representable in f16/bf16 exactly; the generator rounds it
    check_against_oracle(graphs.scaled_masked_softmax(shape, 0.125, "full", dtype),
                         inputs.scaled_masked_softmax(shape, "full", dtype), what=f"softmax {dtype}")


def test_softmax_fully_masked_rows_and_large_values():
    announce("softmax degenerate rows")
    shape = (8, 128)
    ops = graphs.scaled_masked_softmax(shape, 0.125, "full")
    s, m = inputs.scaled_masked_softmax(shape, "full")
    m[0, :] = -1e4          # fully padded row: still a softmax of the shifted row
    s[1, :] = 3.0           # constant row
    s[2, :] = 600.0         # exp would overflow without the max subtraction
    s[3, 5] = -700.0
    check_against_oracle(ops, [s, m], what="softmax degenerate")


# ---------------------------------------------------------------- row schedule, block-composed form

@pytest.mark.parametrize("rows,cols", [(3, 770), (5, 4096), (2, 3001), (7, 10007), (2, 16384), (1, 40000), (9, 1), (4, 3)])
def test_layernorm_long_or_unaligned_rows_f32(rows, cols):
    announce(f"layernorm block form f32 {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols), inputs.layernorm_fwd(rows, cols), what=f"ln block {rows}x{cols}")


@pytest.mark.parametrize("mode", GELU_LN_MODES)
@pytest.mark.parametrize("dtype,rows,cols", [("bf16", 5, 4096), ("f16", 3, 3001), ("bf16", 2, 12), ("f16", 6, 8200)])
def test_gelu_layernorm_long_or_unaligned_rows_16bit(dtype, rows, cols, mode):
    announce(f"bias+gelu+res+ln block form {dtype} {rows}x{cols} {mode}")
    check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype),
                         inputs.bias_gelu_residual_layernorm(rows, cols, dtype), mode, what=f"cfg4 block {dtype} {rows}x{cols}")


@pytest.mark.parametrize("shape,mask", [((5, 94), "full"), ((3, 4100), "full"), ((6, 2049), "none"), ((2, 3, 94, 94), "key_padding"),
                                        ((2, 2, 5, 4096), "key_padding"), ((4, 1), "full")])
def test_softmax_long_or_unaligned_rows(shape, mask):
    announce(f"softmax block form {shape} {mask}")
    check_against_oracle(graphs.scaled_masked_softmax(shape, 0.125, mask),
                         inputs.scaled_masked_softmax(shape, mask), what=f"softmax block {shape} {mask}")


# rows whose length is no multiple of the 16-byte vector: one vector and a bit, the edges of the lane tiles (8 .. 64 lanes, 1 .. 8
# vectors), of a wavefront (2048) and of a team; row counts that leave the last workgroup partly empty
RAGGED = [(5, 9), (70, 31), (131, 33), (67, 129), (1000, 197), (37, 255), (41, 513), (29, 999), (9, 1025), (5, 2047), (3, 2049), (4, 3001), (2, 8193),
          (2, 32767)]


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("rows,cols", RAGGED)
def test_ragged_rows(dtype, rows, cols):
    announce(f"ragged rows {dtype} {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols, dtype), inputs.layernorm_fwd(rows, cols, dtype), what=f"ln ragged {rows}x{cols}")
    check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype), inputs.bias_gelu_residual_layernorm(rows, cols, dtype), "prebuilt",
                         what=f"cfg4 ragged {rows}x{cols}")
    for mask in ("none", "full"):
        check_against_oracle(graphs.scaled_masked_softmax((rows, cols), 0.125, mask, dtype), inputs.scaled_masked_softmax((rows, cols), mask, dtype),
                             what=f"softmax ragged {rows}x{cols} {mask}")
    shape = (2, 2, rows, cols)
    ops, ins = graphs.scaled_masked_softmax(shape, 0.125, "key_padding", dtype), inputs.scaled_masked_softmax(shape, "key_padding", dtype)
    ref, _ = check_against_oracle(ops, ins, what=f"softmax ragged {shape}")
    for opts in (dict(grid=3), dict(wg_size=128), dict(rows_per_wave=4, grid=2)):       # several trips of the row loop, other tiles
        got, _ = check_against_oracle(ops, ins, what=f"softmax ragged {shape} {opts}", **opts)
        assert cols > 2048 or np.array_equal(got[0], ref[0])                             # (a team's size decides the order of its sums)


@pytest.mark.parametrize("opts", [dict(wg_size=1024), dict(wg_size=576), dict(rows_per_wave=16), dict(wg_size=128, grid=2)], ids=str)
@pytest.mark.parametrize("rows,cols", [(37, 11), (70, 333), (9, 2047)])
def test_ragged_rows_under_options_of_other_forms(rows, cols, opts):
    """Launch options that the wavefront form does not take (recorded for the block form, say): a team, most of it idle, or a row block."""
    announce(f"ragged rows {rows}x{cols} {opts}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols, "f16"), inputs.layernorm_fwd(rows, cols, "f16"), what="ln", **opts)
    check_against_oracle(graphs.scaled_masked_softmax((rows, cols), 0.125, "full"), inputs.scaled_masked_softmax((rows, cols), "full"), what="softmax", **opts)


# more wavefronts than start at once (16 per CU): gamma and beta requested with the row, not late
@pytest.mark.parametrize("dtype,rows,cols", [("f32", 4099, 1024), ("f32", 4097, 1000), ("f32", 16391, 200), ("bf16", 4099, 1024), ("f16", 4097, 1000), ("bf16", 33000, 136)])
def test_layernorm_of_many_wavefronts(dtype, rows, cols):
    announce(f"layernorm of many wavefronts {dtype} {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols, dtype), inputs.layernorm_fwd(rows, cols, dtype), what=f"ln {rows}x{cols}")
    check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype), inputs.bias_gelu_residual_layernorm(rows, cols, dtype), "prebuilt",
                         what=f"cfg4 {rows}x{cols}")


@pytest.mark.parametrize("rows,cols", [(3, 2052), (5, 5000), (4, 8192), (2, 32768), (3, 20480)])
def test_layernorm_team_form_f32(rows, cols):
    announce(f"layernorm team form f32 {rows}x{cols}")
    check_against_oracle(graphs.layernorm_fwd(rows, cols), inputs.layernorm_fwd(rows, cols), what=f"ln team {rows}x{cols}")


@pytest.mark.parametrize("dtype,cols", [("f32", 64), ("f32", 768), ("f32", 333), ("f32", 2048), ("f32", 4096), ("f32", 3001), ("bf16", 1024), ("bf16", 999), ("bf16", 5003)])
def test_layernorm_variance_beyond_and_below_the_normal_range(dtype, cols):
    """A variance that overflows fp32 gives 1 / sqrt(inf) = 0, that is beta; a subnormal one (eps = 0) still normalises."""
    announce(f"layernorm variance limits {dtype} {cols}")
    ops, ins = graphs.layernorm_fwd(7, cols, dtype, eps=0.0), inputs.layernorm_fwd(7, cols, dtype)
    x = ins[0]
    x[1::2] = np.where(np.arange(cols) % 2, 1.0, -1.0) * 2.0 ** 65             # squares of 2^130
    x[2] *= 2.0 ** -65                                                          # squares around 2^-130, known to 2^-149: 1e-6 of the variance
    (want,) = interp.run(ops, ins)
    for mode in ("stitched", "generated"):
        (got,) = run_gpu(ops, ins, mode)
        assert np.array_equal(got[1::2], np.broadcast_to(ins[2], got[1::2].shape)), mode
        assert_close(got[0::2], want[0::2], TOLERANCE[dtype], f"LN {mode}")


@pytest.mark.parametrize("mode", GELU_LN_MODES)
@pytest.mark.parametrize("dtype,rows,cols", [("bf16", 3, 2056), ("f16", 5, 4096), ("bf16", 2, 32768), ("f16", 3, 12288)])
def test_gelu_layernorm_team_form_16bit(dtype, rows, cols, mode):
    announce(f"bias+gelu+res+ln team form {dtype} {rows}x{cols} {mode}")
    check_against_oracle(graphs.bias_gelu_residual_layernorm(rows, cols, dtype),
                         inputs.bias_gelu_residual_layernorm(rows, cols, dtype), mode, what=f"cfg4 team {dtype} {rows}x{cols}")


@pytest.mark.parametrize("shape,mask", [((5, 4096), "full"), ((2, 2, 3, 8192), "key_padding"), ((3, 16000), "none")])
def test_softmax_team_form(shape, mask):
    announce(f"softmax team form {shape} {mask}")
    check_against_oracle(graphs.scaled_masked_softmax(shape, 0.125, mask),
                         inputs.scaled_masked_softmax(shape, mask), what=f"softmax team {shape} {mask}")


@pytest.mark.parametrize("rows", [512, 513])
def test_team_of_any_number_of_wavefronts(rows):
    """Whole vectors: teams of a power of two up to 512 rows, beyond it of as many wavefronts as the row keeps busy."""
    announce(f"team form, odd teams {rows}")
    ops, ins = graphs.layernorm_fwd(rows, 5000, "bf16"), inputs.layernorm_fwd(rows, 5000, "bf16")
    with Plan(ops) as plan:
        assert ("cta_size=512" if rows == 512 else "cta_size=320") in plan.describe()
    check_against_oracle(ops, ins, what=f"ln team {rows}x5000")
    check_against_oracle(graphs.scaled_masked_softmax((rows, 4104), 0.125, "full", "f16"), inputs.scaled_masked_softmax((rows, 4104), "full", "f16"), what=f"softmax team {rows}x4104")


def test_team_form_launch_options():
    announce("row team form options")
    ops, ins = graphs.layernorm_fwd(77, 8192), inputs.layernorm_fwd(77, 8192)
    ref = run_gpu(ops, ins)
    for opts in (dict(wg_size=256), dict(wg_size=1024), dict(grid=5), dict(wg_size=512, grid=3)):
        got = run_gpu(ops, ins, **opts)
        assert_close(got[0], ref[0], 1e-6, f"team form {opts}")


def test_block_form_launch_options():
    announce("row block form options")
    ops, ins = graphs.layernorm_fwd(300, 4096), inputs.layernorm_fwd(300, 4096)
    ref = run_gpu(ops, ins)
    for opts in (dict(wg_size=64), dict(wg_size=1024), dict(grid=7)):
        got = run_gpu(ops, ins, **opts)
        assert_close(got[0], ref[0], 1e-6, f"block form {opts}")


# ---------------------------------------------------------------- launch parameters

@pytest.mark.parametrize("opts", [dict(wg_size=64), dict(wg_size=512), dict(rows_per_wave=1), dict(rows_per_wave=2),
                                  dict(grid=7), dict(wg_size=128, rows_per_wave=4, grid=3)])
def test_row_schedule_launch_options_do_not_change_results(opts):
    announce(f"row options {opts}")
    shape = (1030, 128)
    ops, ins = graphs.scaled_masked_softmax(shape, 0.125, "full"), inputs.scaled_masked_softmax(shape, "full")
    ref = run_gpu(ops, ins)
    got = run_gpu(ops, ins, **opts)
    assert np.array_equal(ref[0], got[0])
    ops, ins = graphs.layernorm_fwd(517, 768), inputs.layernorm_fwd(517, 768)
    ref = run_gpu(ops, ins)
    got = run_gpu(ops, ins, **opts)
    assert np.array_equal(ref[0], got[0])


# ---------------------------------------------------------------- LayerNorm backward

# both forms of the group: the hand-written row kernel + combine kernel (default) and the generated
# row kernel + combine kernel (mode "generated")
LNBWD_MODES = ["stitched", "generated"]


@pytest.mark.parametrize("mode", LNBWD_MODES)
@pytest.mark.parametrize("rows,cols", [(1, 4), (5, 64), (517, 1024), (4099, 1000), (33, 768), (700, 256)])
def test_layernorm_bwd_shapes(rows, cols, mode):
    announce(f"layernorm_bwd {rows}x{cols} {mode}")
    check_against_oracle(graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols), mode, what=f"lnbwd {rows}x{cols}")


@pytest.mark.parametrize("rows,cols", [(1025, 128), (1030, 260), (1100, 772), (4096, 1024), (4097, 1024), (12287, 128), (12288, 128), (12291, 252), (12290, 4)])
def test_layernorm_bwd_through_the_caches(rows, cols):
    """A wavefront to a row, up to 48 MiB with ordinary loads: one to four vectors a lane, whole sets of lanes and not, the largest such group and the next; four
    and eight wavefronts to a workgroup (the sums of 12288 terms have the room that their roundings take, 4 * 2^-24 * sqrt(sum t^2) < 3e-5)."""
    announce(f"layernorm_bwd cached {rows}x{cols}")
    if rows > 12000:
        ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
        for k, (got, want) in enumerate(zip(run_gpu(ops, ins), interp.run(ops, ins))):
            assert_close(got, want, 1e-5, f"lnbwd {rows}x{cols} output {k}", 3e-5 if want.ndim == 1 else None)
        return
    check_against_oracle(graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols), what=f"lnbwd {rows}x{cols}")


PARTIAL_ROWS = (1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 47, 48, 64, 65, 80, 128, 129, 256, 257)


@pytest.mark.parametrize("mode,rows,cols,groups", [("stitched", 2048, 520, PARTIAL_ROWS + (272, 273, 400, 511, 512)), ("generated", 2048, 520, PARTIAL_ROWS),
                                                   ("generated", 520, 6200, (4, 16, 17, 32, 33, 65, 128, 129, 257, 513))])
def test_any_number_of_partial_rows_is_added_up(mode, rows, cols, groups):
    """The second kernel reads up to sixteen partial rows a thread at a time, eight where it has many blocks, the rest in batches of half as many down to one, and has
    a form for four rows and for sixteen: the edges of them all, through the workgroups that a launch option names."""
    announce(f"partial rows {mode} {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    want = interp.run(ops, ins)
    for n in groups:
        with Plan(ops, mode, grid=n) as p:
            assert f" {n} partial rows" in p.describe()
        for k, (a, b) in enumerate(zip(run_gpu(ops, ins, mode, grid=n), want)):
            assert_close(a, b, 1e-5, f"{n} partial rows, output {k}")


@pytest.mark.parametrize("rows,cols,threads,keep", [
    (21001, 200, 512, (0, 1, 2)), (32769, 132, 512, (0, 1, 2)), (18001, 244, 512, (0, 1, 2)), (24601, 228, 256, (0, 1, 2)), (16500, 256, 256, (0, 1, 2)),
    (9001, 500, 256, (0, 1, 2)), (8200, 512, 256, (0, 1, 2)), (5701, 740, 256, (0, 1, 2)), (5500, 768, 256, (0, 1, 2)), (4301, 1000, 256, (0, 1, 2)),
    (12290, 128, 512, (0,)), (12297, 128, 512, (1, 2)), (12289, 220, 512, (2,)), (12288, 64, 512, (0, 1)), (1500, 1000, 256, (0,)), (1501, 768, 256, (2,))])
def test_layernorm_bwd_nontemporally(rows, cols, threads, keep):
    """A wavefront to a row with nontemporal loads: all outputs beyond 48 MiB and some of them at any size, one to four vectors a lane, whole sets of lanes and
    not, four and eight wavefronts to a workgroup; bit-reproducible.  Column sums have the room of a sum of fp32 terms t, each with the rounding of the chain
    that made it: 4 * 2^-24 * sqrt(sum t^2)."""
    announce(f"layernorm_bwd nontemporal {rows}x{cols} {keep}")
    assert len(keep) < 3 or 12 * rows * cols > 48 << 20
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    dy, x, _, mean, rstd = (np.asarray(a, dtype=np.float64) for a in ins)
    terms = [dy * (x - mean.reshape(-1, 1)) * rstd.reshape(-1, 1), dy]
    slack = [None] + [4.0 * 2.0 ** -24 * np.sqrt((t * t).sum(axis=0)) for t in terms]
    ops = with_outputs(ops, keep)
    ins = [ins[["dy", "x", "gamma", "mean", "rstd"].index(op.name)] for op in ops if op.kind == "parameter"]
    with Plan(ops) as p:
        assert "hand-written" in p.describe() and f"cta_size={threads}" in p.describe()
    got, want = run_gpu(ops, ins), interp.run(ops, ins)
    for k, a, b in zip(keep, got, want):
        assert_close(a, b, 1e-5, f"lnbwd {rows}x{cols} output {k}", slack[k])
    for a, b in zip(got, run_gpu(ops, ins, launches=2)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("rows,cols", [(256, 4), (257, 5), (300, 31), (1024, 33), (401, 255), (400, 257), (999, 511), (1024, 1024), (513, 1025), (301, 1027), (260, 2048), (450, 2049), (258, 4095), (256, 4096)])
def test_layernorm_bwd_in_one_launch(rows, cols):
    """Few rows: the row path and strips of columns as workgroups of one launch; edges of vectors, strips, wavefronts and teams, the rule's
    corners; bit-reproducible.  Where the generated kernel is the only other form, an update in place is taken as by that one."""
    announce(f"layernorm_bwd in one launch {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops) as p:
        assert p.info()["n_kernels"] == 1 and p.info()["workspace_bytes"] == 0 and "strip of" in p.describe()
    got, want = check_against_oracle(ops, ins, what=f"lnbwd {rows}x{cols}")
    for a, b in zip(got, run_gpu(ops, ins, launches=2)):
        assert np.array_equal(a, b)
    dev_in, outs = to_device(ops, ins), alloc_outputs(ops)
    with Plan(ops) as p:
        if cols % 4 == 0 and cols <= 1024:
            with pytest.raises(FsError):
                p.launch(dev_in, [dev_in[0]] + outs[1:])
            return
        p.launch(dev_in, outs)
        for launch in (p.launch_static, p.launch):
            dev_in = to_device(ops, ins)
            launch(dev_in, [dev_in[0]] + outs[1:])
            torch.cuda.synchronize()
            for a, b in zip([dev_in[0]] + outs[1:], want):
                assert_close(a.double().cpu().numpy(), b, 1e-5, f"lnbwd in place {rows}x{cols}")


@pytest.mark.parametrize("rows,cols", [(1025, 129), (1100, 255), (2051, 257), (1030, 513), (4099, 767), (1500, 769), (1033, 1021), (1040, 1022), (1027, 1023)])
def test_layernorm_bwd_rows_of_no_whole_vectors(rows, cols):
    """The hand-written rows kernel at element alignment: one to three elements over, one vector over a set of 64, trips of every length;
    bit-reproducible, updates in place as by the generated form, the prebuilt mode as before."""
    announce(f"layernorm_bwd ragged {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    with Plan(ops) as p:
        assert "hand-written" in p.describe() and p.info()["n_kernels"] == 2
    with pytest.raises(FsError):
        Plan(ops, "prebuilt")
    got, want = check_against_oracle(ops, ins, what=f"lnbwd {rows}x{cols}")
    for a, b in zip(got, run_gpu(ops, ins, launches=2)):
        assert np.array_equal(a, b)
    dev_in, outs = to_device(ops, ins), alloc_outputs(ops)
    with Plan(ops) as p:
        p.launch(dev_in, outs)
        for launch in (p.launch_static, p.launch, p.launch_static):
            dev_in = to_device(ops, ins)
            launch(dev_in, [dev_in[0]] + outs[1:])
            torch.cuda.synchronize()
            for a, b in zip([dev_in[0]] + outs[1:], want):
                assert_close(a.double().cpu().numpy(), b, 1e-5, f"lnbwd in place {rows}x{cols}")


@pytest.mark.parametrize("rows,cols", [(1025, 1025), (1026, 1028), (1100, 1537), (1500, 1536), (2049, 2048), (1030, 2049), (1031, 3072), (1200, 3075), (1027, 4095), (1300, 4096),
                                       (4099, 1100), (7300, 1540), (12001, 1280), (7203, 2048), (4703, 3072), (3502, 4096)])
def test_layernorm_bwd_with_teams_of_wavefronts(rows, cols):
    """Two and four wavefronts to a row: edges of the lanes' vectors, rows at element alignment, trips of odd length, workgroups whose second team has no row
    left, nontemporal loads (beyond 160 MiB, every number of vectors a lane); bit-reproducible, updates in place of dy and of x as by the generated form, the prebuilt mode as before.
    dgamma over more than 2048 rows has the room of a sum of so many fp32 terms t, each with the rounding of the chain that made it: 4 * 2^-24 * sqrt(sum t^2)."""
    announce(f"layernorm_bwd teams {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    dy, x, _, mean, rstd = (np.asarray(a, dtype=np.float64) for a in ins)
    terms = dy * (x - mean.reshape(-1, 1)) * rstd.reshape(-1, 1)
    slack = [None, 4.0 * 2.0 ** -24 * np.sqrt((terms * terms).sum(axis=0)) if rows > 2048 else None, None]
    assert [op.shape for op in ops if op.kind == "output"] == [(rows, cols), (cols,), (cols,)]
    with Plan(ops) as p:
        assert "wavefronts to a row" in p.describe() and p.info()["n_kernels"] == 2
    with pytest.raises(FsError):
        Plan(ops, "prebuilt")
    got, want = run_gpu(ops, ins), interp.run(ops, ins)
    for i in range(3):
        assert_close(got[i], want[i], 1e-5, f"lnbwd {rows}x{cols} output {i}", slack[i])
    for a, b in zip(got, run_gpu(ops, ins, launches=2)):
        assert np.array_equal(a, b)
    with Plan(ops) as p:
        launches = [p.launch] + ([p.launch_static] if p.info()["workspace_bytes"] <= 8 << 20 else [])
        for k in (0, 1):
            for launch in launches:
                dev_in, outs = to_device(ops, ins), alloc_outputs(ops)
                outs[0] = dev_in[k]
                launch(dev_in, outs)
                torch.cuda.synchronize()
                assert all(np.array_equal(a.double().cpu().numpy(), b) for a, b in zip(outs, got)), (k, launch.__name__)


@pytest.mark.parametrize("rows,cols", [(300, 31), (700, 1600), (301, 1027), (256, 4095), (1027, 1023)])
def test_layernorm_bwd_in_place_beside_other_launches(rows, cols):
    """Updates in place need no more than the plan reports: bit for bit what a launch with buffers of its own gives, in dy's buffer and in x's, captured after
    one plain launch, and, where the plan owns no workspace, several at once on two streams."""
    announce(f"layernorm_bwd in place, captured and overlapping {rows}x{cols}")
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    names = [op.name for op in ops if op.kind == "parameter"]
    dx = [op.shape for op in ops if op.kind == "output"].index((rows, cols))
    with Plan(ops) as p:
        free = p.info()["workspace_bytes"] == 0
        assert free == (rows <= 1024) and "in place of dy or x" in p.describe()
        want = alloc_outputs(ops)
        p.launch(to_device(ops, ins), want)

        def buffers(name):
            dev_in, outs = to_device(ops, ins), alloc_outputs(ops)
            outs[dx] = dev_in[names.index(name)]
            return dev_in, outs
        for name in ("dy", "x"):
            dev_in, outs = buffers(name)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                p.launch(dev_in, outs)
            for _ in range(2):
                for t, s in zip(dev_in, to_device(ops, ins)):
                    t.copy_(s)
                graph.replay()
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(outs, want)), name
        sets = [buffers(("dy", "x")[k % 2]) for k in range(8)]
        streams = [torch.cuda.Stream() for _ in range(2 if free else 1)]
        torch.cuda.synchronize()
        for k, (dev_in, outs) in enumerate(sets):
            p.launch(dev_in, outs, streams[k % len(streams)].cuda_stream)
        torch.cuda.synchronize()
        for _, outs in sets:
            assert all(torch.equal(a, b) for a, b in zip(outs, want))


@pytest.mark.parametrize("mode", LNBWD_MODES)
@pytest.mark.parametrize("opts", [dict(grid=1), dict(grid=3, wg_size=64), dict(grid=100, wg_size=256), dict(grid=1024)])
def test_layernorm_bwd_launch_options(opts, mode):
    announce(f"layernorm_bwd options {opts} {mode}")
    rows, cols = 2100, 1024
    check_against_oracle(graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols), mode, what=f"lnbwd {opts}", **opts)


@pytest.mark.parametrize("mode", LNBWD_MODES)
def test_layernorm_bwd_is_bit_reproducible_and_reusable(mode):
    announce(f"layernorm_bwd determinism {mode}")
    rows, cols = 3000, 1024
    ops, ins = graphs.layernorm_bwd(rows, cols), inputs.layernorm_bwd(rows, cols)
    dev_in = to_device(ops, ins)
    runs = []
    with Plan(ops, mode) as plan:
        for _ in range(5):
            out = alloc_outputs(ops)
            plan.launch(dev_in, out)
            torch.cuda.synchronize()
            runs.append([t.cpu().numpy() for t in out])
    for r in runs[1:]:
        for a, b in zip(runs[0], r):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("mode", LNBWD_MODES)
def test_layernorm_bwd_output_subsets(mode):
    announce(f"layernorm_bwd subsets {mode}")
    rows, cols = 300, 512
    full = graphs.layernorm_bwd(rows, cols)
    ins = inputs.layernorm_bwd(rows, cols)
    outs = [i for i, op in enumerate(full) if op.kind == "output"]
    for keep in ([0], [1, 2], [2], [0, 2]):
        ops = [op for i, op in enumerate(full) if op.kind != "output" or outs.index(i) in keep]
        check_against_oracle(ops, ins, mode, what=f"lnbwd outputs {keep}")


# ---------------------------------------------------------------- attention

@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("seq,dim", [(64, 64), (1, 32), (7, 64), (16, 32), (33, 64), (94, 64), (128, 32), (48, 128), (128, 64), (128, 128), (100, 128), (17, 32)])
def test_attention_shapes(seq, dim, dtype):
    announce(f"attention {dtype} seq={seq} dim={dim}")
    B = 5
    check_against_oracle(graphs.causal_attention(B, seq, dim, dtype), inputs.causal_attention(B, seq, dim, dtype),
                         what=f"attn {dtype} {seq}x{dim}")


def _attention_variant(B, S, d, causal, fill, dtype="f16"):
    g = graphs.Graph()
    q = g.parameter("q", dtype, (B, S, d))
    k = g.parameter("k", dtype, (B, S, d))
    v = g.parameter("v", dtype, (B, S, d))
    z = g.multiply(g.dot(q, k, transpose_b=True), g.constant(d ** -0.5))
    if causal:
        z = g.causal_mask(z, fill)
    zmax = g.reduce_max(z, -1)
    e = g.exp(g.subtract(z, g.row_broadcast(zmax, z)))
    p = g.divide(e, g.row_broadcast(g.reduce_sum(e, -1), e))
    o = g.dot(g.convert(p, dtype), v)
    g.output(g.convert(o, dtype))
    return g.ops


@pytest.mark.parametrize("causal,fill", [(False, 0.0), (True, -1e4), (True, -3.0)])
def test_attention_mask_variants(causal, fill):
    announce(f"attention causal={causal} fill={fill}")
    B, S, d = 3, 40, 64
    ops = _attention_variant(B, S, d, causal, fill)
    check_against_oracle(ops, inputs.causal_attention(B, S, d), what=f"attn causal={causal} fill={fill}")


# ---- schedule 3 with the elementwise ops around the two dots (Section 3.1's pattern shape): additive
# masks, an epilogue on O, a second output, unequal query and key lengths

ATTN_BLOCK_CASES = [
    # (batch, sq, sk, dim, dtype, kwargs)
    (3, 40, 72, 64, "f16", dict()),                                            # more keys than queries
    (2, 100, 24, 32, "bf16", dict()),                                          # more queries than keys
    (2, 16, 128, 128, "f16", dict(causal=True)),                               # one query tile, eight key tiles
    (3, 64, 64, 64, "f16", dict(mask="key")),                                  # key padding, vector mask loads
    (3, 50, 37, 64, "bf16", dict(mask="key")),                                 # ... ragged: scalar mask loads
    (2, 48, 64, 32, "f16", dict(mask="full")),
    (2, 33, 45, 64, "f16", dict(mask="full", causal=True)),
    (4, 64, 64, 64, "bf16", dict(mask="shared")),                              # one bias for the whole batch
    (2, 40, 40, 64, "f16", dict(mask="key", causal=True, mask_outside_causal=True)),
    (3, 64, 64, 64, "f16", dict(gate=True)),
    (3, 40, 72, 64, "bf16", dict(residual=True)),
    (2, 70, 50, 128, "f16", dict(gate=True, residual=True)),
    (3, 64, 64, 64, "f16", dict(lse=True, causal=True)),
    (2, 35, 90, 32, "bf16", dict(lse=True, mask="key")),
    (5, 64, 64, 64, "f16", dict(causal=True, mask="key", gate=True, residual=True, lse=True)),   # everything at once
    (2, 128, 128, 128, "bf16", dict(causal=True, mask="full", gate=True, residual=True, lse=True)),   # maximum sizes
    (1, 1, 1, 32, "f16", dict(lse=True, gate=True)),                           # a single score
]
# 128 MB and more: ordinary stores of the result
ATTN_BLOCK_CASES += [(1320, 100, 100, 128, "bf16", dict(causal=True, mask="key")), (1030, 128, 128, 128, "f16", dict(gate=True))]
# one query per batch element: every number of key tiles, whole and partial, every head dim, one wavefront to a workgroup
DECODE_CASES = [(b, 1, sk, d, dt, kw) for b, sk, d, dt, kw in [
    (5, 1, 64, "f16", dict()), (3, 16, 32, "bf16", dict()), (6, 17, 128, "f16", dict()), (7, 31, 64, "bf16", dict(mask="key")), (9, 48, 128, "bf16", dict(mask="key", lse=True)),
    (4, 50, 32, "f16", dict(mask="full", gate=True)), (1, 64, 64, "f16", dict(mask="shared", residual=True)), (130, 77, 64, "bf16", dict(mask="key")),
    (5, 90, 128, "f16", dict(gate=True, residual=True, lse=True)), (6, 112, 32, "bf16", dict(mask="key", gate=True, residual=True, lse=True)),
    (33, 127, 64, "f16", dict(mask="key")), (11, 128, 128, "f16", dict(mask="key")), (10, 128, 64, "bf16", dict()), (3, 127, 128, "bf16", dict(mask="full"))]]
# ... both sides of the lines of the rule that picks the kernel; two and four wavefronts to a workgroup (from 2048 and 4096 elements on),
# the last workgroup partly empty; K and V of more than 12 MB (nontemporal loads), whole and partial tiles, bare and with operands
DECODE_CASES += [(b, 1, sk, d, dt, kw) for b, sk, d, dt, kw in [
    (7, 8, 32, "f16", dict()), (7, 9, 32, "bf16", dict(mask="key")), (6, 32, 32, "f16", dict(mask="key", lse=True)), (6, 33, 32, "f16", dict(mask="key", lse=True)),
    (2047, 17, 64, "bf16", dict()), (2049, 40, 32, "bf16", dict(mask="key")), (4095, 5, 32, "f16", dict(gate=True)), (4099, 33, 32, "f16", dict()),
    (4099, 9, 128, "bf16", dict(mask="full", residual=True)), (4098, 16, 64, "f16", dict(lse=True)),
    (2049, 128, 64, "f16", dict()), (2050, 128, 64, "bf16", dict(mask="key")), (4099, 77, 64, "bf16", dict()), (4097, 77, 64, "f16", dict(mask="key", gate=True, residual=True, lse=True)),
    (767, 64, 64, "f16", dict()), (769, 64, 64, "f16", dict()),                          # (12 MB lie between them)
    (1031, 128, 128, "bf16", dict()), (1030, 100, 128, "f16", dict(mask="shared", lse=True)), (1033, 70, 128, "bf16", dict()), (4100, 100, 32, "f16", dict(mask="key"))]]
ATTN_BLOCK_CASES += DECODE_CASES
# a mask of keys in the padding of K: more keys than a workgroup has lanes, a single key, partial groups of four, with and without operands
ATTN_BLOCK_CASES += [(2, 16, 128, 64, "f16", dict(mask="key")), (3, 9, 70, 32, "bf16", dict(mask="key", residual=True)), (2, 128, 1, 64, "f16", dict(mask="key")),
                     (3, 20, 17, 32, "f16", dict(mask="key", lse=True)), (2, 65, 33, 128, "bf16", dict(mask="key", gate=True)), (2, 128, 128, 128, "f16", dict(mask="key")),
                     (2, 100, 100, 64, "bf16", dict(causal=True, mask="key", gate=True, residual=True, lse=True)), (3, 64, 113, 128, "f16", dict(mask="key", residual=True)),
                     (2, 128, 128, 64, "bf16", dict(causal=True, mask="key", residual=True)), (3, 50, 128, 128, "bf16", dict(mask="shared", gate=True, residual=True))]


@pytest.mark.parametrize("case", ATTN_BLOCK_CASES, ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}x{c[3]}-{c[4]}-" + "+".join(sorted(c[5])))
def test_attention_with_prologue_and_epilogue(case):
    B, sq, sk, d, dtype, kw = case
    announce(f"attention block {case}")
    ops = graphs.attention_block(B, sq, sk, d, dtype, **kw)
    ins = inputs.attention_block(B, sq, sk, d, dtype, **kw)
    with Plan(ops) as plan:
        assert plan.info()["schedule"] == "bdot_softmax" and plan.info()["n_kernels"] == 1
    got, want = check_against_oracle(ops, ins, what=f"attention block {case}")
    if kw.get("lse"):
        assert got[1].shape == (B, sq)


@pytest.mark.parametrize("B,sq,sk,d,dtype", [(8192, 16, 128, 64, "bf16"), (8192, 30, 127, 64, "f16"), (4096, 16, 128, 128, "f16")])
def test_causal_attention_requests_the_keys_it_needs(B, sq, sk, d, dtype):
    """With fewer queries than keys and a fill of -inf most rows of K are read by no one: by the bytes the causal group takes 0.60 (16 x 128) to 0.65 of
    the time of the same group without the mask (0.98 if all of K is read), and what K holds there counts in nothing."""
    announce(f"causal attention {B}x{sq}x{sk}x{d} {dtype}")
    groups = [graphs.attention_block(B, sq, sk, d, dtype, causal=causal) for causal in (True, False)]
    ins = inputs.attention_block(4, sq, sk, d, dtype, causal=True)
    tail = [np.array(a) for a in ins]
    tail[1][:, (sq + 15) // 16 * 16:, :] = np.nan
    small = graphs.attention_block(4, sq, sk, d, dtype, causal=True)
    assert np.array_equal(run_gpu(small, ins)[0], run_gpu(small, tail)[0])
    dev_in = [t.repeat(B // 4, 1, 1) for t in to_device(small, ins)]
    outs = alloc_outputs(groups[0])
    times = [[], []]
    with Plan(groups[0]) as causal, Plan(groups[1]) as full:
        for _ in range(12):
            for plan, took in ((causal, times[0]), (full, times[1])):
                start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                start.record()
                for _ in range(8):
                    plan.launch(dev_in, outs)
                end.record()
                end.synchronize()
                took.append(start.elapsed_time(end))
    assert np.median(times[0]) < 0.8 * np.median(times[1]), [np.median(t) for t in times]


@pytest.mark.parametrize("sq,sk,d,dtype,mask", [(64, 64, 64, "f16", "key"), (100, 100, 64, "bf16", "key"), (33, 70, 32, "f16", "key"), (16, 128, 128, "bf16", "key"),
                                                (64, 64, 64, "f16", "full"), (33, 70, 32, "bf16", "full")])
def test_attention_rounds_a_mask_with_the_score(sq, sk, d, dtype, mask):
    """A bias counts unrounded: one rounding at the size of the score times the scale, one of its sum with the bias, both in units of log 2.  The dots are
    of whole numbers, and one key's bias lies so far above the others that its score alone is the log-sum-exp: bit for bit."""
    announce(f"attention mask rounding {sq}x{sk}x{d} {dtype} {mask}")
    B, scale, f32 = 16, 0.01, np.float32
    rng = np.random.default_rng(sq * sk + d)
    q, k = (rng.integers(-2, 3, (B, n, d)).astype(np.float64) for n in (sq, sk))
    bias = rng.uniform(-64, 0, (B, 1, sk))
    bias[np.arange(B), 0, rng.integers(0, sk, B)] = rng.uniform(66, 90, B)
    bias = inputs.round_to(bias, "f32")
    log2e, ln2 = float(f32(1.4426950408889634)), f32(0.6931471805599453)
    z = (q @ k.transpose(0, 2, 1) * float(f32(scale) * f32(log2e))).astype(f32).astype(np.float64)
    want = (z + bias * log2e).max(axis=-1).astype(f32) * ln2
    full = np.broadcast_to(bias, (B, sq, sk)).copy()
    ops = graphs.attention_block(B, sq, sk, d, dtype, scale=scale, mask=mask, lse=True)
    got = run_gpu(ops, [q, k, rng.normal(size=(B, sk, d)), bias if mask == "key" else full])[1]
    assert np.array_equal(got.reshape(B, sq), want)


# ---------------------------------------------------------------- full-size configs, bench launch shape

def test_full_size_layernorm_fwd():
    announce("full cfg1")
    ops, ins = BY_NAME["layernorm_fwd"].build("full")
    check_against_oracle(ops, ins, what="cfg1 full")


def test_full_size_softmax_whole_tensor():
    announce("full cfg2")
    cfg = BY_NAME["scaled_masked_softmax"]
    ops, ins = cfg.build("full")
    (got,) = run_gpu(ops, ins)
    (want,) = interp.run(ops, ins)
    assert_close(got, want, 1e-5, "cfg2 full, every element")
    # properties that hold for every row
    assert np.abs(got.sum(axis=1) - 1).max() < 1e-5
    assert got.min() >= 0 and not np.isnan(got).any()


def test_full_size_attention_whole_tensor():
    announce("full cfg3")
    cfg = BY_NAME["causal_attention"]
    ops, ins = cfg.build("full")
    (got,) = run_gpu(ops, ins)
    (want,) = interp.run(ops, ins)
    assert_close(got, want, 2e-2, "cfg3 full, every element")
    assert np.allclose(got[:, 0, :], ins[2][:, 0, :], atol=1e-3)   # first query row sees only V[0]
    assert not np.isnan(got).any()


@pytest.mark.parametrize("mode", GELU_LN_MODES)
def test_full_size_bias_gelu_ln_whole_tensor(mode):
    announce(f"full cfg4 {mode}")
    cfg = BY_NAME["bias_gelu_residual_layernorm"]
    ops, ins = cfg.build("full")
    (got,) = run_gpu(ops, ins, mode)
    (want,) = interp.run(ops, ins)
    assert_close(got, want, 2e-2, "cfg4 full, every element")
    assert not np.isnan(got).any()


@pytest.mark.parametrize("mode", LNBWD_MODES)
def test_full_size_layernorm_bwd(mode):
    announce(f"full cfg5 {mode}")
    cfg = BY_NAME["layernorm_bwd"]
    ops, ins = cfg.build("full")
    dx, dgamma, dbeta = run_gpu(ops, ins, mode)
    want_dx, want_dgamma, want_dbeta = interp.run(ops, ins)
    assert_close(dgamma, want_dgamma, 1e-5, "cfg5 full dgamma")
    assert_close(dbeta, want_dbeta, 1e-5, "cfg5 full dbeta")
    assert_close(dx, want_dx, 1e-5, "cfg5 full dx")


# ---------------------------------------------------------------- tuning (Algorithm 3's outer loop)

@pytest.mark.parametrize("cfg", CONFIGS, ids=lambda c: c.name)
def test_plan_tune_returns_a_correct_plan(cfg):
    announce(f"tune {cfg.name}")
    ops, ins = cfg.build("small")
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    plan = Plan.tune(ops, dev_in, dev_out, trials=3)
    try:
        assert plan.tuned["us"] > 0
        want = interp.run(ops, ins)
        tol = TOLERANCE[cfg.dtype]
        # the outputs already hold the winner's result
        torch.cuda.synchronize()
        for got, ref in zip(dev_out, want):
            assert_close(got.double().cpu().numpy(), ref, tol, f"tuned {cfg.name}")
        # and the returned plan is an ordinary plan
        fresh = alloc_outputs(ops)
        plan.launch(dev_in, fresh)
        torch.cuda.synchronize()
        for got, ref in zip(fresh, want):
            assert_close(got.double().cpu().numpy(), ref, tol, f"tuned relaunch {cfg.name}")
        # one stitched kernel; the generated form of a group with column reductions adds its combine kernel
        assert plan.info()["n_kernels"] <= (2 if plan.info()["schedule"] == "row_col" else 1)
    finally:
        plan.close()


def test_tuned_options_are_reused_by_later_plans(tmp_path):
    """'Optimize once, reuse': the winner of fs_plan_tune is what fs_plan_create builds for the same
    group from then on (launch parameters left open), also after a trip through the cache file."""
    from paper_1911_11576_amd import fs_tune_cache_clear, fs_tune_cache_load, fs_tune_cache_save, fs_tune_cache_size
    announce("tuning cache")
    ops, ins = graphs.rmsnorm((2048, 1024), "bf16"), inputs.normal_tensors([(2048, 1024), (1024,)], "bf16")
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    assert fs_tune_cache_size() == 0
    with Plan(graphs.rmsnorm((2047, 1024), "bf16")) as p:
        other_shape = p.describe()
    with Plan.tune(ops, dev_in, dev_out, trials=5) as tuned:
        winner = tuned.describe()
    assert fs_tune_cache_size() == 1
    with Plan(ops) as p:
        assert p.describe() == winner
    check_against_oracle(ops, ins, what="plan from the tuning cache")
    fs_tune_cache_save(tmp_path / "t.txt")
    fs_tune_cache_clear()
    fs_tune_cache_load(tmp_path / "t.txt")
    with Plan(ops) as p:
        assert p.describe() == winner
    # another shape of the same group is another entry
    with Plan(graphs.rmsnorm((2047, 1024), "bf16")) as p:
        assert p.describe() == other_shape


def test_plan_tune_rejects_unsupported_groups_and_bad_arguments():
    announce("tune errors")
    g = graphs.Graph()
    x = g.parameter("x", "f32", (4, 8, 6, 64))
    g.output(g.reduce_sum(g.exp(x), 1))       # a reduction over an outer dim that keeps the dims between: no stitched schedule
    t = torch.zeros(4, 8, 6, 64, device="cuda:0")
    with pytest.raises(FsError) as e:
        Plan.tune(g.ops, [t], [torch.empty(4, 6, 64, device="cuda:0")])
    assert e.value.status == binding.FS_ERR_UNSUPPORTED
    ops, ins = graphs.layernorm_fwd(4, 768), inputs.layernorm_fwd(4, 768)
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with pytest.raises(FsError) as e:
        Plan.tune(ops, dev_in[:2], dev_out)
    assert e.value.status == binding.FS_ERR_INVALID
    with pytest.raises(FsError) as e:
        Plan.tune(ops, dev_in, dev_out, trials=0)
    assert e.value.status == binding.FS_ERR_INVALID


# ---------------------------------------------------------------- edge cases and error paths

def test_empty_inputs_launch_nothing_and_succeed():
    announce("empty inputs")
    for ops, ins in [(graphs.layernorm_fwd(0, 768), inputs.layernorm_fwd(0, 768)),
                     (graphs.causal_attention(0, 64, 64), inputs.causal_attention(0, 64, 64))]:
        for mode in ("stitched", "per_op"):
            out = run_gpu(ops, ins, mode)
            assert out[0].size == 0


def test_launch_rejects_bad_pointers_and_counts():
    announce("launch argument errors")
    ops, ins = graphs.layernorm_fwd(4, 768), inputs.layernorm_fwd(4, 768)
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with Plan(ops) as plan:
        with pytest.raises(FsError) as e:
            plan.launch(dev_in[:2], dev_out)
        assert e.value.status == binding.FS_ERR_INVALID
        with pytest.raises(FsError) as e:
            plan.launch([dev_in[0].data_ptr() + 4, dev_in[1], dev_in[2]], dev_out)
        assert e.value.status == binding.FS_ERR_INVALID
        with pytest.raises(FsError) as e:
            plan.launch([0, dev_in[1], dev_in[2]], dev_out)
        assert e.value.status == binding.FS_ERR_INVALID
        plan.launch(dev_in, dev_out)      # the plan still works afterwards
        torch.cuda.synchronize()
    (want,) = interp.run(ops, ins)
    assert_close(dev_out[0].double().cpu().numpy(), want, 1e-5, "after errors")


def test_stream_copy_matches_source():
    announce("stream copy")
    src = torch.randint(0, 255, (3 * 1024 * 1024 + 16,), dtype=torch.uint8, device="cuda:0")
    dst = torch.zeros_like(src)
    binding.fs_stream_copy(dst, src, src.numel())
    torch.cuda.synchronize()
    assert torch.equal(src, dst)


def test_launch_on_a_side_stream():
    announce("side stream")
    ops, ins = graphs.layernorm_fwd(64, 768), inputs.layernorm_fwd(64, 768)
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with Plan(ops) as plan:
        plan.launch(dev_in, dev_out, stream=s.cuda_stream)
        s.synchronize()
    (want,) = interp.run(ops, ins)
    assert_close(dev_out[0].double().cpu().numpy(), want, 1e-5, "side stream")


# ---------------------------------------------------------------- launches recorded into a HIP graph

@pytest.mark.parametrize("name", ["scaled_masked_softmax", "layernorm_bwd", "causal_attention", "multi_tensor_momentum"])
def test_launches_replay_from_a_captured_graph(name):
    """After one ordinary launch (which loads the kernels and allocates the plan's workspace) a launch is
    nothing but kernel launches on the caller's stream, so it can be recorded into a HIP graph.
    The graph is replayed three times, with eager work and new input values between the replays,
    and every replay is compared with the oracle."""
    announce(f"graph capture {name}")
    cfg = BY_NAME[name]
    ops, ins = cfg.build("small")
    tol = TOLERANCE[cfg.dtype]
    dev_in, dev_out = to_device(ops, ins), alloc_outputs(ops)
    with Plan(ops) as plan:
        plan.launch(dev_in, dev_out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=side):
            plan.launch(dev_in, dev_out)                      # torch's current stream is the capturing one here
        for rep in range(3):
            # new values in the same buffers: the first tensor is scaled, eagerly, between replays
            scale = [1.0, 0.5, -1.5][rep]
            cur = [a * scale if k == 0 else a for k, a in enumerate(ins)]
            cur[0] = inputs.round_to(cur[0], ops[0].dtype)
            dev_in[0].copy_(to_device(ops, cur)[0])
            for t in dev_out:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            want = interp.run(ops, cur)
            for got, ref in zip(dev_out, want):
                assert_close(got.double().cpu().numpy(), ref, tol, f"graph replay {rep} of {name}")
