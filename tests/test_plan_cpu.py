"""The sizes of the parity tests reach the kernels that their comments name (the plans are host code)."""
import pytest

import test_parity_gpu as t


@pytest.mark.parametrize("dims,B,plan", [(r[0], r[-2], r[-1]) for r in t.F32_EDGES + t.F32_FEW_ROWS] + t.SPLIT_SIZES)
def test_f32_cases_run_the_kernels_they_name(dims, B, plan):
    assert t.f32_plan(dims, B) == plan


@pytest.mark.parametrize("dims,B,plan", [(r[0], r[-2], r[-1]) for r in t.BF16_WIDE + t.BF16_SMALL_TILES + t.BF16_SHORT])
def test_bf16_cases_run_the_kernels_they_name(dims, B, plan):
    assert t.bf16_plan(dims, B) == plan


@pytest.mark.parametrize("dims,B,kernels", [(r[0], r[2], r[3]) for r in t.F32_LONG_FORWARD])
def test_f32_long_forward_cases_run_the_kernels_they_name(dims, B, kernels):
    assert t.f32_plan(dims, B).split("; ")[0].split()[:-1] == kernels


@pytest.mark.parametrize("dims,B,pairs", [(r[0], r[2], r[3]) for r in t.BF16_PAIRS])
def test_bf16_cases_share_the_launches_they_name(dims, B, pairs):
    assert t.bf16_pairs(dims, B) == pairs


def test_the_cases_reach_every_form_of_the_small_products():
    for r in t.F32_SMALL:
        assert t.f32_small_forms(r[0], r[2]) == r[3]
    for r in t.SAME_SUMS:
        assert (t.f32_small_forms(r[0], r[2]), t.f32_small_forms(r[1], r[2])) == r[3:]
    forms = [r[3].split("; ") for r in t.F32_SMALL]
    assert {k for f in forms for k in f[0].split()} == {"16", "32", "32s"}
    assert {k for f in forms for k in f[1].split()} == {"-", "16", "16w1", "16w2", "32", "32w1", "32w2"}
    assert {f[2] for f in forms} == {"-", "32", "32w1", "32w2"}
    assert {t.small_net_rows(dims, B) for dims, _, _, B in t.SMALL_NETS} == {16, 32, 64}


def test_the_cases_reach_every_kernel():
    forward, pairs, alone = ({k for r in t.F32_EDGES for k in r[-1].split("; ")[q].split()} for q in range(3))
    forward |= {k for r in t.F32_LONG_FORWARD for k in r[-1]}
    assert forward == set(t.F32_KERNELS) and pairs == alone == set(t.F32_KERNELS) - {"64x32"}
    bf16 = [r[-1].split("; ") for r in t.BF16_WIDE + t.BF16_SMALL_TILES + t.BF16_SHORT]
    forward, da, dw = ({k.split("/")[0] for r in bf16 for k in r[q].split()} for q in range(3))
    assert forward | {r[-1] for r in t.BF16_SHIFTED} == {"dma", "128", "128s", "64", "64s", "64S", "64sS", "128S", "128sS"}
    assert da == {"dma", "128", "128s", "64", "64s"}
    assert dw == {"dma", "dmaB", "128", "64", "64B", "64s", "64sB"}


def test_the_widest_input_keeps_its_batch_major_weight_gradient():
    """Rows of 2^24 values, the largest d_0, fit the kernels' 32-bit offsets: no transposed copy of X (32 MB a row)."""
    from paper_2004_08771_amd import lib
    for d_in in ((1 << 24) - 8, 1 << 24):
        assert lib().hb_plan_bf16_kernel(2, 64, d_in, 300, 1) & 32, d_in


@pytest.mark.parametrize("d_out,d_in,line", [(256, 256, 7500), (1024, 1024, 7500), (1025, 1024, 5120), (1280, 1280, 5120)])
def test_bf16_weight_gradients_are_split_where_the_small_tiles_fall_behind(d_out, d_in, line):
    """Up to 256 tiles of 64 x 64 the small tiles keep the whole batch for longer; the slice buffer, sized for the largest
    batch, holds what every smaller one asks for."""
    from paper_2004_08771_amd import lib
    slices, kernel = lib().hb_plan_bf16_dw_slices, lib().hb_plan_bf16_kernel
    assert slices(d_out, d_in, line - 1, 1) == 1 and slices(d_out, d_in, line, 1) == line // 1024
    assert t.BF16_KERNELS[kernel(2, d_out, d_in, line - 1, 0) & 15] in ("64", "64s")
    assert t.BF16_KERNELS[kernel(2, d_out, d_in, line, 0) & 15] == "dma"
    caps = [slices(d_out, d_in, B, 1) for B in range(2048, 12000, 7)]
    assert caps == sorted(caps)


@pytest.mark.parametrize("dims,rows", [
    # {batch: rows per workgroup}: every block size fits
    ((54, 32, 7), {1: 16, 16: 16, 17: 32, 33: 64, 64: 64, 65: 16, 2048: 16, 2049: 32, 4097: 64, 8192: 64, 8193: 0}),
    # blocks of 32 rows at most, and of 16: more rows in several blocks of 16, also below 65
    ((64, 64, 64, 64, 5), {32: 32, 33: 16, 48: 16, 64: 16, 65: 16, 4096: 32, 4097: 0}),
    ((100, 64, 64, 64, 64, 64, 4), {16: 16, 17: 16, 33: 16, 64: 16, 65: 16, 2048: 16, 2049: 0}),
    # two layers: apart where a block of all rows does not fit
    ((80, 100, 4), {32: 32, 33: 0, 64: 0, 65: 16}),
    ((100, 100, 100, 3), {16: 0, 100: 0}), ((54, 32, 17), {16: 0}), ((54, 7), {16: 0}),
])
def test_small_networks_take_any_batch_up_to_their_largest(dims, rows):
    assert {B: t.small_net_rows(dims, B) for B in rows} == rows
    if len(dims) > 3 and rows.get(16, 16):  # no gap
        most = max(B for B in rows if rows[B])
        assert all(t.small_net_rows(dims, B) for B in range(1, most + 1))


def test_plans_refuse_invalid_arguments():
    from paper_2004_08771_amd import lib
    f, b = lib().hb_plan_f32_kernel, lib().hb_plan_bf16_kernel
    assert f(0, 0, 5, 5, 5, None) == -1 and f(3, 5, 5, 5, 5, None) == -1 and f(0, 5, 5, 6, 5, None) == -1
    s = lib().hb_plan_f32_small_form
    assert s(0, 0, 5, 5, 5) == -1 and s(3, 5, 5, 5, 5) == -1 and s(0, 5, 5, 6, 5) == -1 and s(0, 512, 512, 4096, 4096) == 0
    import ctypes
    p, dims = lib().hb_plan_bf16_pair, (ctypes.c_int32 * 3)(6, 5, 5)
    assert p(dims, 3, 5, 0) == -1 and p(dims, 3, 5, 3) == -1 and p(dims, 3, 0, 1) == -1 and p(None, 3, 5, 1) == -1
    assert p((ctypes.c_int32 * 3)(5, 0, 5), 3, 5, 1) == -1 and p(dims, 3, 5, 1) == 0 and p(dims, 3, 5, 2) == 1
    assert t.small_net_rows((5,), 5) == -1 and t.small_net_rows((5, 0, 5), 5) == -1 and t.small_net_rows((5, 5, 5), 0) == -1
    assert b(0, 5, 0, 5, 0) == -1 and b(-1, 5, 5, 5, 0) == -1 and b(0, 5, (1 << 24) + 1, 5, 0) == -1
