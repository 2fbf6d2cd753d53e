"""The matrix-core form of the tiled entry point against the oracle, where its tiling can go wrong: channel counts off
the blocks of 16 and 64, batches whose flat padded array ends inside a tile, every filter shape, one tile and many."""
import numpy as np
import pytest

import paper_1802_10280_amd as esc
from helpers import DeviceLayer, assert_within_bound, oracle_full
from paper_1802_10280_amd import workloads as wl

gpu = pytest.mark.gpu

# N, C, H, W, M, R, S, pad, sparsity
SHAPES = [
    (96, 64, 16, 16, 64, 3, 3, 1, 0.0),      # whole blocks of channels
    (105, 49, 15, 17, 65, 3, 3, 1, 0.0),     # one channel over on both sides, an odd batch
    (301, 47, 7, 7, 129, 3, 3, 1, 0.0),      # small maps, channels short of a block
    (80, 17, 33, 20, 60, 5, 5, 2, 0.2),
    (120, 33, 18, 13, 112, 3, 4, 0, 0.0),    # no padding: taps reach the end of a row, not past it
    (90, 24, 13, 18, 120, 5, 3, 1, 0.0),     # padding smaller than the reach
    (23, 48, 60, 61, 64, 3, 3, 1, 0.3),      # windows of 382 positions,
    (24, 33, 40, 63, 96, 3, 3, 1, 0.0),      # of 386: one workgroup to a compute unit from here on,
    (29, 40, 31, 30, 72, 5, 5, 2, 0.3),      # of 388,
    (13, 65, 20, 126, 64, 3, 3, 1, 0.0),     # of 512, the most there is
    (150, 250, 14, 14, 120, 1, 1, 0, 0.0),   # one tap
]


def mfma_layer(L):
    """The layer on the device with its default plan; a forward_tiled on it takes the matrix-core kernel."""
    dl = DeviceLayer(esc, L)
    dl.forward_tiled()
    assert esc.escoin_sconv_tiled_on_matrix_cores(dl.desc, dl.plan) and dl.d_plan.data_ptr() % 16 == 0
    return dl


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_the_matrix_cores(shape):
    N, C, H, W, M, R, S, pad, sparsity = shape
    L = wl.custom_layer(N, C, H, W, M, R, S, 1, pad, sparsity, seed=71, dist="normal")
    d = esc.desc_of(L.spec)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    assert esc.escoin_sconv_tiled_on_matrix_cores(d, plan)
    one = esc.make_desc(1, C, H, W, M, R, S, 1, pad)
    assert not esc.escoin_sconv_tiled_on_matrix_cores(one, plan)
    with pytest.raises(esc.EscoinError):
        esc.escoin_sconv_tiled_on_matrix_cores(esc.make_desc(N, C, H, W, M + 1, R, S, 1, pad), plan)


@gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_against_the_oracle(oracle, shape):
    print("mfma", shape, flush=True)
    N, C, H, W, M, R, S, pad, sparsity = shape
    L = wl.custom_layer(N, C, H, W, M, R, S, 1, pad, sparsity, seed=71, dist="normal")
    dl = mfma_layer(L)
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got = dl.forward_tiled(flags)
        ref, bound = oracle_full(oracle, L, flags)
        assert np.isfinite(got).all()
        worst = assert_within_bound(got, ref, bound, (shape, flags))
        # the split is exact and the products left out are below 2^-24 of |x*w|: a sum of at most C*R*S fp32
        # roundings, of which a random walk's share shows
        assert worst <= 2.0 ** -24 * 4 * np.sqrt(C * R * S), worst


@gpu
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[9]], ids=str)
def test_unaligned_buffers_guards_and_one_plan_for_two_batches(oracle, shape):
    """Input and output one word off alignment, NaN around the output; then the same plan at batch 1 (tiled kernel)."""
    import torch
    print("mfma unaligned", shape, flush=True)
    N, C, H, W, M, R, S, pad, sparsity = shape
    L = wl.custom_layer(N, C, H, W, M, R, S, 1, pad, sparsity, seed=80, dist="normal")
    dl = mfma_layer(L)
    ref, bound = oracle_full(oracle, L)
    n_in, n_out, guard = L.input.size, ref.size, 1 << 16
    room = torch.full((n_in + 4,), float("nan"), device="cuda")
    d_in = room[1:1 + n_in].copy_(dl.d_in.flatten())
    out = torch.full((guard + 1 + n_out + guard,), float("nan"), device="cuda")
    d_out = out[guard + 1:guard + 1 + n_out]
    assert d_in.data_ptr() % 16 == 4 and d_out.data_ptr() % 16 == 4
    esc.escoin_sconv_forward_tiled(dl.desc, dl.plan, dl.d_plan, d_in, d_out)
    assert_within_bound(d_out.cpu().numpy().reshape(ref.shape), ref, bound, shape)
    assert bool(out[:guard + 1].isnan().all()) and bool(out[guard + 1 + n_out:].isnan().all())
    one = esc.make_desc(1, C, H, W, M, R, S, 1, pad)
    assert not esc.escoin_sconv_tiled_on_matrix_cores(one, dl.plan)
    dl.d_out.fill_(float("nan"))
    esc.escoin_sconv_forward_tiled(one, dl.plan, dl.d_plan, dl.d_in[:1], dl.d_out[:1])
    assert_within_bound(dl.d_out[:1].cpu().numpy(), ref[:1], bound[:1], shape)
    assert bool(dl.d_out[1:].isnan().all())


@pytest.mark.parametrize("W, N, tiled_us, taken", [
    (62, 35, 95.0, False),     # windows of 384: two workgroups share a compute unit, 552 take two rounds of 49.8 us
    (63, 35, 95.0, True),      # 386: they cannot, and 560 take three of 29.0
    (63, 35, 80.0, False),
    (63, 62, 108.0, False),    # 992 take four
    (63, 62, 115.0, True),
    (63, 64, 115.0, True),     # 1024
    (63, 65, 120.0, False),    # 1040: five
])
def test_wide_windows_count_as_one_workgroup_to_a_compute_unit(W, N, tiled_us, taken):
    """64 channels, 3x3, as many nonzeros as the tiled kernel is put at that time for."""
    L = wl.custom_layer(1, 64, 63, W, 64, 3, 3, 1, 1, 0.0, seed=81, dist="normal")
    per_row = int(tiled_us * 36e6 / (2 * N * 63 * W) / 64)
    rowptr = np.arange(65, dtype=np.int32) * np.int32(per_row)
    colidx = np.concatenate([L.colidx[L.rowptr[m]:L.rowptr[m] + per_row] for m in range(64)])
    d = esc.make_desc(N, 64, 63, W, 64, 3, 3, 1, 1)
    plan = esc.escoin_sconv_plan_build(d, rowptr, esc.escoin_sconv_pack(d, rowptr, colidx), np.ones(64 * per_row, dtype=np.float32))
    assert esc.escoin_sconv_tiled_on_matrix_cores(d, plan) == taken


def set_weight(L, m, c, tap, value):
    """The weight of channel m at (input channel c, tap); the CSR has to hold it."""
    row = slice(L.rowptr[m], L.rowptr[m + 1])
    at = np.flatnonzero(L.colidx[row] == c * L.spec.R * L.spec.S + tap)
    assert len(at) == 1
    L.value[L.rowptr[m] + at[0]] = value


@gpu
def test_products_around_the_largest_float(oracle):
    """Finite operands whose product overflows: Inf with its sign, never NaN (the parts of such a product overflow
    with both signs); a product just below the largest float stays finite (the leading parts' product is above it)."""
    print("mfma overflow", flush=True)
    L = wl.custom_layer(105, 49, 15, 17, 65, 3, 3, 1, 1, 0.0, seed=75, dist="normal")
    L.value *= np.float32(0.2)               # every other product of these inputs stays far below the limit
    L.input[:] = 0
    near = np.float32(1.00391 * 2.0 ** 20)
    for image, c, m, x, w in ((3, 4, 2, 1e38, 2057.0), (9, 7, 33, 3e38, 4117.0), (17, 20, 64, -3e38, 4117.0),
                              (104, 48, 0, 1e38, 2057.0), (50, 30, 40, 3.4028e38 / float(near), near)):
        L.input[image, c, 5, 6] = x
        set_weight(L, m, c, 4, w)
    with np.errstate(over="ignore"):
        ref, bound = oracle_full(oracle, L)
    dl = mfma_layer(L)
    got = dl.forward_tiled()
    over = np.isinf(ref)
    assert over.sum() == 4 and (got[over] == ref[over]).all()
    assert_within_bound(got[~over], ref[~over], bound[~over])


@gpu
def test_non_finite_inputs_reach_only_nonzero_weights(oracle):
    print("mfma non-finite", flush=True)
    L = wl.custom_layer(200, 50, 12, 13, 98, 3, 3, 1, 1, 0.05, seed=72, dist="normal")
    L.input[1, 2, 5, 6] = np.inf
    L.input[2, 0, 0, 0] = np.nan
    L.input[199, 49, 11, 12] = -np.inf
    L.input[20, 3, 4, 4] = 3.4e38            # finite, but not in bf16
    for flags in (0, esc.F_BIAS):
        dl = mfma_layer(L)
        got = dl.forward_tiled(flags)
        with np.errstate(invalid="ignore", over="ignore"):
            ref, bound = oracle_full(oracle, L, flags)
        bad = ~np.isfinite(ref)
        assert bad.any() and (bad == ~np.isfinite(got)).all()
        assert (np.abs(got[~bad] - ref[~bad]) <= 1e-4 * bound[~bad]).all()


def test_what_the_form_cannot_hold_stays_with_the_tiled_kernel():
    """A repeated column and a weight that is not finite in bf16 leave the plan without the section."""
    L = wl.custom_layer(40, 64, 12, 12, 64, 3, 3, 1, 1, 0.0, seed=73, dist="normal")
    d = esc.desc_of(L.spec)
    st = esc.escoin_sconv_pack(d, L.rowptr, L.colidx)
    assert esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, st, L.value))["mfma"] == 1
    twice = st.copy()
    twice[1] = twice[0]
    assert esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, twice, L.value))["mfma"] == 0
    for v in (np.inf, np.nan, 3.4e38):
        value = L.value.copy()
        value[5] = v
        assert esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, st, value))["mfma"] == 0


def test_explicit_zeros_do_not_count_as_nonzeros():
    """A layer that keeps a full pattern with most values zero is a heavily pruned one."""
    L = wl.custom_layer(40, 64, 12, 12, 64, 3, 3, 1, 1, 0.0, seed=79, dist="normal")
    d = esc.desc_of(L.spec)
    st = esc.escoin_sconv_pack(d, L.rowptr, L.colidx)
    kept = np.random.default_rng(79).random(L.nnz)
    for share, held in ((1.0, 1), (0.6, 1), (0.1, 0)):
        value = np.where(kept < share, L.value, np.float32(0))
        h = esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, st, value))
        assert h["mfma"] == held and h["mfma_nnz"] == held * np.count_nonzero(value), share


def test_weights_out_of_the_range_that_splits_exactly_stay_with_the_tiled_kernel():
    L = wl.custom_layer(40, 64, 12, 12, 64, 3, 3, 1, 1, 0.0, seed=73, dist="normal")
    d = esc.desc_of(L.spec)
    st = esc.escoin_sconv_pack(d, L.rowptr, L.colidx)
    least, most = np.float32(2.0 ** -50), np.float32(2.0 ** 30)
    for v, kept in ((least, 1), (np.nextafter(least, np.float32(0)), 0), (np.float32(2.0 ** -118), 0), (np.float32(1e-45), 0),
                    (most, 1), (np.nextafter(most, np.float32(np.inf)), 0)):
        for sign in (1, -1):
            value = L.value.copy()
            value[5] = sign * v
            h = esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, st, value))
            assert h["mfma"] == kept and h["mfma_nnz"] == kept * L.nnz, v


@gpu
@pytest.mark.parametrize("power", [-60, -100, -112, -118, -123])
def test_small_weights(oracle, power):
    print("mfma small weights", power, flush=True)
    L = wl.custom_layer(105, 49, 15, 17, 65, 3, 3, 1, 1, 0.0, seed=76, dist="normal")
    L.value *= np.float32(2.0 ** power)
    L.input *= np.float32(1024)
    dl = DeviceLayer(esc, L)  # the tiled kernel, down to 2^-50
    got = dl.forward_tiled()
    ref, bound = oracle_full(oracle, L)
    # fp32: every one of the C*R*S products and sums rounds by 2^-24 of sum|w*x|, or by half a subnormal's 2^-149
    n = L.spec.C * L.spec.R * L.spec.S
    assert (np.abs(got - ref) <= 2.0 ** -24 * 4 * np.sqrt(n) * bound + n * 2.0 ** -150).all()


@gpu
@pytest.mark.parametrize("power", [-72, -100, -112, -123, -134, -145])
@pytest.mark.parametrize("everywhere", [True, False])
def test_small_inputs(oracle, power, everywhere):
    """Inputs too small for three bf16 parts, everywhere or in one channel of some images beside zeros."""
    print("mfma small inputs", power, everywhere, flush=True)
    L = wl.custom_layer(105, 49, 15, 17, 65, 3, 3, 1, 1, 0.0, seed=77, dist="normal")
    small = L.input * np.float32(2.0 ** power)
    if everywhere:
        L.input[:] = small
    else:
        L.input[::5] = 0
        L.input[::5, 7] = small[::5, 7]
    L.value *= np.float32(16)
    dl = mfma_layer(L)
    got = dl.forward_tiled()
    ref, bound = oracle_full(oracle, L)
    # as above: fp32 rounding of C*R*S products and sums, or half a subnormal's step each
    n = L.spec.C * L.spec.R * L.spec.S
    assert (np.abs(got - ref) <= 2.0 ** -24 * 4 * np.sqrt(n) * bound + n * 2.0 ** -150).all()


@gpu
@pytest.mark.parametrize("where", ["a row", "a column", "an image", "every image"])
def test_many_non_finite_inputs(oracle, where):
    """From a few positions of a workgroup to all of them are computed from the nonzeros: several lanes to an output,
    one, full and part-filled runs of positions, a ragged last group of channels."""
    print("mfma many non-finite", where, flush=True)
    L = wl.custom_layer(105, 49, 15, 17, 65, 3, 3, 1, 1, 0.2, seed=78, dist="normal")
    place = {"a row": np.s_[3, 7, 4], "a column": np.s_[104, 7, :, 16], "an image": np.s_[50, 11], "every image": np.s_[:, 48]}
    L.input[place[where]] = np.inf
    L.input[1, 0, 0, 0] = np.nan
    dl = mfma_layer(L)
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got = dl.forward_tiled(flags)
        with np.errstate(invalid="ignore"):
            ref, bound = oracle_full(oracle, L, flags)
        bad = ~np.isfinite(bound)            # an output that met one; ReLU may have made it finite
        assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
        assert (np.abs(got[~bad] - ref[~bad]) <= 1e-4 * bound[~bad]).all()


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_split_weights_add_up_to_the_csr(shape):
    N, C, H, W, M, R, S, pad, sparsity = shape
    L = wl.custom_layer(1, C, H, W, M, R, S, 1, pad, sparsity, seed=74, dist="normal")
    d = esc.desc_of(L.spec)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    h = esc.plan_header(plan)
    blocks, chunks = -(-M // 64) * 2, -(-C // 16)
    raw = plan[h["off_mfma"]:h["off_mfma"] + blocks * chunks * R * S * 3072].view(np.uint16)
    w = (raw.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    w = w.reshape(blocks, chunks, R * S, 3, 2, 32, 8).sum(3)        # the three parts add up exactly
    w = w.transpose(0, 4, 1, 3, 5, 2).reshape(blocks * 32, chunks * 16, R * S)
    want = np.zeros((blocks * 32, chunks * 16 * R * S))
    for m in range(M):
        row = slice(L.rowptr[m], L.rowptr[m + 1])
        want[m, L.colidx[row]] = L.value[row]
    assert (w.reshape(want.shape) == want).all()
