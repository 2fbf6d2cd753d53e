"""The fp16-pair form of the tiled entry point against the oracle, where its tiling and its scaling can go wrong: channel
counts off the blocks of 16 and 64, ragged last tiles and rounds, filters three wide and not, inputs and weights of any size."""
import numpy as np
import pytest

import paper_1802_10280_amd as esc
from helpers import DeviceLayer, assert_within_bound, oracle_full, to_dev
from paper_1802_10280_amd import workloads as wl

gpu = pytest.mark.gpu

# N, C, H, W, M, R, S, pad, sparsity, workgroup layout
SHAPES = [
    (40, 64, 28, 28, 64, 3, 3, 1, 0.75, 122),      # whole blocks of channels
    (48, 49, 19, 23, 100, 3, 3, 1, 0.70, 212),     # channels over on both sides; a last round of two chunks of which one is a channel
    (37, 100, 25, 21, 90, 3, 3, 1, 0.70, 212),
    (20, 64, 56, 56, 64, 3, 3, 1, 0.80, 122),      # taps that reach far: windows of 244
    (30, 47, 18, 13, 112, 3, 4, 0, 0.60, 118),     # no padding, a filter four wide; three chunks for eight waves
    (24, 64, 13, 18, 120, 5, 3, 1, 0.65, 118),     # padding smaller than the reach
    (26, 384, 13, 13, 384, 3, 3, 1, 0.80, 114),    # many rounds
    (10, 512, 13, 13, 384, 3, 3, 1, 0.50, 118),    # sums long enough to go before three bf16 parts
    (16, 250, 14, 14, 250, 3, 3, 1, 0.80, 118),
    (60, 90, 28, 28, 250, 2, 2, 0, 0.60, 212),     # fewer steps a round than staging tasks
    (30, 100, 27, 31, 180, 3, 3, 1, 0.70, 122),
    (20, 196, 20, 20, 284, 3, 3, 1, 0.75, 212),   # 64 channels more than whole workgroups: a wave of the last ones has none
    (16, 192, 28, 28, 192, 3, 3, 1, 0.80, 212),    # ... and no remainder
]
SMALL = SHAPES[1]


def layer(shape, N=None, seed=91):
    n, C, H, W, M, R, S, pad, sparsity, _ = shape
    return wl.custom_layer(N or n, C, H, W, M, R, S, 1, pad, sparsity, seed=seed, dist="normal")


def pair_layer(L, layout):
    dl = DeviceLayer(esc, L)
    dl.forward_tiled()
    assert esc.escoin_sconv_tiled_kernel(dl.desc, dl.plan) == layout and dl.d_plan.data_ptr() % 16 == 0
    return dl


def limit(L, bound):
    """The split and the product left out: 2^-21 of every |w*x| at most.  The matrix cores' sums: as fp32 roundings of
    every product, of which a random walk's share shows.  Results below the least normal number: half its last bit."""
    n = L.spec.C * L.spec.R * L.spec.S
    return (2.0 ** -21 + 2.0 ** -24 * 4 * np.sqrt(n)) * bound + 2.0 ** -149


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_shapes_take_the_pairs(shape):
    N, C, H, W, M, R, S, pad, sparsity, layout = shape
    L = layer(shape, N=1)
    d = esc.make_desc(N, C, H, W, M, R, S, 1, pad)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    assert esc.escoin_sconv_tiled_kernel(d, plan) == layout and esc.escoin_sconv_tiled_on_matrix_cores(d, plan)
    assert esc.escoin_sconv_tiled_kernel(esc.desc_of(L.spec), plan) == 0
    with pytest.raises(esc.EscoinError):
        esc.escoin_sconv_tiled_kernel(esc.make_desc(N, C, H, W, M + 1, R, S, 1, pad), plan)


def test_pairs_add_up_to_the_csr():
    for shape in SHAPES:
        N, C, H, W, M, R, S, pad, sparsity, _ = shape
        L = layer(shape, N=1)
        d = esc.make_desc(N, C, H, W, M, R, S, 1, pad)
        plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
        h = esc.plan_header(plan)
        blocks, chunks = -(-M // 64) * 2, -(-C // 16)
        size = (blocks * chunks * R * S + 2) * 2048
        w = plan[h["off_pair"]:h["off_pair"] + size - 4096].view(np.float16).astype(np.float64)
        w = w.reshape(blocks, chunks, R * S, 2, 2, 32, 8)
        w = w[:, :, :, 0] + w[:, :, :, 1] / 2048
        w = w.transpose(0, 4, 1, 3, 5, 2).reshape(blocks * 32, chunks * 16 * R * S)
        exps = plan[h["off_pair"] + size:h["off_pair"] + size + 4 * M].view(np.int32)
        want = np.zeros_like(w)
        for m in range(M):
            row = slice(L.rowptr[m], L.rowptr[m + 1])
            want[m, L.colidx[row]] = L.value[row].astype(np.float64) * 2.0 ** exps[m]
            assert 2.0 ** 14 <= np.abs(want[m]).max() < 2.0 ** 15
        assert (np.abs(w - want) <= 2.0 ** -23 * np.abs(want)).all() and not w[M:].any()


def test_what_the_pairs_cannot_hold_stays_off_them():
    """A row that spans 28 binades, a short one, an Inf, a repeated column; explicit zeros are no nonzeros; a row of any size is fine."""
    L = layer(SMALL, N=1)
    N, C, H, W, M, R, S, pad, _, _ = SMALL
    d = esc.make_desc(N, C, H, W, M, R, S, 1, pad)
    st = esc.escoin_sconv_pack(d, L.rowptr, L.colidx)
    held = lambda stretched, value: esc.plan_header(esc.escoin_sconv_plan_build(d, L.rowptr, stretched, value))["pair"]
    assert held(st, L.value) == 1
    row = slice(L.rowptr[7], L.rowptr[8])
    most = np.abs(L.value[row]).max()
    for v, kept in ((most * 2.0 ** -26, 1), (most * 2.0 ** -28, 0), (np.inf, 0), (np.nan, 0)):
        value = L.value.copy()
        value[L.rowptr[7] + np.argmin(np.abs(L.value[row]))] = v
        assert held(st, value) == kept, v
    for power, kept in ((-100, 1), (100, 1)):
        value = L.value.copy()
        value[row] = np.clip(np.abs(value[row]), most / 100, most) * np.float32(2.0 ** power)
        assert held(st, value) == kept, power
    for left, kept in ((32, 1), (31, 0)):
        value = L.value.copy()
        value[L.rowptr[7] + left:L.rowptr[8]] = 0
        assert held(st, value) == kept, left
    twice = st.copy()
    twice[1] = twice[0]
    assert held(twice, L.value) == 0


# Layers of which some rows are cut to so many nonzeros: too few for pairs to be as exact as fp32 sums, about the batches of 16
# that those are computed in; the last layer's chains are split over two waves, so that the line lies higher.
SHORT = [SHAPES[2], SHAPES[5], SHAPES[6], SHAPES[10], (44, 272, 10, 10, 64, 3, 3, 1, 0.50, 118)]


def short_layer(shape, N=None):
    """The layer, and which of its rows were cut."""
    L = layer(shape, N=N, seed=99)
    M, rows = L.spec.M, np.diff(L.rowptr)
    lengths = [32, 33, 47, 48, 49, 56] if shape[1] != 272 else [33, 63, 64, 65, 100, 128]
    cut = np.unique(np.linspace(0, M - 1, 6).astype(int))
    rows[cut] = lengths
    keep = np.concatenate([np.arange(b - a) < k for a, b, k in zip(L.rowptr, L.rowptr[1:], rows)])
    L.colidx, L.value = L.colidx[keep], L.value[keep]
    L.rowptr = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    return L, cut


def plan_of(L, N):
    s = L.spec
    d = esc.make_desc(N, s.C, s.H, s.W, s.M, s.R, s.S, 1, s.pad)
    return d, esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)


@pytest.mark.parametrize("shape", SHORT, ids=str)
def test_short_rows_are_known(shape):
    """What the plan says of them: the least, and the batches of those below each layout's line."""
    L, cut = short_layer(shape, N=1)
    d, plan = plan_of(L, shape[0])
    h = esc.plan_header(plan)
    n, WS = np.diff(L.rowptr), h["WS"]
    assert h["pair"] == 1 and h["pair_least"] == n.min() and esc.escoin_sconv_tiled_kernel(d, plan) > 1
    for KW, base, slope in ((2, 0.81, 0.0044), (4, 0.81, 0.0020), (8, 0.92, 0.00105)):
        line = base / (0.0163 / WS - slope)
        assert h[f"pair_few{KW}"] == sum(-(-int(k) // 16) for k in n if k < line), KW
        assert (n[cut] < line).all()


@pytest.mark.parametrize("cut, kernel", [(8, 114), (32, 114), (47, 0)])
def test_many_short_rows_stay_with_the_tiled_kernel(cut, kernel):
    """Every short row costs the pairs' workgroups a walk over its nonzeros: with 8 and 32 of 166 rows such a call takes 22 and 30 us, 41
    and 37 on the tiled kernel; with 47 the two come out nearly even and it stays there."""
    L = layer((57, 97, 10, 12, 166, 3, 3, 1, 0.53, 0), N=1, seed=5)
    rows = np.diff(L.rowptr)
    rows[np.linspace(0, len(rows) - 1, cut).astype(int)] = 50
    keep = np.concatenate([np.arange(b - a) < k for a, b, k in zip(L.rowptr, L.rowptr[1:], rows)])
    L.colidx, L.value, L.rowptr = L.colidx[keep], L.value[keep], np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    d, plan = plan_of(L, 57)
    assert esc.plan_header(plan)["pair"] == 1 and esc.escoin_sconv_tiled_kernel(d, plan) == kernel


def test_short_rows_before_three_bf16_parts():
    """Beside the kernel of three bf16 parts, which is the more exact below 1023 nonzeros, a layer with a shorter row stays off the pairs."""
    shape = SHAPES[7]
    L = layer(shape, N=1)
    for left, kernel in ((1023, 118), (1022, 1)):
        L.value[L.rowptr[7] + left:L.rowptr[8]] = 0
        d, plan = plan_of(L, 32)
        assert esc.plan_header(plan)["pair_least"] == left and esc.escoin_sconv_tiled_kernel(d, plan) == kernel


def test_plans_saved_before_keep_off_the_pairs():
    """A plan whose header does not tell of pairs, or of its shortest row, is for the other kernels."""
    for fields in (("pair", "pair_nnz", "off_pair", "off_nz", "pair_least"), ("pair_least",)):
        for shape, N, without in ((SHAPES[1], 48, 0), (SHAPES[7], 32, 1)):
            L = layer(shape, N=1)
            d, plan = plan_of(L, N)
            assert esc.escoin_sconv_tiled_kernel(d, plan) == shape[-1]
            forget(plan, fields)
            assert esc.escoin_sconv_tiled_kernel(d, plan) == without


def test_no_batch_is_less_exact_than_without_the_pairs():
    """Which kernel the pairs stand in for goes with the batch; in place of three bf16 parts only eight shares of rows long enough do."""
    L = layer((1, 256, 28, 28, 256, 3, 3, 1, 0.78, 0))
    _, plan = plan_of(L, 64)
    old = plan.copy()
    forget(old, ("pair_least",))
    seen = set()
    for N in range(1, 129):
        d = esc.make_desc(N, 256, 28, 28, 256, 3, 3, 1, 1)
        taken, without = esc.escoin_sconv_tiled_kernel(d, plan), esc.escoin_sconv_tiled_kernel(d, old)
        assert without in (0, 1) and (taken == without or without == 0)
        seen.add((taken > 1, without))
    assert seen == {(False, 0), (True, 0), (False, 1)}


def rewrite(plan, **fields):
    from paper_1802_10280_amd.binding import _PlanHeader
    for f, v in fields.items():
        at = getattr(_PlanHeader, f)
        plan[at.offset:at.offset + at.size] = np.frombuffer(int(v).to_bytes(at.size, "little"), np.uint8)


def forget(plan, fields):
    rewrite(plan, **dict.fromkeys(fields, 0))


@gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_against_the_oracle(oracle, shape):
    print("pair", shape, flush=True)
    L = layer(shape)
    dl = pair_layer(L, shape[-1])
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got = dl.forward_tiled(flags)
        ref, bound = oracle_full(oracle, L, flags)
        assert_within_bound(got, ref, bound, (shape, flags))
        assert (np.abs(got - ref) <= limit(L, bound)).all()
    # and as exact as the fp32 chain of the tiled kernel, in the mean
    one = DeviceLayer(esc, L, tuning=dict(B=2))
    got, chain = dl.forward_tiled(), one.forward_tiled()
    ref, _ = oracle_full(oracle, L)
    assert esc.escoin_sconv_tiled_kernel(one.desc, one.plan) == 0
    assert np.linalg.norm(got - ref) <= np.linalg.norm(chain - ref)


# In place of three bf16 parts, in launches that fill the compute units: two shares, flushed every other round or so.
FLUSHED = [
    (74, 384, 14, 14, 250, 3, 3, 1, 0.55, 212),    # every third of twelve rounds
    (74, 272, 14, 14, 250, 3, 3, 1, 0.45, 212),    # nine rounds, the last of one chunk that two waves share
    (62, 496, 17, 17, 250, 2, 2, 0, 0.30, 212),    # filters two wide, every third round of sixteen
    (240, 250, 16, 16, 64, 3, 3, 1, 0.40, 122),    # two waves by positions
]


@gpu
@pytest.mark.parametrize("shape", FLUSHED, ids=str)
def test_flushed_sums(oracle, shape):
    print("pair flushed", shape, flush=True)
    L = layer(shape, seed=101)
    L.input[1, 7, 3, 4] = np.inf                    # ends in a sum that was flushed, and leads to the second pass
    dl, old = pair_layer(L, shape[-1]), DeviceLayer(esc, L)
    old.forward_tiled()
    forget(old.plan, ("pair_least",))
    old.d_plan = to_dev(old.plan)
    assert esc.escoin_sconv_tiled_kernel(old.desc, old.plan) == 1  # so unflushed pairs would not do
    with np.errstate(invalid="ignore", over="ignore"):
        ref, bound = oracle_full(oracle, L)
        got, parts = dl.forward_tiled().astype(np.float64), old.forward_tiled().astype(np.float64)
        off, parts_off = got - ref, parts - ref
    ok = np.isfinite(bound)
    assert not ok.all() and np.array_equal(got[~ok], ref[~ok], equal_nan=True)
    assert (np.abs(off[ok]) <= limit(L, bound)[ok]).all() and np.linalg.norm(off[ok]) <= np.linalg.norm(parts_off[ok])


# Stride 2: maps of odd and even sizes, so that the last row or column of a phase is there or not; filters that leave a phase without taps.
STRIDED = [
    (32, 100, 27, 31, 180, 3, 3, 1, 0.70, 212),
    (26, 250, 14, 13, 500, 3, 3, 1, 0.80, 114),    # rounds of four chunks, the last ragged
    (60, 60, 31, 31, 64, 4, 3, 3, 0.70, 122),      # padding as wide as the filter; one round
    (60, 113, 41, 20, 64, 3, 3, 0, 0.70, 114),
    (20, 64, 33, 30, 96, 5, 5, 2, 0.70, 114),
    (30, 200, 30, 30, 200, 2, 2, 0, 0.60, 114),
    (64, 200, 50, 30, 250, 1, 3, 1, 0.50, 212),    # one row of taps: two phases
    (64, 256, 40, 40, 40, 3, 1, 1, 0.50, 114),
    (64, 500, 28, 28, 256, 1, 1, 0, 0.50, 212),    # one tap: one phase
]


@gpu
@pytest.mark.parametrize("shape", STRIDED, ids=str)
def test_stride_two(oracle, shape):
    print("pair stride 2", shape, flush=True)
    N, C, H, W, M, R, S, pad, sparsity, layout = shape
    L = wl.custom_layer(N, C, H, W, M, R, S, 2, pad, sparsity, seed=102, dist="normal")
    dl, one = pair_layer(L, layout), DeviceLayer(esc, L, tuning=dict(B=2))
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got, chain = dl.forward_tiled(flags), one.forward_tiled(flags)
        ref, bound = oracle_full(oracle, L, flags)
        assert_within_bound(got, ref, bound, (shape, flags))
        assert (np.abs(got - ref) <= limit(L, bound)).all()
        if flags == 0:
            assert np.linalg.norm(got - ref) <= np.linalg.norm(chain - ref)
    # the second pass, the way back to the nonzeros, and rows too short for the pairs
    L.colidx, L.value, L.rowptr = cut_rows(L, [1, M // 2, M - 1], [33, 48, 40])
    L.input[N - 1, :, H // 2] *= np.float32(2.0 ** 12)
    L.input[1, 3, 2, 4] = np.inf
    L.input[2] = np.nan
    dl = DeviceLayer(esc, L)
    got = dl.forward_tiled(esc.F_BIAS)
    assert esc.escoin_sconv_tiled_kernel(dl.desc, dl.plan) > 1
    with np.errstate(invalid="ignore", over="ignore"):
        ref, bound = oracle_full(oracle, L, esc.F_BIAS)
    bad = ~np.isfinite(bound)
    assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
    assert (np.abs(got[~bad] - ref[~bad]) <= limit(L, bound)[~bad]).all()


# Stride 2, a plan for few images (whose tiled kernel splits its rows over waves, for shorter chains) and a call on many.
# N, C, H, W, M, R, sparsity, images of the plan, waves to a row, workgroup layout
REPLANNED = [
    (48, 336, 41, 41, 172, 3, 0.82, 1, 4, 114),    # two shares of the channels would need their sums flushed to be as exact
    (24, 66, 44, 44, 162, 5, 0.68, 3, 2, 212),
]


def replanned(shape, N):
    _, C, H, W, M, R, sparsity, few, WS, _ = shape
    L = wl.custom_layer(N, C, H, W, M, R, R, 2, R // 2, sparsity, seed=106, dist="normal")
    d = esc.make_desc(few, C, H, W, M, R, R, 2, R // 2)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    assert esc.plan_header(plan)["WS"] == WS
    return L, plan


@pytest.mark.parametrize("shape", REPLANNED, ids=str)
def test_stride_two_is_taken_for_what_it_is_exact_to(shape):
    """Whatever the batch, the layout's squared error by the rule (nothing is flushed at stride 2) is below the plan's tiled kernel's."""
    _, C, H, W, M, R, sparsity, few, WS, _ = shape
    _, plan = replanned(shape, 1)
    n = esc.plan_header(plan)["pair_nnz"] / M
    taken = {N: esc.escoin_sconv_tiled_kernel(esc.make_desc(N, C, H, W, M, R, R, 2, R // 2), plan) for N in (1, 2, 4, 8, 16, 24, 32, 48, 64, 100, 128, 256)}
    assert taken[shape[0]] == shape[-1]
    for N, kernel in taken.items():
        base, slope = {2: (0.81, 0.0044), 4: (0.81, 0.0020)}.get(kernel % 10, (0, 0))
        assert kernel == 0 or base + slope * n <= 0.95 * 0.0154 / WS * n, (N, kernel)


@gpu
@pytest.mark.parametrize("shape", REPLANNED, ids=str)
def test_stride_two_with_a_plan_for_few_images(oracle, shape):
    print("pair stride 2, plan for few", shape, flush=True)
    L, plan = replanned(shape, shape[0])
    results = []
    for tiled in (False, True):
        if tiled:
            forget(plan, ("pair", "pair_nnz", "off_pair", "off_nz", "pair_least"))
        dl = DeviceLayer(esc, L)
        dl.plan, dl.d_plan = plan, to_dev(plan)
        assert esc.escoin_sconv_tiled_kernel(dl.desc, plan) == (0 if tiled else shape[-1])
        results.append(dl.forward_tiled())
    ref, bound = oracle_full(oracle, L)
    got, chains = results
    assert (np.abs(got - ref) <= limit(L, bound)).all()
    assert np.linalg.norm(got - ref) <= np.linalg.norm(chains - ref)


@pytest.mark.parametrize("shape, kernel", [
    ((32, 18, 42, 42, 75, 5, 2, 0.62), 212),      # 24 us; 266 workgroups of the other kind, one to a compute unit, 35; the tiled kernel 29
    ((63, 358, 30, 30, 39, 5, 2, 0.67), 122),     # 139; 285 workgroups, one to a compute unit, 154
    ((12, 18, 26, 26, 371, 3, 2, 0.30), 114),     # 13 and 18
    ((12, 18, 26, 26, 371, 3, 2, 0.57), 0),       # some rows too short: 16 and 14
    ((37, 377, 29, 29, 171, 3, 1, 0.59), 118),    # 157; 163 with two flushed shares
    ((74, 384, 14, 14, 250, 3, 1, 0.55), 212),
], ids=str)
def test_layers_take_what_they_are_fastest_with(shape, kernel):
    N, C, H, W, M, R, stride, sparsity = shape
    L = wl.custom_layer(1, C, H, W, M, R, R, stride, R // 2, sparsity, seed=3, dist="normal")
    d = esc.make_desc(N, C, H, W, M, R, R, stride, R // 2)
    assert esc.escoin_sconv_tiled_kernel(d, esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)) == kernel


@pytest.mark.parametrize("H, kernel", [(450001, 114), (491519, 114), (493447, 114), (493449, 0), (524287, 0)])
def test_stride_two_keeps_a_round_of_channels_in_32_bits(H, kernel):
    """28 channels of a tall map: a wave asks for the inputs of up to 64 before it holds itself to the last, at byte offsets below 2^31."""
    C, W, M, R = 28, 17, 64, 2
    L = wl.custom_layer(1, C, 16, W, M, R, R, 2, 0, 1 - 78 / 112, seed=107, dist="normal")
    d = esc.make_desc(1, C, 4095, W, M, R, R, 2, 0)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    h = esc.plan_header(plan)
    assert h["pair"] == 1 and esc.escoin_sconv_tiled_kernel(esc.make_desc(100, C, 4095, W, M, R, R, 2, 0), plan) == 114
    tall = esc.make_desc(1, C, H, W, M, R, R, 2, 0)
    E, _ = esc.escoin_output_dims(tall)
    rewrite(plan, H=H, E=E, n_tiles=-(-E // h["TH"]))  # what its own plan, of a gigabyte, says of it
    assert esc.escoin_sconv_tiled_kernel(tall, plan) == kernel
    assert kernel == 0 or 64 * H * W * 4 < 1 << 31


@pytest.mark.parametrize("shape, kernel, most", [
    ((3, 16, 18, 508, 8, 2, 1, 0.2), 141, (1 << 20) - 1),     # 8 workgroups of 512 threads an image
    ((44, 3, 5, 373, 4, 1, 1, 0.5), 212, 14913072),           # 24 positions an image, 64 to each of 3 workgroups of 256
    ((45, 1, 11, 349, 5, 2, 2, 0.5), 212, 14913072),          # ... and at stride 2
], ids=str)
def test_batches_whose_grid_would_not_fit(shape, kernel, most):
    """A launch of 2^32 threads or more is none the runtime takes: such batches go where they went."""
    C, H, W, M, R, stride, pad, sparsity = shape
    L = wl.custom_layer(1, C, H, W, M, R, R, stride, pad, sparsity, seed=108, dist="normal")
    desc = lambda N: esc.make_desc(N, C, H, W, M, R, R, stride, pad)
    plan = esc.escoin_sconv_plan_build(desc(1024), L.rowptr, esc.escoin_sconv_pack(desc(1024), L.rowptr, L.colidx), L.value)
    assert [esc.escoin_sconv_tiled_kernel(desc(N), plan) for N in (most, most + 8)] == [kernel, 0]


# N, C, H, W, M, R, S, pad, stride, sparsity: few channels and an even stride.
FIRST = [
    (6, 3, 224, 224, 64, 7, 7, 3, 2, 0.50),     # whole tiles
    (60, 4, 61, 61, 128, 6, 6, 2, 2, 0.40),     # ragged last tiles; two columns of a group without weights
    (60, 1, 64, 200, 100, 9, 9, 4, 4, 0.10),    # two groups to a filter row; channels over
    (100, 7, 50, 61, 33, 4, 7, 0, 2, 0.40),     # no padding, 28 groups
    (60, 4, 50, 61, 45, 4, 8, 0, 2, 0.30),      # whole groups
    (40, 2, 70, 150, 140, 5, 11, 2, 2, 0.20),   # padding smaller than the reach
    (150, 3, 33, 40, 100, 7, 7, 3, 2, 0.45),    # a tile of nearly all rows; an odd number of groups
]


def cut_rows(L, cut, lengths):
    rows = np.diff(L.rowptr)
    rows[cut] = lengths
    keep = np.concatenate([np.arange(b - a) < k for a, b, k in zip(L.rowptr, L.rowptr[1:], rows)])
    return L.colidx[keep], L.value[keep], np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)


def first_layer(shape):
    N, C, H, W, M, R, S, pad, stride, sparsity = shape
    return wl.custom_layer(N, C, H, W, M, R, S, stride, pad, sparsity, seed=103, dist="normal")


@gpu
@pytest.mark.parametrize("shape", FIRST, ids=str)
def test_few_channels(oracle, shape):
    print("pair few channels", shape, flush=True)
    L = first_layer(shape)
    L.input[:] = np.random.default_rng(104).standard_normal(L.input.shape, dtype=np.float32)
    dl, one = pair_layer(L, 141), DeviceLayer(esc, L, tuning=dict(B=2))
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got, chain = dl.forward_tiled(flags), one.forward_tiled(flags)
        ref, bound = oracle_full(oracle, L, flags)
        assert_within_bound(got, ref, bound, (shape, flags))
        assert (np.abs(got - ref) <= limit(L, bound)).all()
        if flags == 0:
            assert np.linalg.norm(got - ref) <= np.linalg.norm(chain - ref)
    # rows too short for the pairs; inputs past what the others' scale leaves bits for, inputs that lose them, Inf and NaN
    L.input[0, :, shape[2] // 2] *= np.float32(2.0 ** 90)
    L.input[1] *= np.float32(2.0 ** -60)
    L.input[1, 0, 9, 7] = 1.0
    L.input[1, 0, 30:] = 0
    L.input[2, 0, 5, 8] = -np.inf
    L.input[2, 0, 25] = np.nan
    L.colidx, L.value, L.rowptr = cut_rows(L, [1, shape[4] // 2, shape[4] - 1], [33, 40, 48])
    dl = pair_layer(L, 141)
    got = dl.forward_tiled(esc.F_BIAS)
    with np.errstate(invalid="ignore", over="ignore"):
        ref, bound = oracle_full(oracle, L, esc.F_BIAS)
    bad = ~np.isfinite(bound)
    assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
    assert (np.abs(got[~bad] - ref[~bad]) <= limit(L, bound)[~bad]).all()
    short = np.zeros(shape[4], bool)
    short[[1, shape[4] // 2, shape[4] - 1]] = True  # chains of 48 products at most, and the bias
    assert (np.abs(got - ref)[:, short][~bad[:, short]] <= 49 * 2.0 ** -24 * bound[:, short][~bad[:, short]] + 2.0 ** -149).all()


@gpu
@pytest.mark.parametrize("count", [8, 9])
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[3]], ids=str)
def test_a_few_sums_of_tiny_inputs(oracle, shape, count):
    """Positions all of whose inputs lose bits: up to eight of a workgroup are computed from the nonzeros, more send it through its second pass."""
    print("pair tiny sums", shape, count, flush=True)
    L = layer(shape, seed=105)
    s = L.spec
    pitch, plane, positions = s.W + s.pad, (s.H + s.pad) * (s.W + s.pad), 64 * (shape[-1] // 10 % 10)
    group = lambda n, h, w: (n * plane + h * pitch + w) // positions
    h, w = next((h, w) for h in range(5, s.H - 1) for w in range(2, s.W - 1 - count) if group(1, h, w) == group(1, h, w + count - 1))
    L.input[1, :, h - 1:h + 2, w - 1:w + count + 1] *= np.float32(2.0 ** -40)
    tiny = np.ones((s.N, s.H + 2, s.W + 2), bool)  # what lies outside counts as tiny
    tiny[:, 1:-1, 1:-1] = False
    tiny[1, h:h + 3, w:w + count + 2] = True
    at = np.argwhere(np.lib.stride_tricks.sliding_window_view(tiny, (3, 3), axis=(1, 2)).all(axis=(3, 4)))
    assert [group(*p) for p in at] == [group(1, h, w)] * count
    got = pair_layer(L, shape[-1]).forward_tiled(esc.F_RELU)
    ref, bound = oracle_full(oracle, L, esc.F_RELU)
    assert (np.abs(got - ref) <= limit(L, bound)).all()


def test_what_few_channels_leave_to_the_tiled_kernel():
    """Odd strides, rows too short for the pairs to be as exact, single images, tuned plans."""
    for shape, N, kernel in ((FIRST[0], 3, 141), (FIRST[0], 1, 0), (FIRST[6][:-1] + (0.8,), 60, 0), (FIRST[6][:8] + (1, 0.45), 60, 0)):
        L = first_layer((1,) + shape[1:])
        s = L.spec
        d = esc.make_desc(N, s.C, s.H, s.W, s.M, s.R, s.S, s.stride, s.pad)
        stretched = esc.escoin_sconv_pack(d, L.rowptr, L.colidx)
        assert esc.escoin_sconv_tiled_kernel(d, esc.escoin_sconv_plan_build(d, L.rowptr, stretched, L.value)) == kernel
        assert esc.escoin_sconv_tiled_kernel(d, esc.escoin_sconv_plan_build(d, L.rowptr, stretched, L.value, esc.make_tuning(B=2))) == 0


@pytest.mark.parametrize("shape, loads", [
    ((3, 224, 224, 7, 3, 2), 20),     # 63 rows of 229 columns, two at a time by eight waves
    ((3, 240, 240, 7, 3, 2), 20),
    ((3, 256, 256, 7, 3, 2), 33),     # columns of 262: one at a time
    ((3, 448, 448, 7, 3, 2), 33),
    ((4, 224, 224, 7, 3, 2), 26),
    ((3, 227, 227, 11, 0, 4), 47),
    ((3, 512, 512, 7, 3, 2), 0),      # more columns than eight waves have
    ((1, 256, 256, 11, 5, 2), 15),
    ((6, 120, 120, 5, 2, 2), 23),
    ((8, 56, 56, 5, 2, 2), 25),
], ids=str)
def test_how_much_input_few_channels_may_have(shape, loads):
    """A tile's padded rows pass through 24 registers a lane, so many words of a row each; layers of more stay with the tiled kernel."""
    C, H, W, R, pad, stride = shape
    d = esc.make_desc(32, C, H, W, 64, R, R, stride, pad)
    E, F = esc.escoin_output_dims(d)
    rows, columns = (min(E, (254 + F) // F + 1) - 1) * stride + R, (F - 1) * stride + 8 * -(-R // 8)
    together = 8 // -(-columns // 64)
    assert loads == (-(-C * rows // together) if together else 0)
    L = wl.custom_layer(1, C, H, W, 64, R, R, stride, pad, 0.1, seed=109, dist="normal")
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    assert (esc.escoin_sconv_tiled_kernel(d, plan) == 141) == (0 < loads <= 24)


@pytest.mark.parametrize("cut, kernel", [(0, 141), (2, 141), (9, 0), (32, 0)])
def test_short_rows_of_few_channels_count_for_what_they_cost(cut, kernel):
    """12 of 2x236x236, 63 11x11 filters of stride 2: 51 us, 82 with two rows of 76 nonzeros, 121 with nine and 255 with 32; the tiled kernel 122."""
    L = wl.custom_layer(1, 2, 236, 236, 63, 11, 11, 2, 5, 0.3, seed=3, dist="normal")
    at = np.linspace(0, 62, cut).astype(int)
    if cut:
        L.colidx, L.value, L.rowptr = cut_rows(L, at, [76] * cut)
    d = esc.make_desc(12, 2, 236, 236, 63, 11, 11, 2, 5)
    plan = esc.escoin_sconv_plan_build(d, L.rowptr, esc.escoin_sconv_pack(d, L.rowptr, L.colidx), L.value)
    assert esc.plan_header(plan)["pair_few2"] == cut and esc.escoin_sconv_tiled_kernel(d, plan) == kernel


@gpu
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[4]], ids=str)
def test_unaligned_buffers_guards_and_one_plan_for_two_batches(oracle, shape):
    import torch
    print("pair unaligned", shape, flush=True)
    L = layer(shape)
    dl = pair_layer(L, shape[-1])
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
    s = L.spec
    one = esc.make_desc(1, s.C, s.H, s.W, s.M, s.R, s.S, 1, s.pad)
    assert not esc.escoin_sconv_tiled_on_matrix_cores(one, dl.plan)
    dl.d_out.fill_(float("nan"))
    esc.escoin_sconv_forward_tiled(one, dl.plan, dl.d_plan, dl.d_in[:1], dl.d_out[:1])
    assert_within_bound(dl.d_out[:1].cpu().numpy(), ref[:1], bound[:1], shape)
    assert bool(dl.d_out[1:].isnan().all())


@gpu
@pytest.mark.parametrize("power", [-146, -130, -100, -40, 60, 100, 120])
def test_inputs_of_any_size(oracle, power):
    """Everything scaled, down to subnormal inputs; the weights the other way where sums would leave fp32's range."""
    print("pair input scale", power, flush=True)
    L = layer(SMALL, seed=92)
    L.input *= np.float32(2.0) ** np.float32(power / 2)
    L.input *= np.float32(2.0) ** np.float32(power - power / 2)
    L.value *= np.float32(2.0 ** (-20 if power > 0 else 20))
    dl = pair_layer(L, SMALL[-1])
    got = dl.forward_tiled()
    ref, bound = oracle_full(oracle, L)
    assert np.abs(ref).max() > 0 and (np.abs(got - ref) <= limit(L, bound)).all()


@gpu
@pytest.mark.parametrize("late, early", [(2.0 ** 10, 1.0), (2.0 ** 60, 1.0), (1.0, 2.0 ** 40), (1.0, 0.0), (2.0 ** -60, 0.0), (2.0 ** 90, 2.0 ** -60)])
def test_channels_of_different_sizes(oracle, late, early):
    """The scale is taken from the first channels: later ones are far larger or smaller, beside zeros, in some images."""
    print("pair channel sizes", late, early, flush=True)
    L = layer(SHAPES[2], seed=93)
    L.input[::3, :40] *= np.float32(early)
    L.input[::3, 40:] *= np.float32(late)
    dl = pair_layer(L, SHAPES[2][-1])
    for flags in (0, esc.F_BIAS):
        got = dl.forward_tiled(flags)
        ref, bound = oracle_full(oracle, L, flags)
        assert (np.abs(got - ref) <= limit(L, bound)).all()


@gpu
def test_small_values_beside_large_ones(oracle):
    """Outputs that meet only inputs 2^-40 to 2^-120 of others in their window, or zeros."""
    print("pair small beside large", flush=True)
    L = layer(SMALL, seed=94)
    rng = np.random.default_rng(94)
    L.input[:] *= np.float32(2.0) ** rng.integers(-120, -40, size=(L.spec.N, 1, 1, 1)).astype(np.float32)
    L.input[:, :, 5, 7] = 1.0
    L.input[3] = 0
    dl = pair_layer(L, SMALL[-1])
    got = dl.forward_tiled()
    ref, bound = oracle_full(oracle, L)
    assert (np.abs(got - ref) <= limit(L, bound)).all() and not got[3].any()


@gpu
def test_results_around_the_largest_float(oracle):
    print("pair overflow", flush=True)
    L = layer(SMALL, seed=95)
    L.input[:] = 0
    for image, x in ((3, 3e38), (9, 1e38), (32, -3e38)):
        L.input[image, image, 5, 6] = x
    L.value *= np.float32(40)
    with np.errstate(over="ignore"):
        ref, bound = oracle_full(oracle, L)
        ref = ref.astype(np.float32).astype(np.float64)
    got = pair_layer(L, SMALL[-1]).forward_tiled()
    over = np.isinf(ref)
    assert over.any() and (got[over] == ref[over]).all()
    assert (np.abs(got[~over] - ref[~over]) <= limit(L, bound)[~over]).all()


@gpu
@pytest.mark.parametrize("where", ["a word", "a row", "a column", "an image", "every image"])
def test_non_finite_inputs_reach_only_nonzero_weights(oracle, where):
    print("pair non-finite", where, flush=True)
    L = layer(SMALL, seed=96)
    place = {"a word": np.s_[2, 0, 0, 0], "a row": np.s_[3, 7, 4], "a column": np.s_[32, 7, :, 16], "an image": np.s_[20, 11],
             "every image": np.s_[:, 48]}
    L.input[place[where]] = np.inf
    L.input[1, 0, 0, 0] = np.nan
    L.input[5, 48, 18, 22] = 3.4e38
    dl = pair_layer(L, SMALL[-1])
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got = dl.forward_tiled(flags)
        with np.errstate(invalid="ignore", over="ignore"):
            ref, bound = oracle_full(oracle, L, flags)
        bad = ~np.isfinite(bound)            # an output that met one; ReLU may have made it finite
        assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
        assert (np.abs(got[~bad] - ref[~bad]) <= 1e-4 * bound[~bad]).all()


@gpu
def test_captured_calls_replay(oracle):
    """One launch, no memset: replays give the same bits as eager calls, with eager work between them."""
    import torch
    print("pair capture", flush=True)
    L = layer(SMALL, seed=97)
    dl = pair_layer(L, SMALL[-1])
    want = torch.from_numpy(dl.forward_tiled()).cuda()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        esc.escoin_sconv_forward_tiled(dl.desc, dl.plan, dl.d_plan, dl.d_in, dl.d_out, stream=torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        dl.d_out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dl.d_out, want)
        assert bool((dl.d_out * 2).isfinite().all())


@gpu
def test_outputs_from_the_nonzeros_past_four_giga_words(oracle):
    """Inputs of more than 2^32 words: what the last images' outputs need from the nonzeros is read from those images."""
    import torch
    print("pair, 2^32 words", flush=True)
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 35 GB")
    N, last = 86000, 6
    L = wl.custom_layer(last, 64, 28, 28, 64, 3, 3, 1, 1, 0.75, seed=98, dist="normal")
    assert (N - last) * L.input[0].size > 1 << 32
    L.input[2, 5, 7, 9] = np.inf
    L.input[3, 40, :, 3] = np.nan
    L.input[4] *= np.float32(2.0 ** -30)
    L.input[4, 9, 20, 20] = 1.0
    ref_d = esc.make_desc(40, 64, 28, 28, 64, 3, 3, 1, 1)
    plan = esc.escoin_sconv_plan_build(ref_d, L.rowptr, esc.escoin_sconv_pack(ref_d, L.rowptr, L.colidx), L.value)
    d = esc.make_desc(N, 64, 28, 28, 64, 3, 3, 1, 1)
    assert esc.escoin_sconv_tiled_kernel(d, plan) > 1
    d_in = torch.zeros((N, 64, 28, 28), device="cuda")
    d_in[N - last:] = to_dev(L.input)
    d_out = torch.full((N, 64, 28, 28), float("nan"), device="cuda")
    esc.escoin_sconv_forward_tiled(d, plan, to_dev(plan), d_in, d_out)
    torch.cuda.synchronize()
    for at in range(0, N - last, 1 << 13):
        assert not d_out[at:min(at + (1 << 13), N - last)].any()
    got = d_out[N - last:].cpu().numpy()
    with np.errstate(invalid="ignore", over="ignore"):
        ref, bound = oracle_full(oracle, L)
    bad = ~np.isfinite(bound)
    assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
    assert (np.abs(got[~bad] - ref[~bad]) <= 1e-4 * bound[~bad]).all()


@gpu
@pytest.mark.parametrize("shape", SHORT, ids=str)
def test_short_rows_are_as_exact_as_fp32_sums(oracle, shape):
    print("pair short rows", shape, flush=True)
    L, cut = short_layer(shape)
    L.input[1, 3, 2, 4] = np.inf                   # the window's other outputs, and its second pass
    L.input[2, :, 5] *= np.float32(2.0 ** 12)
    dl, one = DeviceLayer(esc, L), DeviceLayer(esc, L, tuning=dict(B=2))
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        got, chain = dl.forward_tiled(flags), one.forward_tiled(flags)
        assert esc.escoin_sconv_tiled_kernel(dl.desc, dl.plan) > 1 and esc.escoin_sconv_tiled_kernel(one.desc, one.plan) == 0
        with np.errstate(invalid="ignore", over="ignore"):
            ref, bound = oracle_full(oracle, L, flags)
        bad = ~np.isfinite(bound)
        assert bad.any() and np.array_equal(got[bad], ref[bad], equal_nan=True)
        assert (np.abs(got[~bad] - ref[~bad]) <= limit(L, bound)[~bad]).all()
        # four chains of a row's products, their sum and the bias: n / 4 + 5 roundings; as a whole no further off than one chain
        n = np.diff(L.rowptr)[cut]
        ok = ~bad[:, cut]
        err, roundings = np.abs(got[:, cut][ok] - ref[:, cut][ok]), np.broadcast_to((n / 4 + 5)[:, None, None], ok.shape)[ok]
        assert (err <= roundings * 2.0 ** -24 * bound[:, cut][ok] + 2.0 ** -149).all()
        if flags == 0:
            assert np.linalg.norm(err) <= np.linalg.norm(chain[:, cut][ok] - ref[:, cut][ok])


@gpu
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[7]], ids=str)
def test_plans_saved_before_give_the_same_layer(oracle, shape):
    print("pair old plan", shape, flush=True)
    L = layer(shape)
    dl = pair_layer(L, shape[-1])
    ref, bound = oracle_full(oracle, L)
    forget(dl.plan, ("pair", "pair_nnz", "off_pair", "off_nz", "pair_least"))
    dl.d_plan = to_dev(dl.plan)
    assert esc.escoin_sconv_tiled_kernel(dl.desc, dl.plan) < 2
    assert_within_bound(dl.forward_tiled(), ref, bound, shape)


@gpu
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[5], SHAPES[6], SHAPES[10]], ids=str)
def test_outputs_of_few_products(oracle, shape):
    """Sparse inputs: an output of k products is off by 2^-21 of each at most, and by a rounding of the sum for each of them and of the
    waves' shares; where the input is a power of two, by the weight's own pair alone, 2^-23 of it."""
    print("pair few products", shape, flush=True)
    L = layer(shape, seed=100)
    N, C, H, W = L.input.shape
    rng = np.random.default_rng(100)
    L.input *= rng.random(L.input.shape) < 0.01
    L.input[0] = L.input[1] = 0
    for y in range(1, H, 5):  # one input in reach of any output
        for x in range(1, W, 5):
            L.input[0, rng.integers(C), y, x] = 1.0
            L.input[1, rng.integers(C), y, x] = -2.0 ** rng.integers(0, 8)
    got = pair_layer(L, shape[-1]).forward_tiled().astype(np.float64)
    ref, bound = oracle_full(oracle, L)
    s = L.spec
    kept = oracle.csr_to_dense(s.M, s.C, s.R, s.S, L.rowptr, L.colidx, (L.value != 0).astype(np.float32))
    k, _ = oracle.conv((L.input != 0).astype(np.float32), kept, s.stride, s.pad)
    one = k[:2] <= 1
    assert one.mean() > 0.9 and (np.abs(got - ref)[:2] <= 2.0 ** -23 * bound[:2])[one].all() and not got[k == 0].any()
    assert (np.abs(got - ref) <= (2.0 ** -21 + 2.0 ** -24 * (k + shape[-1] % 10)) * bound).all()
