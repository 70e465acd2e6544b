"""Units that share a launch: short rows, ragged tails and unquantized tensors behind full tiles, behind wide groups, and
in the short-list kernel (at most 44 tensors, every class of group in one launch).  The comparison bar is the one of
tests/gpu_util.py: the same fp32 sequence on both sides, so no code, scale or state bit may differ."""
import pytest
import torch

import oracle
import workloads
from gpu_util import bf16_bits, bytes_per_element, compare, host_copy, oracle_step, step_config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = workloads.TensorSpec


def short_rows(fmt):
    """Groups of 8 .. 504 elements that are no power of two: one lane to 63, rows that fill a wave's last lane and that
    do not, tensors of fewer rows than a wave takes, a ragged last unit."""
    shapes = [(130, 8), (65, 16), (43, 24), (13, 40), (25, 96), (6, 120), (5, 168), (3, 336), (4, 384), (3, 504), (2, 248), (1, 72)]
    return [T(f"r{c}", (r, c), fmt, grad_std=1e-3 * (1 + c % 3), granularity="row") for r, c in shapes]


def lists(which, fmt):
    plain = [T(f"p{n}", (n,), "bf16_plain") for n in (1, 511, 512, 1027)]
    tails = [T(f"t{n}", (n,), fmt) for n in (1, 127, 300, 511)]
    if which == "tiles":                   # a full-tile launch, more tensors than the short-list kernel takes
        return short_rows(fmt) + plain + tails + [T(f"b{i}", (1024 + 8 * i + i % 3,), fmt) for i in range(40)]
    if which == "wide":                    # no full tile: the units ride in the launch of the wide groups
        return short_rows(fmt) + plain + tails + [T(f"w{i}", (1 + i % 5, 1408), fmt, granularity="row") for i in range(40)]
    if which == "short":                   # several launches' worth of classes in one
        wide = [T(f"w{c}_{r}", (r, c), fmt, granularity="row") for r, c in
                ((8, 576), (5, 1408), (8, 1408), (3, 8192), (7, 520), (2, 6912), (33, 1024), (9, 2048))]
        return short_rows(fmt) + plain + tails + wide + [T("b", (3, 700), fmt), T("b2", (4096,), fmt)]
    return short_rows(fmt)                 # one-wave units alone


@pytest.mark.parametrize("which", ["tiles", "wide", "short", "rows"])
@pytest.mark.parametrize("fmt,bf16,over", [("fp8", False, {}), ("fp8", True, dict(mode=3, weight_decay=0.1)), ("int4", True, {}),
                                           ("int4", False, dict(opt=1, round=1, lr=0.05)), ("fp8", False, dict(opt=1, mode=2, lr=0.05))])
def test_units_that_share_a_launch(which, fmt, bf16, over):
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    wl = workloads.Workload("share_" + which, lists(which, fmt), steps=2, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    for k in (1, 2):
        dw.fill_gradients(k)
        hp = dw.hparams(k)
        for tv, h in zip(dw.tensors, host):
            h["grad"] = bf16_bits(tv.grad)
        dw.plan.step(hp)
        torch.cuda.synchronize()
        for tv, h in zip(dw.tensors, host):
            oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
            st = compare(host_copy(tv), h, f"{which} step {k} {tv.spec.name}", bf16)
            assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


def grouped(numel, group, fmt):
    """A tensor of any length in scale groups of any length: the last one may be cut off, within a lane's 8 elements too."""
    t = T(f"g{group}_{numel}", (numel,), fmt, grad_std=1e-3 * (1 + numel % 3), granularity="row")
    t.group_size = lambda block_size: group
    return t


@pytest.mark.parametrize("fmt,bf16,over", [("fp8", False, {}), ("fp8", True, dict(mode=3, weight_decay=0.1)), ("int4", True, {}),
                                           ("int4", False, dict(opt=1, round=1, lr=0.05)), ("fp8", False, dict(opt=1, mode=2, lr=0.05)),
                                           ("fp8", False, dict(eps=0.0)), ("fp8", True, {}), ("int4", False, dict(opt=1, mode=3, lr=0.05))])
@pytest.mark.parametrize("path", ["classes", "list", "own_list", "noalloc"])
def test_rows_that_leave_lanes_idle(path, fmt, bf16, over):
    """Rows of which several share a workgroup and rows that have one to themselves, their last waves part idle: numbers of rows
    that fill the last workgroup and that do not, a last row that is cut off behind a whole piece of 8 elements and within one;
    and tensors of any length with one scale that are one group.  In a launch for each class of group (a large tensor beside
    them), in one launch with a plan's tables, and in launches of 44 with the descriptors as arguments.  From 96 MB of arrays on rows
    are grouped in another way, with idle lanes: in a launch for each class, and in one launch beside a large tensor of the other format."""
    from paper_2601_22101_amd import binding as eco
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    specs = [grouped(n, g, fmt) for g in (520, 576, 664, 720, 800, 896, 1000, 1152, 1280, 1408, 1800, 2304, 2816, 8000)
             for n in (g, 2 * g, 4 * g, 7 * g, 3 * g + 8, 2 * g + 5, 5 * g - 3)]
    specs += [grouped(n, n, fmt) for n in (1, 5, 100, 511, 513, 1001, 4097, 8191)] + [T(f"p{n}", (n,), "bf16_plain") for n in (7, 1027)]
    specs += [grouped(1000, 24, fmt), grouped(700, 336, fmt), grouped(1500, 128, fmt)]
    other = "int4" if fmt == "fp8" else "fp8"
    if path in ("classes", "own_list"):
        which = fmt if path == "classes" else other
        rows = max(9000, int(100e6 / bytes_per_element(which, bf16, over) / 1024) + 1)
        specs.append(T("large", (rows, 1024), which, granularity="row"))
        assert rows * 1024 > 1 << 23 and rows * 1024 * bytes_per_element(which, bf16, over) > 96e6
    wl = workloads.Workload("idle_lanes", specs, steps=2, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    for k in (1, 2):
        dw.fill_gradients(k)
        hp = dw.hparams(k)
        for tv, h in zip(dw.tensors, host):
            tv.grad[tv.grad == 0] = 1e-4              # (with eps = 0 a gradient of zero in the first step is 0 / 0)
            h["grad"] = bf16_bits(tv.grad)
        if path == "noalloc":
            eco.eco_step_tensors_noalloc([dw.descriptor(tv) for tv in dw.tensors], hp)
        else:
            dw.plan.step(hp)
        torch.cuda.synchronize()
        for tv, h in zip(dw.tensors, host):
            oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
            st = compare(host_copy(tv), h, f"step {k} {tv.spec.name}", bf16)
            assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("others", [False, True])
@pytest.mark.parametrize("fmt,bf16,over", [("fp8", False, {}), ("int4", True, dict(round=1)), ("fp8", False, dict(mode=3)), ("int4", False, dict(opt=1, lr=0.05))])
def test_short_tensors_of_odd_length_along_with_longer_ones(fmt, bf16, over, others, noalloc):
    """One scale each: lengths from 1 to 8191 that are no multiple of 8, in the launches of tensors beyond 8192 elements; tensors of
    other kinds in the list or none."""
    from paper_2601_22101_amd import binding as eco
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    specs = [grouped(n, n, fmt) for n in (1, 5, 7, 9, 511, 513, 770, 2627, 8191, 8193, 11942, 100003)]
    if others:
        specs += [T("p", (700,), "bf16_plain"), grouped(2304, 1152, fmt), grouped(800, 800, fmt), grouped(3000, 1000, fmt)]
    wl = workloads.Workload("odd_along", specs, steps=2, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    for k in (1, 2):
        dw.fill_gradients(k)
        hp = dw.hparams(k)
        for tv, h in zip(dw.tensors, host):
            h["grad"] = bf16_bits(tv.grad)
        if noalloc:
            eco.eco_step_tensors_noalloc([dw.descriptor(tv) for tv in dw.tensors], hp)
        else:
            dw.plan.step(hp)
        torch.cuda.synchronize()
        for tv, h in zip(dw.tensors, host):
            oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
            st = compare(host_copy(tv), h, f"step {k} {tv.spec.name}", bf16)
            assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


@pytest.mark.parametrize("opt", [0, 1])
@pytest.mark.parametrize("fmt,bf16", [("fp8", False), ("int4", True), ("int4", False)])
def test_master_weights_with_one_scale_in_two_passes(fmt, bf16, opt):
    """Pass 1 stores the master weights and the moments, pass 2 reads the former alone: whole and partial last tiles, a last piece of 8
    elements that is cut off (such a tail keeps the list, a short one, out of the one-pass form)."""
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    specs = [grouped(n, n, fmt) for n in (8193, 8200, 512 * 17, 512 * 17 + 5, 100003)]
    wl = workloads.Workload("master_two_passes", specs, steps=2, state_bf16=bf16, scale_bf16=bf16, lr=1e-3 if opt == 0 else 0.05)
    dw = harness.DeviceWorkload(wl, DEV, layout=dict(opt=opt, mode=3, weight_decay=0.1))
    host = [host_copy(tv) for tv in dw.tensors]
    for k in (1, 2):
        dw.fill_gradients(k)
        hp = dw.hparams(k)
        for tv, h in zip(dw.tensors, host):
            h["grad"] = bf16_bits(tv.grad)
        dw.plan.step(hp)
        torch.cuda.synchronize()
        for tv, h in zip(dw.tensors, host):
            oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
            st = compare(host_copy(tv), h, f"step {k} {tv.spec.name}", bf16)
            assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


@pytest.mark.parametrize("opt", [0, 1])
@pytest.mark.parametrize("noalloc", [False, True])
def test_identity_weights_step_alike_alone_and_beside_quantized_tensors(opt, noalloc):
    from paper_2601_22101_amd import binding as eco
    gen = torch.Generator(device=DEV).manual_seed(4)
    n = 1500
    arr = lambda scale: torch.randn(n, generator=gen, device=DEV) * scale  # noqa: E731
    w, m, v, grad = arr(0.02), arr(1e-3), arr(1e-3).square(), arr(1e-3).to(torch.bfloat16)
    hp = eco.make_hparams(opt=opt, step=7, weight_decay=0.1)
    got = []
    for beside in (False, True):
        mine = [x.clone() for x in (w, m, v)]
        ts = [eco.make_tensor(mine[0], None, grad, mine[1], mine[2], n, 0, eco.ECO_FMT_FP32_IDENTITY)]
        if beside:
            q = [torch.zeros(n, dtype=torch.uint8, device=DEV), torch.ones(12, device=DEV), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)]
            ts.append(eco.make_tensor(q[0], q[1], grad, q[2], q[3], n, 1, eco.ECO_FMT_FP8_E4M3))
        if noalloc:
            eco.eco_step_tensors_noalloc(ts, hp)
        else:
            with eco.Plan(ts, hp) as plan:
                plan.step(hp)
        torch.cuda.synchronize()
        got.append(mine)
    assert not torch.equal(got[0][0], w)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("fmt,scale_bf16", [(0, False), (1, True)])
@pytest.mark.parametrize("src_bf16", [False, True])
@pytest.mark.parametrize("numel", [5, 509, 513, 8191, 8201, 256 * 8 * 3 + 1, 1024 * 8 * 256 + 8, 1024 * 8 * 256 * 5 + 4099])
def test_tensor_wise_quantizer_at_the_edges_of_its_shares(fmt, scale_bf16, src_bf16, numel):
    """One partial maximum per 8192 elements up to 256 of them, then several turns to a workgroup; the largest element in
    the first and in the last place."""
    import numpy as np

    from paper_2601_22101_amd import binding as eco
    o32 = oracle.get("f32")
    gen = torch.Generator(device=DEV).manual_seed(numel)
    for at in (0, numel - 1):
        x = torch.randn(numel, generator=gen, device=DEV) * 0.02
        x[at] = -0.5
        src = x.to(torch.bfloat16) if src_bf16 else x
        codes = torch.zeros(numel if fmt == 0 else (numel + 1) // 2, dtype=torch.uint8, device=DEV)
        scales = torch.zeros(1, dtype=torch.bfloat16 if scale_bf16 else torch.float32, device=DEV)
        eco.eco_quantize_init(src, int(src_bf16), numel, fmt, numel, int(scale_bf16), codes, scales)
        rc, rs = o32.quantize_rtn(oracle.FMT_E4M3 if fmt == 0 else oracle.FMT_INT4, src.float().cpu().numpy(), numel, scale_bf16=scale_bf16)
        assert np.array_equal(codes.cpu().numpy(), rc) and float(scales.float()[0]) == float(rs[0])


@pytest.mark.parametrize("numel", [8200, 8201, 1024 * 8 * 256 * 4 + 8])
def test_tensor_wise_quantizer_folds_not_a_number_as_the_groups_in_a_wave_do(numel):
    """Eight elements of a lane: NaN among numbers is passed over, NaN alone makes the group's maximum NaN and with it the
    scale zero; infinity is the maximum.  The same array with a scale for every 32 elements says what a group of each does."""
    from paper_2601_22101_amd import binding as eco
    x = torch.full((numel,), 0.25, device=DEV)
    for at in (0, 8 * 1023, numel // 8 * 8 - 8):
        for bad, width in ((float("nan"), 1), (float("nan"), 7), (float("nan"), 8), (float("inf"), 1)):
            src = x.clone()
            src[at:at + width] = bad
            codes, one, many = torch.zeros(numel, dtype=torch.uint8, device=DEV), torch.zeros(1, device=DEV), torch.zeros(-(-numel // 32), device=DEV)
            eco.eco_quantize_init(src, 0, numel, 0, numel, 0, codes, one)
            eco.eco_quantize_init(src, 0, numel, 0, 32, 0, codes, many)
            want = 0.0 if width == 8 else bad if bad == bad else float(torch.tensor(0.25) / 448)
            assert float(one[0]) == float(many[at // 32]) == want, (at, bad, width)


@pytest.mark.parametrize("group", [8, 48, 248, 256, 264, 400, 504, 512, 520, 576, 768, 896, 1024, 1152, 1408, 1664, 1920, 2304, 6912, 8192])
@pytest.mark.parametrize("fmt,scale_bf16,src_bf16", [(0, False, False), (1, True, True)])
def test_quantizer_of_rows(group, fmt, scale_bf16, src_bf16):
    """One group to a wave from 264 elements on, several below; one to a workgroup from 520 on, or several that fill a whole
    number of waves; numbers of rows that are and are not whole bundles, the last one ragged, the only one ragged."""
    import numpy as np

    from paper_2601_22101_amd import binding as eco
    o32 = oracle.get("f32")
    gen = torch.Generator(device=DEV).manual_seed(group)
    for numel in (group * 40, group * 37, group * 37 + 8, group * 3 + group // 2 + 3, group - 3):
        if eco_group_is_whole(group, numel):
            continue
        x = torch.randn(numel, generator=gen, device=DEV) * torch.logspace(-3, 0, numel, device=DEV)
        src = x.to(torch.bfloat16) if src_bf16 else x
        n_scales = -(-numel // group)
        codes = torch.zeros(numel if fmt == 0 else (numel + 1) // 2, dtype=torch.uint8, device=DEV)
        scales = torch.full((n_scales + 8,), 7.0, dtype=torch.bfloat16 if scale_bf16 else torch.float32, device=DEV)
        eco.eco_quantize_init(src, int(src_bf16), numel, fmt, group, int(scale_bf16), codes, scales)
        rc, rs = o32.quantize_rtn(oracle.FMT_E4M3 if fmt == 0 else oracle.FMT_INT4, src.float().cpu().numpy(), group, scale_bf16=scale_bf16)
        assert np.array_equal(codes.cpu().numpy(), rc), numel
        assert np.array_equal(scales.float().cpu().numpy()[:n_scales], rs.astype(np.float32)) and bool((scales[n_scales:] == 7).all()), numel


def eco_group_is_whole(group, numel):
    """A tensor shorter than its group, of a length that is no multiple of 8, has one scale and no groups."""
    return numel < group and numel % 8 != 0


@pytest.mark.parametrize("group", [9, 13, 100, 768, 1000, 1500, 3 * 4096])
@pytest.mark.parametrize("fmt", [0, 1])
def test_dequantizer_finds_the_group_of_every_element(fmt, group):
    """Group lengths that are no power of two, multiples of 8 or not: all codes 1.0 (4 in INT4: 4.0) and scales that name
    their group."""
    from paper_2601_22101_amd import binding as eco
    n = 300 * group + group // 2
    groups = -(-n // group)
    codes = torch.full((n if fmt == 0 else (n + 1) // 2,), 0x38 if fmt == 0 else 0x44, dtype=torch.uint8, device=DEV)
    scales = torch.arange(1, groups + 1, device=DEV, dtype=torch.float32)
    out = torch.zeros(n, device=DEV)
    eco.eco_dequantize(codes, scales, n, fmt, group, 0, out)
    ref = scales.repeat_interleave(group)[:n] * (1.0 if fmt == 0 else 4.0)
    assert torch.equal(out, ref)
    src = torch.randn(n, device=DEV)
    err = torch.zeros(n, device=DEV)
    eco.eco_quantize_error(src, 0, codes, scales, n, fmt, group, 0, err)
    assert torch.equal(err, src - ref)


@pytest.mark.parametrize("src_bf16,numel", [(0, (1 << 24) - 8), (0, (1 << 24) + 1027), (1, (1 << 28) - 8), (1, (1 << 28) + 1027)])
def test_quantization_error_either_side_of_its_long_form(src_bf16, numel):
    from paper_2601_22101_amd import binding as eco
    group = 1000
    codes = torch.full((numel,), 0x38, dtype=torch.uint8, device=DEV)                     # 1.0
    scales = torch.rand(-(-numel // group), device=DEV)
    src = torch.randn(numel, device=DEV).to(torch.bfloat16 if src_bf16 else torch.float32)
    err = torch.full((numel + 8,), 7.0, device=DEV)
    eco.eco_quantize_error(src, src_bf16, codes, scales, numel, 0, group, 0, err)
    assert torch.equal(err[:numel], src.float() - scales.repeat_interleave(group)[:numel])
    assert bool((err[numel:] == 7).all())
