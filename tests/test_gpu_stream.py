"""Steps whose arrays come from HBM (310 MB and more with fp32 state, 384 MB with bf16) load and store past the caches, and waves exchange
halves of their fp32 pieces to do it: every class of scale group and of unit, whole and partial waves, pieces that are cut off, beside
a large tensor that takes the step over the line.  The comparison bar is the one of tests/gpu_util.py, and no bit may differ."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_util import bf16_bits, bytes_per_element, compare, host_copy, oracle_step, step_config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = workloads.TensorSpec


def grouped(numel, group, fmt):
    t = T(f"g{group}_{numel}", (numel,), fmt, grad_std=1e-3 * (1 + numel % 3), granularity="row")
    t.group_size = lambda block_size: group
    return t


def small(fmt):
    """Full tiles and every cut of the last one that matters: within a lane's piece, at a lane's end, in the wave's first and second half."""
    tiles = [T(f"t{n}", (n,), fmt) for n in (512, 1024 + 8, 512 + 255, 512 + 256, 512 + 257, 2048 + 509, 3, 5 * 512 + 264)]
    # units of whole lines and of parts of lines; last rows that are cut off
    rows = [grouped(n * g - cut, g, fmt) for g in (64, 192, 200, 320, 384, 576, 1024, 1056, 1152, 1408, 2048, 2304, 4096, 6912)
            for n, cut in ((5, 0), (9, 3), (4, 8))]
    plain = [T(f"p{n}", (n,), "bf16_plain") for n in (1, 511, 512, 1027)]
    return tiles + rows + plain


@pytest.mark.parametrize("home", ["tiles", "rows", "plain"])
@pytest.mark.parametrize("fmt,bf16,over", [("fp8", False, {}), ("fp8", False, dict(mode=3, weight_decay=0.1)), ("int4", True, {}),
                                           ("fp8", True, dict(opt=1, mode=3, lr=0.05)), ("int4", False, dict(opt=1, round=1, lr=0.05)),
                                           ("fp8", False, dict(opt=1, mode=2, lr=0.05))])
def test_steps_past_the_caches(home, fmt, bf16, over):
    """home: what the large tensor is, and with it which launch the one-wave units ride in."""
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    state = (2 if bf16 else 4) * (1 if over.get("opt") else 2)
    n = int(400e6 / (state + 4 if home == "plain" else bytes_per_element(fmt, bf16, over)))
    big = T("big", (n,), "bf16_plain") if home == "plain" else T("big", (n,), fmt) if home == "tiles" else grouped(n // 2048 * 2048, 2048, fmt)
    specs = [t for t in small(fmt) if home != "rows" or not t.name.startswith("t")]
    wl = workloads.Workload("stream_" + home, specs + [big], steps=2, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    views = dw.tensors if home != "plain" else dw.tensors[:-1]
    host = [host_copy(tv) for tv in views]
    for k in (1, 2):
        dw.fill_gradients(k)
        hp = dw.hparams(k)
        for tv, h in zip(views, host):
            h["grad"] = bf16_bits(tv.grad)
        dw.plan.step(hp)
        torch.cuda.synchronize()
        for tv, h in zip(views, host):
            if k == 2 and tv.spec.name == "big":
                continue
            oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv) if h.get("codes") is not None else 0))
            st = compare(host_copy(tv), h, f"{home} step {k} {tv.spec.name}", bf16)
            assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


@pytest.mark.parametrize("off", [8, 32])
def test_arrays_that_begin_off_a_line(off):
    """Arrays at 16 and 64 bytes past a line, without a plan: stepped the usual way, with the same results as arrays on lines."""
    from paper_2601_22101_amd import binding as eco
    n = 29_000_001
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    base = {"w": torch.randint(0, 120, (n,), generator=gen, device=DEV, dtype=torch.uint8), "s": torch.full((n // 128 + 1,), 1e-4, device=DEV),
            "g": (torch.randn(n, generator=gen, device=DEV) * 1e-3).to(torch.bfloat16), "m": torch.randn(n, generator=gen, device=DEV) * 1e-3,
            "v": torch.rand(n, generator=gen, device=DEV) * 1e-6 + 1e-9}
    out = []
    for shift in (0, off):
        x = {k: torch.cat([t.new_zeros(shift * 2 if k == "w" else shift), t])[shift * 2 if k == "w" else shift:] for k, t in base.items()}
        t = eco.make_tensor(x["w"], x["s"], x["g"], x["m"], x["v"], n, 7, eco.ECO_FMT_FP8_E4M3)
        eco.eco_step_tensors_noalloc([t], eco.make_hparams(step=3, seed=11))
        torch.cuda.synchronize()
        out.append(x)
    for k in base:
        assert torch.equal(out[0][k].contiguous().view(torch.uint8), out[1][k].contiguous().view(torch.uint8)), k


@pytest.mark.parametrize("longer", [False, True])
@pytest.mark.parametrize("fmt,bf16,over", [("fp8", False, {}), ("fp8", False, dict(mode=3, weight_decay=0.1)), ("int4", True, {}),
                                           ("fp8", False, dict(opt=1, mode=2, lr=0.05))])
def test_one_scale_per_tensor_past_the_caches(longer, fmt, bf16, over):
    """In one pass and in two: tensors that end within a slab, within a wave's tile and within a lane's piece."""
    from paper_2601_22101_amd import harness
    o32 = oracle.get("f32")
    n = int(420e6 / bytes_per_element(fmt, bf16, over))
    sizes = [n] if longer else [n // 16 + d for d in (0, 8, 256, 264, -8, 1)] + [n // 16 // 6144 * 6144] * 10
    specs = [T(f"l{k}_{m}", (m,), fmt, granularity="tensor") for k, m in enumerate(sizes + [6144, 300_000, 300_003, 70_000])]
    wl = workloads.Workload("stream_tensorwise", specs, steps=1, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    dw.fill_gradients(1)
    hp = dw.hparams(1)
    for tv, h in zip(dw.tensors, host):
        h["grad"] = bf16_bits(tv.grad)
    dw.plan.step(hp)
    torch.cuda.synchronize()
    for tv, h in zip(dw.tensors, host):
        oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
        st = compare(host_copy(tv), h, f"{tv.spec.name}", bf16)
        assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec.name, st)
    dw.close()


def _quantized(eco, src, fmt, group, scale_dtype, step):
    """Codes, scales, errors and de-quantized values of src, in calls of `step` elements."""
    n, per = src.numel(), 1 if fmt == eco.ECO_FMT_FP8_E4M3 else 2
    sd, dt = (eco.ECO_DT_BF16, torch.bfloat16) if scale_dtype else (eco.ECO_DT_FP32, torch.float32)
    out = {"w": torch.zeros(-(-n // per), dtype=torch.uint8, device=DEV), "s": torch.zeros(-(-n // group), dtype=dt, device=DEV),
           "e": torch.zeros(n, device=DEV), "d": torch.zeros(n, device=DEV)}
    kind = eco.ECO_DT_BF16 if src.dtype == torch.bfloat16 else eco.ECO_DT_FP32
    for at in range(0, n, step):
        m = min(step, n - at)
        w, s = out["w"][at // per:], torch.zeros(-(-m // group), dtype=dt, device=DEV)
        eco.eco_quantize_init(src[at:], kind, m, fmt, group, sd, w, s)
        eco.eco_quantize_error(src[at:], kind, w, s, m, fmt, group, sd, out["e"][at:])
        eco.eco_dequantize(w, s, m, fmt, group, sd, out["d"][at:])
        out["s"][at // group:at // group + s.numel()] = s
    return out


@pytest.mark.parametrize("src_bf16", [False, True])
@pytest.mark.parametrize("fmt,scale_bf16", [(0, False), (1, True)])
@pytest.mark.parametrize("group", [32, 512, 200, 320, 576, 1000, 1152, 2048, 6912])
def test_quantizer_past_the_caches(group, fmt, scale_bf16, src_bf16):
    """Whole arrays, past the caches, against the same in slices, the usual way: no bit may differ, infinities and NaN among the values.
    The last group has 5 elements, a hundredth of those before them, and it and its neighbours are also compared with the oracle."""
    from paper_2601_22101_amd import binding as eco
    step = 20_000_000 // (group * 32) * (group * 32)                 # slices of whole groups that begin on 16 bytes
    n = int(340e6 / ((2 if src_bf16 else 4) + (0.5 if fmt else 1))) // group * group + 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(group)
    src = torch.randn(n, generator=gen, device=DEV) * 0.02
    src[torch.randint(0, n - 8 * group, (50,), generator=gen, device=DEV)] = float("nan")
    src[torch.randint(0, n - 8 * group, (50,), generator=gen, device=DEV)] = float("inf")
    src[group * 7:group * 8] = float("nan")
    src[-5:] *= 0.01
    src = src.to(torch.bfloat16) if src_bf16 else src
    a, b = (_quantized(eco, src, eco.ECO_FMT_INT4 if fmt else eco.ECO_FMT_FP8_E4M3, group, scale_bf16, k) for k in (n, step))
    for key in a:
        assert torch.equal(a[key].view(torch.uint8), b[key].view(torch.uint8)), key
    rc, rs = oracle.get("f32").quantize_rtn(oracle.FMT_INT4 if fmt else oracle.FMT_E4M3, src[-5 - 4 * group:].float().cpu().numpy(), group, scale_bf16=scale_bf16)
    assert np.array_equal(a["w"][-rc.size:].cpu().numpy(), rc)
    assert np.array_equal(a["s"][-5:].float().cpu().numpy(), rs.astype(np.float32))


@pytest.mark.parametrize("src_bf16", [False, True])
@pytest.mark.parametrize("fmt,scale_bf16", [(0, False), (1, True)])
@pytest.mark.parametrize("streamed", [False, True])
def test_last_group_of_less_than_a_lane(streamed, fmt, scale_bf16, src_bf16):
    """1 to 7 elements over, behind groups of a thousand times their size in the same wave or workgroup: the last scale is that of
    the last elements alone.  Every group below 512 that has several lanes, some above, and those that go past the caches."""
    from paper_2601_22101_amd import binding as eco
    o32 = oracle.get("f32")
    f, of, per = (eco.ECO_FMT_INT4, oracle.FMT_INT4, 2) if fmt else (eco.ECO_FMT_FP8_E4M3, oracle.FMT_E4M3, 1)
    groups = [16, 32, 64, 96, 128, 200, 256] if streamed else [*range(16, 512, 8), 512, 520, 576, 1000, 1152]
    most = int(340e6 / ((2 if src_bf16 else 4) + (0.5 if fmt else 1))) if streamed else 8 * 1152
    big = torch.randn(most + 2000, generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    big = big.to(torch.bfloat16) if src_bf16 else big
    codes = torch.zeros(big.numel() // per, dtype=torch.uint8, device=DEV)
    for group in groups:
        scales = torch.zeros(big.numel() // group + 2, dtype=torch.bfloat16 if scale_bf16 else torch.float32, device=DEV)
        whole = [most // (512 * group) * 512 + k for k in (1, 2, 3, 5)] if streamed else [1, 2, 3, 5, 7]
        for k in whole:
            for rest in range(1, 8):
                n = k * group + rest
                src = big[:n]
                kept = src[-rest:].clone()
                src[-rest:] *= 1e-3
                eco.eco_quantize_init(src, int(src_bf16), n, f, group, int(scale_bf16), codes, scales)
                first = max(0, k - 8)                           # (an even number of elements in)
                rc, rs = o32.quantize_rtn(of, src[first * group:].float().cpu().numpy(), group, scale_bf16=scale_bf16)
                src[-rest:] = kept
                assert np.array_equal(codes[first * group // per:][:rc.size].cpu().numpy(), rc), (group, n)
                assert np.array_equal(scales[first:k + 1].float().cpu().numpy(), rs.astype(np.float32)), (group, n)


@pytest.mark.parametrize("src_bf16", [False, True])
@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("tail", [0, 5, 264])
def test_one_scale_quantizer_past_the_caches(tail, fmt, src_bf16):
    """The same with one scale: every slice ends with the maximum of the whole, wherever that lies, and a NaN beside numbers is no maximum."""
    from paper_2601_22101_amd import binding as eco
    f, step, per = eco.ECO_FMT_INT4 if fmt else eco.ECO_FMT_FP8_E4M3, 8_192_008, 2 if fmt else 1
    n = 290_000_000 // (2 if src_bf16 else 4) // 512 * 512 + tail
    gen = torch.Generator(device=DEV)
    gen.manual_seed(tail)
    x = torch.rand(n, generator=gen, device=DEV) * 0.02 - 0.01
    x[12345] = float("nan")
    for peak in (0, n // 2 + 77, n - 1):
        src = x.clone()
        src[peak] = -0.5
        src = src.to(torch.bfloat16) if src_bf16 else src
        got = _quantized(eco, src, f, n, False, n)
        for at in (0, n // 3 // 32 * 32, (n - step) // 32 * 32):
            part = src[at:at + step].clone()
            part[-1] = -0.5
            want = _quantized(eco, part, f, part.numel(), False, part.numel())
            m = (part.numel() - 1) // 2 * 2
            assert torch.equal(got["s"], want["s"])
            assert torch.equal(got["w"][at // per:(at + m) // per], want["w"][:m // per])
            for key in ("e", "d"):
                assert torch.equal(got[key][at:at + m].view(torch.int32), want[key][:m].view(torch.int32)), key


def test_bandwidth_probe_past_the_caches():
    """In calls that pass the caches by (40 M elements, 440 and 320 MB): every byte as it has to be, the guards around the arrays among them."""
    from paper_2601_22101_amd import binding as eco
    n, guard = 39_063 * 1024, 1024
    gen = torch.Generator(device=DEV)
    gen.manual_seed(9)
    full = {k: torch.randint(-2**31, 2**31, (words + 2 * guard,), generator=gen, device=DEV, dtype=torch.int32)
            for k, words in (("codes", n // 4), ("scales", n // 128), ("grad", n // 2), ("m", n), ("v", n))}
    for k in ("scales", "m"):                                       # finite values: one of m's passes through an addition of zero
        full[k] &= 0x3FFFFFFF
    was = {k: t.clone() for k, t in full.items()}
    x, b = ({k: t[guard:-guard] for k, t in d.items()} for d in (full, was))
    eco.eco_bandwidth_probe(0, x["codes"], x["scales"], x["grad"], x["m"], x["v"], n)
    torch.cuda.synchronize()
    g = b["grad"].view(-1, 4)
    assert torch.equal(x["m"], b["v"]) and torch.equal(x["v"], b["m"])
    assert torch.equal(x["codes"].view(-1, 2), b["codes"].view(-1, 2) ^ torch.stack([g[:, 0] ^ g[:, 2], g[:, 1] ^ g[:, 3]], dim=1))
    for k in full:
        assert torch.equal(full[k][:guard], was[k][:guard]) and torch.equal(full[k][-guard:], was[k][-guard:]), k
        assert k not in ("scales", "grad") or torch.equal(full[k], was[k]), k
    eco.eco_bandwidth_probe(1, None, None, None, x["m"], x["v"], n)
    torch.cuda.synchronize()
    assert torch.equal(x["v"], b["v"]) and torch.equal(x["m"], b["v"])
    assert torch.equal(full["v"][:guard], was["v"][:guard]) and torch.equal(full["v"][-guard:], was["v"][-guard:])
