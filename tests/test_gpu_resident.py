"""Tensor-wise scaling in one pass (tensors that the chip holds) against the oracle, and with every wait given up.  The
comparison bar is the one of tests/gpu_util.py: the same fp32 sequence on both sides, so no bit may differ."""
import pytest
import torch

import oracle
import workloads
from gpu_util import bf16_bits, bytes_per_element, compare, host_copy, oracle_step, step_config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = workloads.TensorSpec
SLAB = 12 * 512
VARIANTS = [("fp8", False, {}), ("int4", True, {}), ("fp8", False, dict(mode=3, weight_decay=0.1)), ("int4", True, dict(mode=3, round=1)),
            ("int4", False, dict(opt=1, round=1, lr=0.05)), ("fp8", True, dict(opt=1, mode=2, lr=0.05)), ("fp8", True, dict(inject=False, round=1))]


def workload(fmt, bf16, which):
    """edges: lengths around one slab, a wave's tile and a lane, lengths with a tail, tensors of one slab after each
    other; long: more slabs than compute units (two turns and a bit, three: the most that are taken), the first length
    that is too long, a small one behind."""
    if which == "edges":
        sizes = [8200, SLAB * 2, SLAB * 2 + 8, SLAB * 2 - 8, SLAB * 3 + 512, SLAB * 3 + 520, SLAB * 2 + 1, SLAB * 2 + 7, 8193, 1001, 5, 20001] + [8448] * 300
    else:
        sizes = [SLAB * 256 * 2 + 4096, 8200, SLAB * 256 * 3 - 8 * 63, SLAB * 256 * 3 + 8, 100000]
        if bf16:
            sizes = sizes[:2] + [SLAB * 768 + 5, SLAB * 768 + 8 + SLAB] + sizes[4:]
    ts = [T(f"t{i}", (n,), fmt, grad_std=1e-3 * (1 + i % 3), granularity="tensor") for i, n in enumerate(sizes)]
    return workloads.Workload(f"resident_{which}", ts, steps=2, state_bf16=bf16, scale_bf16=bf16)


def check(dw, host, k, bf16):
    o32 = oracle.get("f32")
    hp = dw.hparams(k)
    for tv, h in zip(dw.tensors, host):
        h["grad"] = bf16_bits(tv.grad)
    dw.plan.step(hp)
    torch.cuda.synchronize()
    for tv, h in zip(dw.tensors, host):
        oracle_step(o32, h, tv.spec.numel, step_config(hp, tv.tensor_id, tv.fmt, group_size=dw.group_size(tv)))
        st = compare(host_copy(tv), h, f"step {k} {tv.spec.name} ({tv.spec.numel})", bf16)
        assert not any(v for key, v in st.items() if key.endswith("mismatch")), (tv.spec, st)


@pytest.mark.parametrize("fmt,bf16,over", VARIANTS)
def test_one_pass_matches_the_oracle_at_the_edges(fmt, bf16, over):
    from paper_2601_22101_amd import harness
    dw = harness.DeviceWorkload(workload(fmt, bf16, "edges"), DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    for k in (1, 2):
        dw.fill_gradients(k)
        check(dw, host, k, bf16)
    dw.close()


@pytest.mark.parametrize("fmt,bf16,over", VARIANTS[:2])
def test_one_pass_matches_the_oracle_on_long_tensors(fmt, bf16, over):
    from paper_2601_22101_amd import harness
    dw = harness.DeviceWorkload(workload(fmt, bf16, "long"), DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    dw.fill_gradients(1)
    check(dw, host, 1, bf16)
    dw.close()


@pytest.mark.parametrize("fmt,bf16,over", VARIANTS)
def test_tiles_whose_wait_is_given_up_are_finished_from_memory(fmt, bf16, over):
    """With two workgroups (a small limit on the threads of a launch) no tensor of more than a few slabs can be held: the
    waits run out and the finishing kernel does the rest.  Same bytes; and the next step starts clean."""
    from paper_2601_22101_amd import binding as eco
    from paper_2601_22101_amd import harness
    ts = [T(f"t{i}", (n,), fmt, grad_std=1e-3, granularity="tensor") for i, n in enumerate((SLAB * 30 + 13, 8200, SLAB * 11 + 512 + 8, 60000, SLAB * 25))]
    wl = workloads.Workload("given_up", ts, steps=4, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(wl, DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors]
    try:
        for k, limit in ((1, 2048), (2, -1), (3, 2048), (4, 1024)):
            eco.eco_set_option(3, limit)
            dw.fill_gradients(k)
            check(dw, host, k, bf16)
    finally:
        eco.eco_set_option(3, -1)
    dw.close()


def beside_enough(wl, bf16, over):
    """The workload with tensors behind it that make one pass the faster form of its list (small lists, and those beside a
    longer tensor, are stepped in two): as many of 4.7 M elements as have 420 MB of arrays, 1.1 GB with master weights, whose
    second pass is a short one."""
    fmt = wl.tensors[0].fmt
    n = int((1100e6 if over.get("mode", 1) == 3 else 420e6) / (4_700_000 * bytes_per_element(fmt, bf16, over))) + 1
    wl.tensors = wl.tensors + [T(f"fill{i}", (4_700_000,), fmt, granularity="tensor") for i in range(n)]
    return wl


@pytest.mark.parametrize("which", ["edges", "long"])
@pytest.mark.parametrize("fmt,bf16,over", VARIANTS)
def test_one_pass_matches_the_oracle_in_a_list_that_it_pays_for(fmt, bf16, over, which):
    from paper_2601_22101_amd import harness
    wl = workload(fmt, bf16, which)
    n = len(wl.tensors)
    dw = harness.DeviceWorkload(beside_enough(wl, bf16, over), DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors[:n]]
    for k in (1, 2) if which == "edges" else (1,):
        dw.fill_gradients(k)
        check(dw, host, k, bf16)
    dw.close()


@pytest.mark.parametrize("fmt,bf16,over", VARIANTS)
def test_slabs_whose_wait_is_given_up_in_a_list_that_one_pass_pays_for(fmt, bf16, over):
    from paper_2601_22101_amd import binding as eco
    from paper_2601_22101_amd import harness
    ts = [T(f"t{i}", (n,), fmt, grad_std=1e-3, granularity="tensor") for i, n in enumerate((SLAB * 30 + 13, 8200, SLAB * 11 + 512 + 8, 60000, SLAB * 25))]
    wl = workloads.Workload("given_up_long", ts, steps=4, state_bf16=bf16, scale_bf16=bf16)
    dw = harness.DeviceWorkload(beside_enough(wl, bf16, over), DEV, layout=over)
    host = [host_copy(tv) for tv in dw.tensors[:len(ts)]]
    try:
        for k, limit in ((1, 2048), (2, -1), (3, 100_000), (4, 1024)):
            eco.eco_set_option(3, limit)
            dw.fill_gradients(k)
            check(dw, host, k, bf16)
    finally:
        eco.eco_set_option(3, -1)
    dw.close()


def test_two_plans_on_two_streams_share_the_chip():
    """Neither kernel has all its workgroups resident; each plan has scratch of its own."""
    from paper_2601_22101_amd import harness
    made = []
    for which in range(2):
        ts = [T(f"t{i}", (900_000 + 8 * i + which,), "fp8", grad_std=1e-3, granularity="tensor") for i in range(12)]
        made.append(workloads.Workload(f"stream{which}", ts, steps=3))
    ref = [harness.DeviceWorkload(wl, DEV) for wl in made]
    dut = [harness.DeviceWorkload(wl, DEV) for wl in made]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in (1, 2, 3):
        for dw in ref + dut:
            dw.fill_gradients(k)
        for dw in ref:
            dw.step(k)
            torch.cuda.synchronize()
        for dw, st in zip(dut, streams):
            dw.plan.step(dw.hparams(k), st)
        torch.cuda.synchronize()
        for a, b in zip(ref, dut):
            for ta, tb in zip(a.tensors, b.tensors):
                assert all(torch.equal(x, y) for x, y in ((ta.weights, tb.weights), (ta.scales, tb.scales), (ta.m, tb.m), (ta.v, tb.v)))
    for dw in ref + dut:
        dw.close()
