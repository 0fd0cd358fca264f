"""GPU parity of the mixture-of-experts combine (weighted sum of two rows gathered through routing
tables) against the oracle: one rounding of an fp32 result to bf16/f16."""
import numpy as np
import pytest

import workloads
from oracle import consumers, dm_ops
from oracle.run import run_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    import paper_2604_09558_amd as vt
    from paper_2604_09558_amd import pipelines, torch_io
    vt.lib()
    return vt, torch_io, pipelines, torch


def check(got, ref, rel):
    err = np.abs(got - ref)
    assert (err <= rel * np.abs(ref) + 1e-6).all(), err.max()


@pytest.mark.parametrize("T,E,N,dtype", [(300, 4, 264, "bf16"), (64, 8, 8, "f16"), (1000, 8, 1000, "bf16"), (50, 3, 20, "f16")])
def test_moe_combine_small(gpu, T, E, N, dtype):
    vt, tio, pipelines, torch = gpu
    wl = workloads.moe_combine(seed=1, T=T, E=E, N=N, dtype=dtype)     # N = 20: rows are not 16-byte multiples -> generic path
    ref = run_workload(wl)["out"]
    for materialized in (False, True):
        p = pipelines.WeightedSum(tio.DeviceWorkload(wl), materialized)
        p.run()
        torch.cuda.synchronize()
        # fp32 product-sum (3 roundings of 2^-24) then one rounding to the storage type
        check(tio.to_host_f64(p.out), ref, 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11)


def test_moe_combine_virtual_equals_materialized_bitwise_and_mid_size(gpu):
    vt, tio, pipelines, torch = gpu
    wl = workloads.moe_combine(seed=2, T=4096, E=8, N=2048)
    a = pipelines.WeightedSum(tio.DeviceWorkload(wl))
    b = pipelines.WeightedSum(tio.DeviceWorkload(wl), materialized=True)
    a.run()
    b.run()
    torch.cuda.synchronize()
    assert torch.equal(a.out, b.out)
    check(tio.to_host_f64(a.out), run_workload(wl)["out"], 2.0 ** -8)


def test_moe_combine_full_size_every_output(gpu):
    """The combine at the benchmarked size (16384 tokens x 14336 columns), every output; the oracle
    gathers both operands as dense copies and mixes them in float64, in row blocks to bound memory."""
    vt, tio, pipelines, torch = gpu
    wl = workloads.moe_combine()
    p = pipelines.WeightedSum(tio.DeviceWorkload(wl))
    p.run()
    torch.cuda.synchronize()
    env = dm_ops.run_chain(wl.chain, wl.sources, wl.index_tables, keep={"x", "y"})
    w = wl.consumer["weights"]
    assert env["x"].shape == (16384, 14336)
    for r in range(0, 16384, 2048):
        ref = consumers.weighted_sum(consumers.decode(env["x"][r:r + 2048], "bf16"),
                                     consumers.decode(env["y"][r:r + 2048], "bf16"), w[r:r + 2048])
        check(tio.to_host_f64(p.out[r:r + 2048]), ref, 2.0 ** -8)


# One row in several workgroups (the last of them short), several rows in one, vectors per thread from one to eight and
# their remainders; `pieces`: x is two sources behind each other, which only the evaluator takes
@pytest.mark.parametrize("pieces", [False, True])
@pytest.mark.parametrize("R,C,dtype", [(1, 8, "bf16"), (1, 14336, "f16"), (3, 2056, "bf16"), (700, 8, "f16"), (517, 1000, "bf16"), (2100, 2080, "bf16"),
                                        (5200, 1032, "f16"), (40000, 16, "bf16"), (9, 40960, "bf16")])
def test_row_kernel_shapes(gpu, R, C, dtype, pieces):
    """Against the sum in float64: two products and a sum in fp32 (or fma: 3 roundings of 2^-24) and one to the type."""
    vt, tio, pipelines, torch = gpu
    g = torch.Generator(device="cuda:0")
    g.manual_seed(R + C)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    pool = torch.randn((R + 5, C), generator=g, device="cuda:0").to(dt)
    more = torch.randn((R + 2, C), generator=g, device="cuda:0").to(dt)
    w = torch.rand((R, 2), generator=g, device="cuda:0")
    idx = np.random.default_rng(R).integers(0, R + 5, R).astype(np.int32)
    tab = torch.from_numpy(idx).to("cuda:0")
    src = {"P": (tuple(pool.shape), dtype, pool.data_ptr()), "M": (tuple(more.shape), dtype, more.data_ptr())}
    gather = vt.build_chain([("y", "index_select", ("P",), {"dim": 0, "index": "i"})], src, "y", {"i": idx}, {"i": tab.data_ptr()})
    y = pool[tab.long()]
    if pieces:
        cut = R // 2
        chain = [("c", "concat", ("M", "P"), {"dim": 0}), ("x", "slice", ("c",), {"dim": 0, "start": R + 2 - cut, "stop": 2 * R + 2 - cut})]
        xd = vt.build_chain(chain, src, "x", {}, {})
        x = torch.cat((more, pool))[R + 2 - cut:2 * R + 2 - cut]
    else:
        xd = vt.build_chain([("x", "slice", ("M",), {"dim": 0, "start": 2, "stop": R + 2})], src, "x", {}, {})
        x = more[2:]
    out = torch.full((R + 1, C), 7.0, dtype=dt, device="cuda:0")
    vt.vt_weighted_sum(xd, gather, w, out)
    torch.cuda.synchronize()
    px, py = w[:, :1].double() * x.double(), w[:, 1:].double() * y.double()
    ref = px + py
    bound = ref.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -11) + 2.0 ** -22 * (px.abs() + py.abs()) + 2.0 ** -25
    assert bool(((out[:R].double() - ref).abs() <= bound).all())
    assert bool((out[R] == 7.0).all())


@pytest.mark.parametrize("R,C,dtype", [(700, 264, "bf16"), (700, 264, "f16"), (5, 8192, "bf16")])
def test_every_path_gives_the_same_bits(gpu, kernels, R, C, dtype):
    """The same rows alone and among others, as one tensor and as two behind each other, and with an output that is not
    aligned for whole vectors: the row kernel (both of its maps, every place in a workgroup) and the generic one round alike."""
    vt, tio, pipelines, torch = gpu
    g = torch.Generator(device="cuda:0")
    g.manual_seed(R)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    x = torch.randn((R, C), generator=g, device="cuda:0").to(dt)
    y = (-x.float() + 0.01 * torch.randn((R, C), generator=g, device="cuda:0")).to(dt)          # sums that cancel: roundings show
    w = 0.5 + 0.001 * torch.rand((R, 2), generator=g, device="cuda:0")
    cut = R // 3
    parts = {"X0": ((cut, C), dtype, x[:cut].data_ptr()), "X1": ((R - cut, C), dtype, x[cut:].data_ptr())}
    whole = {"X": ((R, C), dtype, x.data_ptr())}
    xd, yd = vt.build_chain([], whole, "X"), vt.build_chain([], {"Y": ((R, C), dtype, y.data_ptr())}, "Y")
    xc = vt.build_chain([("c", "concat", ("X0", "X1"), {"dim": 0})], parts, "c")
    out, out_c = (torch.zeros((R, C), dtype=dt, device="cuda:0") for _ in range(2))
    store = torch.zeros(R * C + 1, dtype=dt, device="cuda:0")
    names = [kernels(lambda d=d, o=o: vt.vt_weighted_sum(d, yd, w, o)) for d, o in ((xd, out), (xc, out_c), (xd, store[1:]))]
    for n, kernel in zip(names, ("k_weighted_sum_rows", "k_weighted_sum_rows", "k_weighted_sum_generic")):
        assert any(kernel in k for k in n), n
    assert torch.equal(out, out_c) and torch.equal(out, store[1:].view(R, C))
    for r in (0, R // 2, R - 1):
        one = torch.zeros((1, C), dtype=dt, device="cuda:0")
        vt.vt_weighted_sum(vt.build_chain([], {"X": ((1, C), dtype, x[r].data_ptr())}, "X"), vt.build_chain([], {"Y": ((1, C), dtype, y[r].data_ptr())}, "Y"),
                           w[r:r + 1].contiguous(), one)
        torch.cuda.synchronize()
        assert torch.equal(one[0], out[r]), r
