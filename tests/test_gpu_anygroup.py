"""GPU parity of groups outside the job kernels' range, byte for byte against the oracle:
odd groups (8 elements or more, no whole number of chunks) at the edges of every team
shape, and groups beyond a workgroup's registers (split over workgroups), both with
previous messages, with first visits and as backward messages."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2206_01299_amd import binding as B
from paper_2206_01299_amd import workloads as W
from test_gpu_seen import _replay as replay_seen


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X; run them with -m gpu on the GPU box")
    B.lib()
    import oracle
    oracle.build()
    import gpu_harness
    return gpu_harness


def _sweep(H, dtype, bits, group, rounding, gps, batch=3):
    cfg = W.BoundaryConfig(
        name=f"any_{dtype}_b{bits}_g{group}_r{rounding}", n_samples=7, batch=batch, seq=gps, hidden=group,
        dtype=dtype, fwd_bits=bits, fwd_group=group, fwd_rounding=rounding, bwd_bits=bits, bwd_group=group,
        bwd_rounding=rounding, law="normal", drift=0.05, epochs=2, shuffle_ids=True, seed=bits * 7 + group)
    H.replay_and_compare(cfg, calls_per_epoch=2, epochs=2, log=lambda *a, **k: None)


# last chunk shares 1 to 7 elements with the one before; team widths 8 .. 1024 and their last lanes
ODD = {8: [9, 15, 57, 63, 65, 121, 127, 250, 257, 505, 519, 1001, 1023, 1531, 2041, 4001, 8185, 16001, 32767],
       4: [10, 62, 66, 254, 510, 514, 1020, 1026, 2046, 4098, 8194, 16390, 32766],
       6: [12, 60, 252, 1020, 1028, 4100, 32764], 2: [12, 68, 500, 1020, 2044, 8196, 32764]}


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bits", [2, 4, 6, 8])
def test_odd_groups(H, dtype, bits):
    for k, group in enumerate(ODD[bits]):
        for rounding in (W.NEAREST, W.STOCHASTIC):
            print(f"odd {dtype} b{bits} G{group} r{rounding}", flush=True)
            _sweep(H, dtype, bits, group, rounding, 1 if group > 8000 else (67, 5, 130)[k % 3])


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bits,group", [(8, 9), (8, 11), (8, 15), (4, 10), (4, 14), (6, 12), (2, 12), (8, 17)])
def test_odd_groups_of_two_chunks(H, dtype, bits, group):
    """Teams of two lanes, 256 groups to a workgroup's step: whole and ragged steps."""
    for rounding in (W.NEAREST, W.STOCHASTIC):
        for gps in (1, 255, 256, 613):
            print(f"two chunks {dtype} b{bits} G{group} r{rounding} x{gps}", flush=True)
            _sweep(H, dtype, bits, group, rounding, gps)


@pytest.mark.parametrize("bits,group,gps", [(8, 1020, 6169), (8, 1020, 6168), (2, 12, 524288), (6, 252, 24967), (4, 1022, 6157)])
def test_large_odd_groups_of_float32(H, bits, group, gps):
    """Gradients of 48 MiB and more in whole 16-byte pieces are written through the L2; one case lies below, and
    the last has pieces that hold two groups."""
    assert (2 * gps * group * 4 >= 48 << 20) == (gps != 6168)
    _sweep(H, "f32", bits, group, W.NEAREST, gps, batch=2)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bits,group", [(4, 32776), (3, 32776), (8, 32769), (2, 32772), (6, 40004), (8, 65537),
                                        (4, 262144), (3, 262152), (8, 300001),
                                        # the last group one workgroup holds, and the first beyond
                                        (6, 49152), (3, 49152), (8, 49153), (3, 49160), (2, 65536), (3, 65536),
                                        (3, 65544)])
def test_groups_beyond_a_workgroup(H, dtype, bits, group):
    for rounding, gps in ((W.NEAREST, 3), (W.STOCHASTIC, 1)):
        print(f"large {dtype} b{bits} G{group} r{rounding}", flush=True)
        _sweep(H, dtype, bits, group, rounding, gps, batch=2)


@pytest.mark.parametrize("dtype,bits,group,gps", [("bf16", 8, 32776, 16), ("bf16", 8, 32776, 17), ("f32", 3, 49152, 16),
                                                  ("f32", 3, 49152, 17), ("f32", 8, 32769, 16), ("f32", 8, 32769, 17),
                                                  ("f16", 8, 32769, 16), ("f16", 8, 32769, 17),
                                                  ("bf16", 8, 49152, 16), ("bf16", 8, 49153, 16), ("bf16", 8, 49153, 17),
                                                  ("f16", 4, 65536, 16), ("f16", 4, 65536, 17)])
def test_wide_groups_few_and_many(H, dtype, bits, group, gps):
    """The number of groups up to which an encode goes out as spans, and one pair more: 64 with
    stochastic rounding in every type; with nearest rounding 32, in float32 and in 16-bit groups of more
    than 49152 elements (the backward message, which has no previous messages, never).  Two samples a call."""
    for rounding, n in ((W.NEAREST, gps), (W.STOCHASTIC, 2 * gps)):
        print(f"wide {dtype} b{bits} G{group} x {n} r{rounding}", flush=True)
        _sweep(H, dtype, bits, group, rounding, n, batch=2)


@pytest.mark.parametrize("dtype,bits,group", [("bf16", 8, 49152), ("f16", 4, 32776), ("f16", 6, 65536), ("f32", 3, 49152),
                                              ("f32", 8, 36868), ("bf16", 4, 57354)])
def test_wide_groups_shared_by_workgroups(H, dtype, bits, group):
    """grad_quant of few wide groups: as many workgroups a group as keep the launch at one a compute unit,
    shares that are and are not whole divisors of the rounds, and counts around where sharing stops."""
    for rounding in (W.NEAREST, W.STOCHASTIC):
        for groups in (1, 2, 32, 33, 64, 65):
            print(f"shared {dtype} b{bits} G{group} r{rounding} x{groups}", flush=True)
            _sweep(H, dtype, bits, group, rounding, groups, batch=1)


def test_large_groups_without_a_change_send_scale_zero(H):
    """Groups whose maximum is zero or below the 2^-120 floor next to one that is not."""
    import oracle
    d = H.dev()
    G, n_per = 32776, 3 * 32776
    act = np.zeros((1, n_per), dtype=np.float32)
    act[0, G:2 * G] = np.float32(2.0 ** -121)
    act[0, 2 * G + 5] = -3.0
    m_np = np.zeros((2, n_per), dtype=np.float32)
    desc = B.make_desc(batch=1, n_per=n_per, n_samples=2, bits=4, group=G, dtype="f32")
    m = torch.zeros((2, n_per), device=d)
    ids_np = np.array([1], dtype=np.int64)
    codes = torch.full((B.codes_bytes(desc),), 0x5A, dtype=torch.uint8, device=d)
    scales = torch.full((3,), -1.0, device=d)
    B.encode(desc, torch.from_numpy(act).to(d), torch.from_numpy(ids_np).to(d), m, codes, scales)
    wc, ws = oracle.encode(act, ids_np, m_np, dtype="f32", bits=4, group=G)
    torch.cuda.synchronize()
    assert H.same_bytes(scales.cpu().numpy(), ws) and ws[0] == 0 and ws[1] == 0 and ws[2] == 3
    assert H.same_bytes(codes.cpu().numpy(), wc)
    assert H.same_bytes(m.cpu().numpy(), m_np)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("rounding", [W.NEAREST, W.STOCHASTIC])
@pytest.mark.parametrize("bits,group,gps", [(4, 1020, 9), (4, 12, 50), (4, 32772, 2), (4, 40000, 1),
                                            # beyond one workgroup in every type: three launches
                                            (4, 65544, 2), (8, 65537, 1), (3, 131080, 1)])
def test_first_visits(H, dtype, bits, rounding, group, gps):
    replay_seen(H, dtype, bits, group, gps * group, 12, 4, 4, rounding, group)


@pytest.mark.parametrize("max_blocks", [3, 7])
@pytest.mark.parametrize("dtype,bits,group,gps", [("f32", 4, 1020, 9), ("bf16", 8, 11, 700), ("f16", 4, 32776, 3),
                                                  ("f32", 8, 40001, 2), ("bf16", 3, 65544, 2), ("f32", 2, 131080, 1)])
def test_first_visits_with_a_capped_grid(H, dtype, bits, group, gps, max_blocks):
    """The loops over groups and spans, and beside them samples that are new and skip these."""
    B.set_launch_shape(max_blocks, 0)
    try:
        for rounding in (W.NEAREST, W.STOCHASTIC):
            print("capped first visits", dtype, bits, group, max_blocks, rounding, flush=True)
            replay_seen(H, dtype, bits, group, gps * group, 12, 4, 4, rounding, group)
    finally:
        B.set_launch_shape(0, 0)


@pytest.mark.parametrize("dtype,bits,group", [("f16", 8, 2**29 + 9), ("f32", 8, 2**29 + 12), ("bf16", 4, 2**30 + 10),
                                              ("f16", 6, 715828012)])
def test_code_offsets_beyond_32_bits(H, dtype, bits, group):
    """One odd group whose code bits pass 2^32: every element is reconstructed from its own code.
    The oracle would take minutes; the wire format's formula in plain torch, one rounding per
    operation, is compared whole.  The 8-bit message is also quantised, by the large groups' way."""
    d, td = H.dev(), B.DTYPE_NAME[dtype]
    desc = B.make_desc(batch=1, n_per=group, n_samples=1, bits=bits, group=group, dtype=dtype)
    print(f"huge {dtype} b{bits} G{group}", flush=True)
    gen = torch.Generator(device=d)
    gen.manual_seed(group)
    codes = torch.randint(0, 256, (B.codes_bytes(desc),), dtype=torch.uint8, device=d, generator=gen)
    s, half = np.float32(3.0), np.float32(((1 << bits) - 1) / 2)
    scales = torch.full((1,), float(s), device=d)
    step = float(s / half)
    m = torch.randn(group, dtype=torch.float32, device=d, generator=gen).to(td).view(1, -1)
    m_old, out = m.clone(), torch.empty((1, group), dtype=td, device=d)
    grad = torch.empty((1, group), dtype=td, device=d)
    B.decode(desc, codes, scales, torch.zeros(1, dtype=torch.int64, device=d), m, out)
    B.grad_dequant(desc, codes, scales, grad)

    def levels(lo, hi):                                      # of elements lo .. hi, lo a multiple of 8
        b = codes[lo * bits // 8:hi * bits // 8].int()
        if bits == 8:
            return b
        if bits == 4:
            return torch.stack((b & 15, b >> 4), 1).view(-1)
        b = b.view(-1, 3)
        w = b[:, 0] | (b[:, 1] << 8) | (b[:, 2] << 16)
        return torch.stack([(w >> (6 * e)) & 63 for e in range(4)], 1).view(-1)

    span = 1 << 26
    for lo in range(0, group, span):
        hi = min(lo + span, group)
        v = (levels(lo, hi).float() - float(half)) * step
        assert torch.equal(grad[0, lo:hi], v.to(td)), f"grad_dequant, elements from {lo}"
        want = (m_old[0, lo:hi].float() + v).to(td)
        assert torch.equal(out[0, lo:hi], want) and torch.equal(m[0, lo:hi], want), f"decode, elements from {lo}"
    if bits == 8:
        x, got = m_old, torch.empty_like(codes)
        B.grad_quant(desc, x, got, scales)
        top = np.float32(x.abs().max().item())
        assert scales.item() == top
        inv = float(half / top)
        for lo in range(0, group, span):
            hi = min(lo + span, group)
            q = torch.floor((x[0, lo:hi].float() * inv + float(half)) + 0.5).to(torch.uint8)
            assert torch.equal(got[lo:hi], q), f"grad_quant, elements from {lo}"


def test_a_message_of_several_kernels_is_timed_as_one_launch(H):
    """aqsgd_profile_next_launch on a group that takes three kernels (clear, maximum, quantise) and on
    one that takes two.  The first reads act and m twice and writes m once, 1 GiB each and far beyond
    the caches: at 8 TB/s the last pass alone takes 0.4 ms, the kernel that clears one word microseconds."""
    d = H.dev()

    def timed(group, batch, rounding):
        desc = B.make_desc(batch=batch, n_per=group, n_samples=batch, bits=8, group=group, dtype="f32", rounding=rounding)
        act = torch.ones((batch, group), device=d)
        m = torch.zeros_like(act)
        codes = torch.empty(B.codes_bytes(desc), dtype=torch.uint8, device=d)
        scales = torch.empty(batch, device=d)
        ids = torch.arange(batch, device=d)
        a, b, c = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        for e in (a, b):
            e.record()
        torch.cuda.synchronize()
        B.encode(desc, act, ids, m, codes, scales)
        B.profile_next_launch(a, b)
        B.encode(desc, act, ids, m, codes, scales)
        c.record()
        B.encode(desc, act, ids, m, codes, scales)           # the request is over: does not stamp again
        torch.cuda.synchronize()
        print("timed", group, batch, a.elapsed_time(b), a.elapsed_time(c), flush=True)
        assert 0 < a.elapsed_time(b) <= a.elapsed_time(c)
        return a.elapsed_time(b)

    assert timed(1 << 28, 1, B.NEAREST) > 0.4
    assert 0.002 < timed(49152, 8, B.STOCHASTIC) < 1
