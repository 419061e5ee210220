"""The launch-shape settings (workgroups per launch, unroll of the dequantising kernel)
change how the work is cut and never a result bit: a few boundaries are replayed against
the oracle with grids so small that every kernel's grid-stride loops turn over many times."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2206_01299_amd import binding as B
from paper_2206_01299_amd import workloads as W

CASES = [("f16", 4, 1600, W.NEAREST, 41), ("f16", 2, 128, W.STOCHASTIC, 301), ("bf16", 3, 64, W.NEAREST, 517),
         ("bf16", 6, 64, W.NEAREST, 130), ("f32", 4, 4096, W.NEAREST, 9), ("f32", 8, 256, W.STOCHASTIC, 77),
         ("f32", 3, 64, W.NEAREST, 99), ("f16", 8, 8200, W.NEAREST, 5), ("f16", 8, 50, W.NEAREST, 333),
         # odd groups: the looping kernels of every width, of one and several waves to a team
         ("f32", 6, 52, W.STOCHASTIC, 333), ("bf16", 8, 11, W.STOCHASTIC, 700), ("bf16", 4, 1020, W.NEAREST, 77),
         ("f16", 2, 12, W.NEAREST, 601), ("f32", 2, 4100, W.NEAREST, 9), ("f16", 4, 16390, W.STOCHASTIC, 5),
         # wide groups, which a capped grid hands to the large groups' kernels, and large ones: their
         # loops over spans
         ("bf16", 4, 32776, W.NEAREST, 3), ("f32", 8, 32772, W.STOCHASTIC, 3), ("f16", 8, 40001, W.STOCHASTIC, 2),
         ("f32", 3, 65544, W.NEAREST, 3), ("bf16", 8, 65545, W.STOCHASTIC, 2), ("f16", 6, 262148, W.NEAREST, 1)]


def _cfg(dtype, bits, group, rounding, gps, batch=3, n_samples=7):
    return W.BoundaryConfig(name=f"shape_{dtype}_b{bits}_g{group}", n_samples=n_samples, batch=batch, seq=gps,
                            hidden=group, dtype=dtype, fwd_bits=bits, fwd_group=group, fwd_rounding=rounding,
                            bwd_bits=bits, bwd_group=group, bwd_rounding=rounding, law="normal", drift=0.05,
                            epochs=2, shuffle_ids=True, seed=4242 + bits + group)


@pytest.mark.parametrize("max_blocks,unroll", [(3, 1), (7, 4), (64, 2)])
def test_results_do_not_depend_on_the_launch_shape(max_blocks, unroll):
    if not torch.cuda.is_available():
        pytest.fail("needs the MI355X")
    B.lib()
    import oracle
    oracle.build()
    import gpu_harness as H
    B.set_launch_shape(max_blocks, unroll)
    try:
        for case in CASES:
            print("launch shape", max_blocks, unroll, "case", case, flush=True)
            H.replay_and_compare(_cfg(*case), calls_per_epoch=2, epochs=2, log=lambda *a, **k: None)
        # the extension kernels go through the same bound
        import test_gpu_lowbit
        import test_gpu_topk
        test_gpu_lowbit._replay(H, _cfg("f16", 4, 1600, W.NEAREST, 41), 8, calls_per_epoch=2, epochs=2)
        test_gpu_lowbit._replay(H, _cfg("f32", 2, 64, W.STOCHASTIC, 203), 2, calls_per_epoch=2, epochs=2)
        test_gpu_topk._run(H, "f16", 1600, 320, n_groups=67, kind="heavy")
        test_gpu_topk._run(H, "f32", 64, 13, n_groups=1031, kind="ties")
    finally:
        B.set_launch_shape(0, 0)


def test_launch_shape_rejects_bad_values():
    if not torch.cuda.is_available():
        pytest.fail("needs the MI355X")
    L = B.lib()
    assert L.aqsgd_set_launch_shape(-1, 0) == -5
    assert L.aqsgd_set_launch_shape(0, 3) == -5
    assert L.aqsgd_set_launch_shape(0, 0) == 0


@pytest.mark.parametrize("bits,group", [(4, 8), (8, 9)])
def test_more_samples_than_the_grid_has_rows(bits, group):
    """A call of its own gets one grid row per sample; beyond 65535 of them its kernels loop."""
    if not torch.cuda.is_available():
        pytest.fail("needs the MI355X")
    B.lib()
    import oracle
    oracle.build()
    import gpu_harness as H
    H.replay_and_compare(_cfg("f16", bits, group, W.NEAREST, 1, batch=65538, n_samples=65540),
                         calls_per_epoch=1, epochs=2, log=lambda *a, **k: None)


@pytest.mark.parametrize("dtype,bits", [("f32", 4), ("f32", 3), ("f16", 8), ("bf16", 3)])
def test_many_samples_of_about_one_chunk_per_lane(dtype, bits):
    """Reconstruction takes one chunk a lane from 1024 samples of at most 256 chunks on: both
    sides of both limits, and rows far below them."""
    if not torch.cuda.is_available():
        pytest.fail("needs the MI355X")
    B.lib()
    import oracle
    oracle.build()
    import gpu_harness as H
    for n_per, batch in ((2048, 1024), (2056, 1024), (2048, 1023), (8, 1025), (520, 1500)):
        print("short samples", dtype, bits, n_per, batch, flush=True)
        H.replay_and_compare(_cfg(dtype, bits, n_per, W.NEAREST, 1, batch=batch, n_samples=batch + 3),
                             calls_per_epoch=1, epochs=2, log=lambda *a, **k: None)


def test_more_samples_of_a_wide_group_than_the_grid_has_rows():
    """Beyond 65535 samples a wide group's message falls to the large groups' kernels, which loop over
    samples (skipping the new ones).  The oracle would take minutes: the call is compared with the same
    samples in two calls, which go out as one workgroup a group."""
    if not torch.cuda.is_available():
        pytest.fail("needs the MI355X")
    batch, group = 65538, 32776
    d = torch.device("cuda:0")
    gen = torch.Generator(device=d)
    gen.manual_seed(7)
    act = torch.randn((batch, group), device=d, dtype=torch.float16, generator=gen)
    ids = torch.randperm(batch, device=d, generator=gen)
    print("many wide samples", flush=True)

    def encode(parts):
        m = torch.zeros((batch, group), dtype=torch.float16, device=d)
        seen = (torch.arange(batch, device=d) % 3 != 0).int()
        out = []
        for lo, hi in parts:
            desc = B.make_desc(batch=hi - lo, n_per=group, n_samples=batch, bits=8, group=group, dtype="f16")
            codes = torch.full((B.codes_bytes(desc),), 0x5A, dtype=torch.uint8, device=d)
            scales = torch.full((hi - lo,), -1.0, device=d)
            first = torch.full((hi - lo,), -7, dtype=torch.int32, device=d)
            B.encode_seen(desc, act[lo:hi], ids[lo:hi], m, seen, 9, first, codes, scales)
            out.append((codes, scales, first))
        return [torch.cat(x) for x in zip(*out)] + [m, seen]

    one, two = encode([(0, batch)]), encode([(0, 30000), (30000, batch)])
    for name, a, b in zip(("codes", "scales", "first", "m", "seen"), one, two):
        assert torch.equal(a, b), name
    assert one[2].sum().item() == (batch + 2) // 3 and (one[1] > 0).sum().item() == batch - (batch + 2) // 3
