"""GPU parity of aqsgd_run_jobs against the CPU oracle: several independent messages in
one call (the sending stage's encode + grad_dequant, the receiving stage's decode +
grad_quant, the eight boundaries of the stress configuration, more jobs than one grid
holds, jobs that need the any-shape kernels).  Every job's outputs and every touched
row of its m are compared byte for byte with the oracle's result for that job alone."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2206_01299_amd import binding as B
from paper_2206_01299_amd import workloads as W


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X; run them with -m gpu on the GPU box")
    B.lib()
    import oracle
    oracle.build()
    import gpu_harness
    return gpu_harness


class Boundary:
    """One boundary's buffers on the device and on the host, and the four kinds of job on
    them.  Each kind keeps its own message buffers, so any mix of jobs is independent."""

    def __init__(self, H, rng, dtype, fb, fg, fr, bb, bg, br, batch, n_per, n_rows, seed):
        self.H, self.rng, self.dtype = H, rng, dtype
        self.fb, self.fg, self.fr, self.bb, self.bg, self.br = fb, fg, fr, bb, bg, br
        self.batch, self.n_per, self.n_rows, self.seed = batch, n_per, n_rows, seed
        d = H.dev()
        td = B.DTYPE_NAME[dtype]
        npdt = W.storage_numpy_dtype(dtype)
        self.m_s = torch.zeros((n_rows, n_per), dtype=td, device=d)
        self.m_r = torch.zeros_like(self.m_s)
        self.om_s = np.zeros((n_rows, n_per), dtype=npdt)
        self.om_r = self.om_s.copy()
        self.base = rng.standard_normal((n_rows, n_per)).astype(np.float32) * 3.0
        self.fdesc = B.make_desc(batch=batch, n_per=n_per, n_samples=n_rows, bits=fb, group=fg, dtype=dtype,
                                 rounding=fr, rng_seed=seed)
        self.bdesc = B.make_desc(batch=batch, n_per=n_per, n_samples=n_rows, bits=bb, group=bg, dtype=dtype,
                                 rounding=br, rng_seed=seed + 1)
        self.keep = []           # device tensors of jobs in flight
        self.checks = []         # (name, device tensor, expected numpy)

    def _dev(self, x):
        return W.to_torch(x, self.dtype, self.H.dev())

    def _new(self, n, dt, fill):
        t = torch.full((n,), fill, dtype=dt, device=self.H.dev())
        self.keep.append(t)
        return t

    def encode_job(self, step):
        import oracle
        ids_np = self.rng.choice(self.n_rows, size=self.batch, replace=False).astype(np.int64)
        a_np = W.to_storage(self.base[ids_np] + 0.1 * step * self.rng.standard_normal(
            (self.batch, self.n_per)).astype(np.float32), self.dtype)
        act, ids = self._dev(a_np), torch.from_numpy(ids_np).to(self.H.dev())
        codes = self._new(B.codes_bytes(self.fdesc), torch.uint8, 0x5A)
        scales = self._new(B.scales_count(self.fdesc), torch.float32, -1.0)
        self.keep += [act, ids]
        wc, ws = oracle.encode(a_np, ids_np, self.om_s, dtype=self.dtype, bits=self.fb, group=self.fg,
                               rounding=self.fr, seed=self.seed)
        self.checks += [("encode codes", codes, wc), ("encode scales", scales, ws)]
        self.wire = (codes, scales, ids, wc, ws, ids_np)
        return B.encode_job(self.fdesc, act, ids, self.m_s, codes, scales)

    def decode_job(self):
        """Decodes the message of the last encode_job (which must have run already)."""
        import oracle
        codes, scales, ids, wc, ws, ids_np = self.wire
        out = self._dev(W.to_storage(np.full((self.batch, self.n_per), 9.0, dtype=np.float32), self.dtype))
        self.keep += [out, codes, scales, ids]            # a later encode_job replaces self.wire
        wo = oracle.decode(wc, ws, ids_np, self.om_r, dtype=self.dtype, bits=self.fb, group=self.fg)
        self.checks.append(("decode out", out, wo))
        return B.decode_job(self.fdesc, codes, scales, ids, self.m_r, out)

    def grad_quant_job(self):
        import oracle
        g_np = W.to_storage(1e-3 * self.rng.standard_normal((self.batch, self.n_per)).astype(np.float32),
                            self.dtype)
        grad = self._dev(g_np)
        codes = self._new(B.codes_bytes(self.bdesc), torch.uint8, 0xA5)
        scales = self._new(B.scales_count(self.bdesc), torch.float32, -2.0)
        self.keep.append(grad)
        wc, ws = oracle.grad_quant(g_np.reshape(-1), dtype=self.dtype, bits=self.bb, group=self.bg,
                                   rounding=self.br, seed=self.seed + 1)
        self.checks += [("grad_quant codes", codes, wc), ("grad_quant scales", scales, ws)]
        self.gwire = (codes, scales, wc, ws)
        return B.grad_quant_job(self.bdesc, grad, codes, scales)

    def grad_dequant_job(self):
        """Reconstructs the message of the last grad_quant_job (which must have run already)."""
        import oracle
        codes, scales, wc, ws = self.gwire
        out = self._dev(W.to_storage(np.full((self.batch, self.n_per), 7.0, dtype=np.float32), self.dtype))
        self.keep += [out, codes, scales]                 # a later grad_quant_job replaces self.gwire
        wo = oracle.grad_dequant(wc, ws, dtype=self.dtype, bits=self.bb, group=self.bg)
        self.checks.append(("grad_dequant out", out, wo))
        return B.grad_dequant_job(self.bdesc, codes, scales, out)

    def verify(self, tag):
        H = self.H
        torch.cuda.synchronize()
        for name, got_t, want in self.checks:
            got = (W.from_torch(got_t, self.dtype) if name.endswith("out") else got_t.cpu().numpy()).reshape(-1)
            assert H.same_bytes(got, want.reshape(-1)), f"{tag}: {name}: {H.first_diff(got, want.reshape(-1))}"
        for name, dev_m, want_m in (("sender m", self.m_s, self.om_s), ("receiver m", self.m_r, self.om_r)):
            got = W.from_torch(dev_m, self.dtype)
            assert H.same_bytes(got, want_m), f"{tag}: {name}: {H.first_diff(got, want_m)}"
        self.checks.clear()
        self.keep.clear()


PAIRS = [
    # dtype, fwd bits/group/rounding, bwd bits/group/rounding, batch, n_per
    ("f16", 4, 1600, 0, 8, 1600, 0, 3, 1600 * 37),       # the GPT2 boundary's kernels, ragged rows
    ("f16", 2, 128, 1, 4, 128, 1, 2, 128 * 301),         # stochastic, half-wave teams
    ("bf16", 3, 64, 0, 6, 64, 0, 5, 64 * 517),           # 3- and 6-bit pieces, 8-lane teams
    ("f32", 4, 4096, 0, 8, 4096, 0, 2, 4096 * 9),        # float32 in 16-byte units, whole-workgroup teams
    ("f32", 3, 64, 1, 2, 256, 0, 3, 256 * 33),           # float32 at 3 bits: two units share a byte
    ("f16", 8, 16384, 0, 4, 32768, 1, 2, 32768 * 3),     # 1024-lane teams host the dequantising job
    ("bf16", 6, 512, 1, 3, 2048, 0, 2, 2048 * 11),
]


@pytest.mark.parametrize("case", PAIRS, ids=[f"{c[0]}-fw{c[1]}g{c[2]}-bw{c[4]}g{c[5]}" for c in PAIRS])
def test_stage_side_pairs(H, case):
    """Three steps of a boundary driven the way a pipeline stage would: the sending stage's
    launch holds encode(k) and grad_dequant(k-1), the receiving stage's decode(k) and
    grad_quant(k)."""
    dtype, fb, fg, fr, bb, bg, br, batch, n_per = case
    rng = np.random.default_rng(1000 + PAIRS.index(case))
    b = Boundary(H, rng, dtype, fb, fg, fr, bb, bg, br, batch, n_per, n_rows=2 * batch + 1, seed=900)
    pending_grad = False
    for step in range(3):
        print("jobs", case, "step", step, flush=True)
        sender = [b.encode_job(step)] + ([b.grad_dequant_job()] if pending_grad else [])
        B.run_jobs(sender)
        B.run_jobs([b.decode_job(), b.grad_quant_job()])
        pending_grad = True
        b.verify(f"{case} step {step}")
    B.run_jobs([b.grad_dequant_job()])
    b.verify(f"{case} tail")


def test_eight_boundaries_with_mixed_bits_in_one_call(H):
    """The stress configuration's structure at a small size: eight boundaries, 2/4/8-bit
    mixed, all encodes in one call, then all decodes and gradient jobs in another."""
    rng = np.random.default_rng(5)
    bs = [Boundary(H, rng, "f32", bits, 512, 0, 8, 512, 0, 3, 512 * 21, n_rows=7, seed=40 + i)
          for i, bits in enumerate(W.STRESS_BITS)]
    for step in range(2):
        print("eight boundaries step", step, flush=True)
        B.run_jobs([b.encode_job(step) for b in bs])
        B.run_jobs([b.decode_job() for b in bs] + [b.grad_quant_job() for b in bs])
        B.run_jobs([b.grad_dequant_job() for b in bs])
        for i, b in enumerate(bs):
            b.verify(f"boundary {i} step {step}")


THREE_MIXES = [
    # dtype, group, rounding, forward bits of the boundaries, backward bits, batch, groups per sample
    ("bf16", 64, 0, (3, 4, 3), 6, 5, 517),               # the DeBERTa boundary's widths, 8-lane teams
    ("f16", 1600, 0, (3, 8), 2, 2, 37),                  # one-wave teams of four chunks per lane
    ("f32", 512, 1, (2, 3), 4, 2, 19),                   # float32: units of whole bytes and of a byte and a half side by side
    ("f16", 4096, 1, (6, 3), 8, 2, 5),                   # whole-workgroup teams
]


@pytest.mark.parametrize("case", THREE_MIXES, ids=[f"{c[0]}-g{c[1]}-fw{'_'.join(map(str, c[3]))}-bw{c[4]}"
                                                    for c in THREE_MIXES])
def test_3bit_jobs_share_a_grid_with_other_widths(H, case):
    """A whole time slot in one call (encode of step k, decode and grad_quant of step k-1,
    grad_dequant of step k-2) over boundaries whose quantising jobs have 3 bits and other
    widths at one team shape: they share a launch, the kernel variant with the 3-bit bodies."""
    dtype, group, rnd, fws, bw, batch, gps = case
    rng = np.random.default_rng(2000 + THREE_MIXES.index(case))
    bs = [Boundary(H, rng, dtype, fb, group, rnd, bw, group, rnd, batch, group * gps, n_rows=2 * batch + 1,
                   seed=300 + i) for i, fb in enumerate(fws)]
    for step in range(4):
        print("3-bit mix", case, "slot", step, flush=True)
        jobs = []
        if step >= 2:
            jobs += [b.grad_dequant_job() for b in bs]       # message quantised in the slot before
        if step >= 1:
            jobs += [b.decode_job() for b in bs]             # message encoded in the slot before
            jobs += [b.grad_quant_job() for b in bs]
        jobs += [b.encode_job(step) for b in bs]
        B.run_jobs(jobs)
        for i, b in enumerate(bs):
            b.verify(f"{case} boundary {i} slot {step}")


def test_a_time_slot_over_the_launch_budget_of_small_teams(H):
    """Large small-team launches get about as many workgroups as the chip holds, and every
    workgroup loops over several steps: a slot of four messages whose grids would ask for
    several times that, with a ragged last step."""
    rng = np.random.default_rng(8)
    b = Boundary(H, rng, "f16", 2, 128, 1, 4, 128, 1, 3, 128 * 20011, n_rows=4, seed=77)
    for step in range(3):
        print("over budget, slot", step, flush=True)
        jobs = [b.grad_dequant_job()] if step >= 2 else []
        if step >= 1:
            jobs += [b.decode_job(), b.grad_quant_job()]
        jobs.append(b.encode_job(step))
        B.run_jobs(jobs)
        b.verify(f"over budget slot {step}")


@pytest.mark.parametrize("dtype,bits,group,gps", [
    ("f16", 2, 128, 32 * 1023),       # 4092 steps of a workgroup in the last slot: one step each
    ("f16", 2, 128, 32 * 1024),       # 4096: two each
    ("bf16", 3, 64, 64 * 1024 + 5),   # the same with the 3-bit bodies, ragged
    ("f32", 4, 256, 32 * 1024 + 31),  # float32 in units, 32-lane teams, ragged
])
def test_slots_around_the_size_from_which_small_teams_loop(H, dtype, bits, group, gps):
    rng = np.random.default_rng(gps)
    b = Boundary(H, rng, dtype, bits, group, 0, 8, group, 0, 1, group * gps, n_rows=2, seed=78)
    for step in range(3):
        print("slot", dtype, bits, group, gps, step, flush=True)
        jobs = [b.grad_dequant_job()] if step >= 2 else []
        if step >= 1:
            jobs += [b.decode_job(), b.grad_quant_job()]
        jobs.append(b.encode_job(step))
        B.run_jobs(jobs)
        b.verify(f"slot {step}")


def test_more_jobs_than_one_grid_holds_and_any_shape_jobs(H):
    rng = np.random.default_rng(6)
    same = [Boundary(H, rng, "f16", 4, 256, 0, 8, 256, 1, 2, 256 * 13, n_rows=5, seed=70 + i) for i in range(11)]
    odd = Boundary(H, rng, "f16", 8, 50, 0, 4, 6, 1, 3, 150, n_rows=4, seed=99)         # any-shape kernels
    everyone = same + [odd]
    print("many jobs: encode + grad_quant", flush=True)
    B.run_jobs([b.encode_job(1) for b in everyone] + [b.grad_quant_job() for b in everyone])
    print("many jobs: decode + grad_dequant", flush=True)
    B.run_jobs([b.decode_job() for b in everyone] + [b.grad_dequant_job() for b in everyone])
    for i, b in enumerate(everyone):
        b.verify(f"job set member {i}")


ALONE = [
    # dtype, fwd bits/group/rounding, bwd bits/group/rounding, boundaries, batch, groups per sample
    ("f16", 8, 10, 0, 8, 10, 0, 3, 3, 701),              # odd groups: teams of 2 lanes ...
    ("f32", 4, 12, 0, 8, 12, 0, 1, 3, 257),              # ... 2 and 8 lanes apart: float32 nearest with m keeps 8
    ("bf16", 4, 62, 1, 8, 62, 0, 2, 2, 130),             # rounding modes apart
    ("f16", 2, 124, 1, 4, 124, 1, 2, 2, 67),
    ("f32", 8, 250, 1, 8, 250, 1, 3, 2, 33),
    ("bf16", 4, 510, 0, 6, 500, 0, 5, 2, 9),             # ten quantising jobs: a second table
    ("f16", 4, 1020, 0, 8, 1020, 0, 1, 4, 25),
    ("f32", 4, 1530, 0, 8, 1530, 1, 2, 1, 5),
    ("f16", 4, 2046, 1, 4, 2046, 1, 1, 2, 7),
    ("bf16", 8, 4090, 0, 8, 4090, 0, 2, 2, 3),
    ("f16", 4, 8190, 0, 8, 8190, 0, 2, 1, 3),
    ("bf16", 4, 16382, 1, 8, 16382, 1, 2, 1, 2),
    ("f32", 8, 32766, 1, 8, 32766, 1, 1, 2, 2),
    ("f16", 4, 1020, 0, 8, 1024, 0, 2, 2, 256),          # odd forward, whole backward groups
    ("bf16", 8, 32776, 0, 8, 32776, 0, 2, 2, 2),         # wide groups, 16: spans in two launches
    ("f16", 4, 65536, 0, 6, 65536, 0, 3, 6, 1),          # 36: one workgroup each
    ("f16", 2, 36864, 1, 4, 36864, 1, 2, 4, 3),          # stochastic, 48: spans
    ("bf16", 3, 49152, 1, 8, 49152, 1, 3, 17, 1),        # 102: one workgroup each
    ("f32", 4, 49152, 0, 8, 49152, 0, 1, 3, 2),          # float32 with m, 12: spans
    ("f32", 3, 32776, 0, 8, 32776, 0, 3, 11, 1),         # 66: one workgroup each
    ("f32", 8, 49152, 1, 8, 49152, 1, 3, 17, 1),
    ("f16", 4, 32770, 1, 8, 32770, 1, 1, 2, 2),          # wide and odd
    ("f16", 8, 65544, 0, 8, 32772, 0, 1, 1, 3),          # forward groups beyond a workgroup, wide and odd backward ones
]


@pytest.mark.parametrize("case", ALONE, ids=[f"{c[0]}-fw{c[1]}g{c[2]}r{c[3]}-bw{c[4]}g{c[5]}r{c[6]}x{c[7]}" for c in ALONE])
def test_time_slots_of_odd_and_wide_groups(H, case):
    """Whole time slots of several boundaries whose groups are no whole chunks, or larger than the job
    kernels' shapes: their jobs share launches of their own."""
    dtype, fb, fg, fr, bb, bg, br, boundaries, batch, gps = case
    n_per = fg * gps
    if n_per % bg:
        n_per = fg * bg // np.gcd(fg, bg)
    rng = np.random.default_rng(3000 + ALONE.index(case))
    bs = [Boundary(H, rng, dtype, fb, fg, fr, bb, bg, br, batch, int(n_per), n_rows=2 * batch + 1, seed=500 + i)
          for i in range(boundaries)]
    for step in range(4):
        print("odd and wide", case, "slot", step, flush=True)
        jobs = []
        for b in bs:
            if step >= 2:
                jobs.append(b.grad_dequant_job())
            if step >= 1:
                jobs += [b.decode_job(), b.grad_quant_job()]
            jobs.append(b.encode_job(step))
        B.run_jobs(jobs)
        for i, b in enumerate(bs):
            b.verify(f"{case} boundary {i} slot {step}")


@pytest.mark.parametrize("dtype,bits,rounding,batch,gps,boundaries", [
    ("f16", 4, 0, 2, 3, 1), ("bf16", 8, 1, 16, 4, 1), ("bf16", 3, 1, 13, 5, 1),      # 6, 64 and 65 wide groups
    ("f32", 4, 0, 8, 2, 2), ("f32", 8, 0, 9, 4, 2),                                  # 32 and 72
    ("f16", 2, 0, 24, 3, 2), ("f16", 4, 0, 29, 5, 1)])                               # 144 and 145
def test_time_slots_of_wide_groups_forward_and_rows_backward(H, dtype, bits, rounding, batch, gps, boundaries):
    """One scale per 49152 elements forward, one per row of 768 backward: with few and with many wide groups the
    decodes and grad_dequants ride with the rows, in between with the wide groups."""
    rng = np.random.default_rng(batch * gps)
    bs = [Boundary(H, rng, dtype, bits, 49152, rounding, 8, 768, rounding, batch, 49152 * gps, n_rows=batch + 1, seed=70 + i)
          for i in range(boundaries)]
    for step in range(3):
        jobs = []
        for b in bs:
            late = [b.grad_dequant_job()] if step >= 2 else []
            mid = [b.decode_job(), b.grad_quant_job()] if step >= 1 else []
            jobs += [b.encode_job(step)] + mid + late
        print("wide and rows", dtype, batch * gps * boundaries, "groups, slot", step, flush=True)
        B.run_jobs(jobs)
        for i, b in enumerate(bs):
            b.verify(f"{dtype} boundary {i} slot {step}")


@pytest.mark.parametrize("dtype,bits,group,rounding,batch,n_per,boundaries", [
    ("f32", 4, 4096, 0, 3, 4096 * 60, 4),                # one step a workgroup
    ("f16", 3, 1600, 1, 3, 1600 * 512, 2),
    ("bf16", 2, 64, 1, 3, 64 * 16400, 2),                # teams below a wavefront: one step, ...
    ("f32", 3, 128, 0, 4, 128 * 8200, 2),
    ("f32", 4, 128, 1, 8, 128 * 8200, 1),                # ... and loops
    ("f16", 6, 32, 0, 3, 64 * 16400, 2),                 # groups of half a line: streaming
], ids=str)
def test_time_slots_that_write_more_than_24_mib(H, dtype, bits, group, rounding, batch, n_per, boundaries):
    """Shared launches from the size at which those of whole 128-byte lines write through the L2."""
    eb = 4 if dtype == "f32" else 2
    assert boundaries * batch * n_per * eb * 4 > 24 << 20
    rng = np.random.default_rng(group)
    bs = [Boundary(H, rng, dtype, bits, group, rounding, 8, group, rounding, batch, n_per, n_rows=batch + 1, seed=50 + i)
          for i in range(boundaries)]
    for step in range(3):
        jobs = []
        for b in bs:
            if step >= 2:
                jobs.append(b.grad_dequant_job())
            if step >= 1:
                jobs += [b.decode_job(), b.grad_quant_job()]
            jobs.append(b.encode_job(step))
        B.run_jobs(jobs)
        for i, b in enumerate(bs):
            b.verify(f"{dtype} G{group} boundary {i} slot {step}")


def test_a_bad_job_stops_the_whole_call_before_any_launch(H):
    rng = np.random.default_rng(7)
    b = Boundary(H, rng, "f16", 4, 256, 0, 8, 256, 0, 2, 256 * 5, n_rows=4, seed=1)
    good = b.encode_job(0)
    bad = b.grad_quant_job()
    bad.desc.bits = 5
    arr = (B.Job * 2)(good, bad)
    assert B.lib().aqsgd_run_jobs(arr, 2, None) == -2
    bad.desc.bits = 8
    bad.kind = 9
    arr = (B.Job * 2)(good, bad)
    assert B.lib().aqsgd_run_jobs(arr, 2, None) == -5
    assert B.lib().aqsgd_run_jobs(arr, -1, None) == -5
    assert B.lib().aqsgd_run_jobs(None, 1, None) == -1
    assert B.lib().aqsgd_run_jobs(None, 0, None) == 0
    torch.cuda.synchronize()
    assert not bool(b.m_s.any())                         # the good job did not run either
    codes = b.wire[0]
    assert bool((codes == 0x5A).all())
