"""The dispatch as a program sees it from the host: which launches a call makes, with the device runtime's
launch call replaced in a client program (tests/dispatch_client.cpp).  No GPU, and no pointer is followed."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
F32, F16, BF16 = 0, 1, 2
ENCODE, DECODE, GRAD_QUANT, GRAD_DEQUANT = 0, 1, 2, 3


@pytest.fixture(scope="module")
def client(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "g++ is part of the image"
    exe = tmp_path_factory.mktemp("dispatch") / "client"
    lib = ROOT / "paper_2206_01299_amd" / "libaqsgd.so"
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT / 'include'}",
                    str(ROOT / "tests" / "dispatch_client.cpp"), str(lib), f"-Wl,-rpath,{lib.parent}",
                    "-Wl,-rpath,/opt/rocm/lib", "-ldl", "-o", str(exe)], check=True)

    def run(*jobs, options=()):
        """The launches, as (grid, workgroup size, kernel), and the call's status."""
        words = [",".join(str(x) for x in j) for j in jobs]
        out = subprocess.run([str(exe), *options, *words], check=True, capture_output=True, text=True).stdout.splitlines()
        launches = []
        for line in out[:-1]:
            _, gx, gy, gz, _, block, kernel = line.split(maxsplit=6)
            launches.append(((int(gx), int(gy), int(gz)), int(block), kernel))
        return launches, int(out[-1].split()[1])

    return run


def test_nothing_is_allocated_once_something_is_enqueued(client):
    """Want of host memory is reported before anything is enqueued, so a call that has made its first launch
    allocates no more: job lists whose odd and wide groups go out one by one, in pairs, and with whole ones."""
    lists = [
        [(ENCODE, F16, 4, 0, 4, 1020, 1020), (ENCODE, F16, 8, 0, 4, 99990, 9)],               # two team shapes
        [(ENCODE, F16, 4, 0, 4, 1020, 1020), (GRAD_QUANT, F16, 4, 0, 4, 1020, 1020),
         (ENCODE, BF16, 4, 1, 4, 1020, 1020), (GRAD_DEQUANT, F16, 4, 0, 4, 1020, 1020)],
        [(ENCODE, F16, 4, 0, 4, 49152, 49152), (ENCODE, F32, 4, 0, 4, 49152, 49152),
         (DECODE, F32, 4, 0, 4, 49152, 49152)],
        [(ENCODE, F16, 4, 0, 4, 1024, 1024), (ENCODE, F16, 4, 0, 4, 1020, 1020), (DECODE, F16, 4, 0, 4, 1020, 1020)],
    ]
    for jobs in lists:
        plain, status = client(*jobs)
        assert status == 0 and len(plain) >= 2
        starved, status = client(*jobs, options=("starve",))
        assert status == 0, f"{len(starved)} of {len(plain)} launches were made, then {status}"
        assert starved == plain


@pytest.mark.parametrize("lead", [(GRAD_QUANT, F16, 8, 1, 200, 49152, 49152), (GRAD_QUANT, F16, 8, 0, 4, 16384, 16384),
                                  (ENCODE, F16, 8, 0, 4, 16380, 16380)], ids=["wide", "whole", "odd"])
def test_shared_launches_stay_below_the_lanes_of_a_grid(client, lead):
    """A launch takes fewer than 2^32 lanes along a dimension.  Reconstructions of 34 GB each that ride along
    with workgroups of 1024 lanes pass that together (five of them fit the card); every unit of work still
    has a workgroup, or a kernel that loops."""
    n_per = 262144 if lead[6] % 8 == 0 else 261900
    ride = (GRAD_DEQUANT, F16, 2, 0, 65535, n_per, 64 if lead[6] % 8 == 0 else 4 * 291)
    launches, status = client(lead, *[ride] * 5)
    assert status == 0
    for grid, block, kernel in launches:
        assert grid[0] * block < 1 << 32, (grid, block, kernel)
    one, status = client(lead, ride)                     # as before where it fits
    assert status == 0 and len(one) == 1 and "jobs_kernel" in one[0][2]


def _slot(dtype, batch, n_per, group, boundaries=1):
    return [(kind, dtype, bits, 0, batch, n_per, group) for _ in range(boundaries)
            for kind, bits in ((ENCODE, 4), (DECODE, 4), (GRAD_QUANT, 8), (GRAD_DEQUANT, 8))]


@pytest.mark.parametrize("dtype,batch,n_per,group,boundaries,through", [
    (F16, 4, 1024 * 1600, 1600, 1, True),        # 62 MB written, whole 128-byte lines
    (F32, 8, 128 * 4096, 4096, 4, True),
    (F32, 16, 512 * 2048, 128, 1, True),
    (F32, 11, 130 * 3392, 64, 1, True),
    (F16, 8, 512 * 2048, 64, 1, True),           # teams below a wavefront that loop
    (F16, 4, 250 * 1024, 1024, 1, False),        # 10 MB
    (BF16, 18, 175 * 128, 128, 4, False),
    (F16, 8, 1001 * 1000, 1000, 1, False),       # rows of 2000 bytes
    (F32, 4, 2048 * 2704, 2704, 4, False),
    (F16, 8, 512 * 2048, 32, 1, False),          # groups of half a line
])
def test_large_shared_launches_of_whole_lines_write_through(client, dtype, batch, n_per, group, boundaries, through):
    """The store policy is a constant of the kernel (its last template argument), chosen by what the launch writes."""
    launches, status = client(*_slot(dtype, batch, n_per, group, boundaries))
    assert status == 0 and all("codec_jobs_kernel<" in k for _, _, k in launches), launches
    for _, _, kernel in launches:
        assert kernel.split(">(")[0].endswith(", true" if through else ", false"), kernel
    alone, status = client((DECODE, dtype, 4, 0, batch, n_per, group), (GRAD_DEQUANT, dtype, 8, 0, batch, n_per, group))
    assert status == 0 and len(alone) == 1 and "dequant_jobs_kernel<" in alone[0][2]


def test_launches_that_loop_have_a_kernel_for_every_store_policy(client):
    """More samples than a grid has rows: kernels that loop, of teams below and above a wavefront."""
    for group in (64, 128, 256, 512, 1024, 1536, 2048, 4096, 8192, 16384, 32768):
        for dtype in (F32, F16, BF16):
            for bits in (3, 4):
                n_per = group * max(1, 4096 // group)
                launches, status = client((ENCODE, dtype, bits, 0, 70001, n_per, group),
                                          (DECODE, dtype, bits, 1, 70001, n_per, group))
                assert status == 0 and len(launches) == 1, (group, dtype, launches, status)


@pytest.mark.parametrize("dtype,bits,group,rows,through", [
    (F32, 4, 4096, 1366, True), (F32, 4, 4096, 1365, False),         # 24 MiB of m and codes
    (F16, 4, 1600, 5243, True), (F16, 4, 1600, 5242, False),         # 20 MiB
    (BF16, 3, 64, 137971, True), (BF16, 3, 64, 137970, False),
    (F16, 4, 1000, 20000, False), (F16, 4, 32, 600000, False),       # rows, groups that are no whole lines
    (F16, 4, 1020, 20000, False),                                    # groups that are no octets
])
def test_large_encodes_alone_write_through(client, dtype, bits, group, rows, through):
    kinds = {0: "streaming", 1: "3 bits, streaming", 2: "odd, streaming", 4: "through", 5: "3 bits, through"}
    launches, status = client((ENCODE, dtype, bits, 0, 1, rows * group, group), options=("alone",))
    assert status == 0 and len(launches) == 1
    kernel = launches[0][2].split("quant_single_kernel<")[1].split(">(")[0]
    assert kinds[int(kernel.split(",")[-1])].endswith("through" if through else "streaming"), kernel
    grads, status = client((GRAD_QUANT, dtype, bits, 0, 1, rows * group, group), options=("alone",))
    assert status == 0 and int(grads[0][2].split("quant_single_kernel<")[1].split(">(")[0].split(",")[-1]) in (0, 1, 2)


@pytest.mark.parametrize("dtype,bits,group,rows,through", [
    (F16, 4, 256, 8192, True), (F16, 4, 256, 8191, False),           # 4 MiB written
    (BF16, 3, 1024, 2048, True), (BF16, 3, 1024, 2047, False),
    (BF16, 2, 1600, 1600, True),                                     # one element a lane in the last round
    (F16, 8, 16384, 512, True), (BF16, 4, 64, 524288, True),
    (BF16, 4, 2008, 7007, False), (F16, 4, 32, 600000, False),       # rows, groups that are no whole lines
    (F32, 4, 1024, 8192, False),                                     # ordinary stores
])
def test_low_precision_receivers_of_whole_lines_write_through(client, dtype, bits, group, rows, through):
    launches, status = client((DECODE, dtype, bits, 0, 1, rows * group, group), options=("lowbit",))
    assert status == 0 and len(launches) == 1
    mode = launches[0][2].split("lowbit_team_kernel<")[1].split(">(")[0].split(",")[5]
    assert int(mode) == (3 if through else 0), launches


@pytest.mark.parametrize("kind,dtype,bits,group,rows,through", [
    (GRAD_DEQUANT, F32, 8, 1020, 12337, True), (GRAD_DEQUANT, F32, 8, 1020, 12336, False),       # 48 MiB
    (GRAD_DEQUANT, F32, 2, 12, 2000000, True),
    (GRAD_DEQUANT, F32, 4, 1022, 20000, False),          # pieces that hold two groups
    (GRAD_DEQUANT, F16, 4, 1020, 40000, False),
    (DECODE, F32, 4, 1020, 20000, False),                # previous messages
])
def test_large_odd_float32_gradients_write_through(client, kind, dtype, bits, group, rows, through):
    launches, status = client((kind, dtype, bits, 0, 1, rows * group, group), options=("alone",))
    assert status == 0 and len(launches) == 1
    odd_kind = launches[0][2].split("dequant_odd_kernel<")[1].split(">(")[0].split(",")[-1]
    assert int(odd_kind) == (2 if through else 0), launches


@pytest.mark.parametrize("dtype,rounding,groups,with_wide", [
    (F16, 0, 8, True), (BF16, 0, 64, True), (F16, 1, 8, False), (BF16, 1, 64, False), (F16, 1, 65, True),
    (F32, 0, 32, False), (F32, 1, 64, False), (F32, 0, 65, True),
    (F16, 0, 144, True), (F16, 0, 145, False), (BF16, 1, 512, False), (F32, 0, 144, True), (F32, 0, 145, False)])
def test_reconstructions_ride_with_wide_groups_while_those_leave_the_chip_idle(client, dtype, rounding, groups, with_wide):
    """Wide forward groups, a scale for every row backward: the table that takes the decode and the grad_dequant."""
    n_per = 49152
    fwd, bwd = (dtype, 4, rounding, groups, n_per, n_per), (dtype, 8, rounding, groups, n_per, 768)
    launches, status = client((ENCODE, *fwd), (DECODE, *fwd), (GRAD_QUANT, *bwd), (GRAD_DEQUANT, *bwd))
    assert status == 0
    alone, status = client((GRAD_QUANT, *bwd), (ENCODE, *fwd))
    assert status == 0
    name = lambda kernels: {k.split("<")[0].split()[-1]: g[0] for g, _, k in kernels}
    got, bare = name(launches), name(alone)
    rows = next(k for k in got if k.endswith("codec_jobs_kernel"))
    assert (got[rows] == bare[rows]) == with_wide, (launches, alone)
    # without a table of whole groups to come they always ride along
    stage, status = client((ENCODE, *fwd), (GRAD_DEQUANT, *bwd))
    assert status == 0 and all("jobs_kernel" in k for _, _, k in stage), stage


@pytest.mark.parametrize("dtype,elements,through", [
    (F32, 11 << 18, True), (F32, (11 << 18) - 32, False), (F32, (19 << 18) - 32, True), (F32, 19 << 18, False),
    (F16, 11 << 19, True), (F16, (11 << 19) - 64, False), (BF16, (17 << 19) - 64, True), (BF16, 17 << 19, False),
    (F32, 24 << 18, True), (F32, (24 << 18) - 32, False), (F16, 24 << 19, True), (BF16, (24 << 19) - 64, False),
    (F16, (12 << 19) + 32, False),                       # not of whole lines
])
def test_gradients_alone_write_through_at_the_sizes_that_gain(client, dtype, elements, through):
    """From 11 MiB to 17 (float32: 19), and from 24 MiB on."""
    launches, status = client((GRAD_DEQUANT, dtype, 8, 0, 1, elements, 32), options=("alone",))
    assert status == 0 and len(launches) == 1
    assert launches[0][2].split("dequant_single_kernel<")[1].split(">(")[0].endswith("true" if through else "false"), launches
    launches, status = client((DECODE, dtype, 8, 0, 1, elements, 32), options=("alone",))           # m and out
    eb = 4 if dtype == F32 else 2
    big = 2 * elements * eb >= 24 << 20 and elements * eb % 128 == 0
    assert status == 0 and launches[0][2].split(">(")[0].endswith("true" if big else "false"), launches
