"""What the compiler makes of kernels whose speed hangs on it: the listing of the library's own sources (CPU only)."""
import re
import subprocess

import pytest

from paper_2605_07330_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Demangled name -> listing of each kernel."""
    out = str(tmp_path_factory.mktemp("listing") / "srs.s")
    cmd = [a for a in build.hipcc_command(out) if a not in ("-shared", "-fPIC") and not a.startswith("-Wl,")]
    subprocess.run([*cmd, "--cuda-device-only", "-S"], check=True, stderr=subprocess.DEVNULL)
    parts = re.split(r"^(_Z\w+):[^\n]*; @", open(out).read(), flags=re.M)
    names = subprocess.run(["c++filt"], input="\n".join(parts[1::2]), capture_output=True, text=True, check=True).stdout.split("\n")
    return {n.removeprefix("void srs::").split("(")[0]: body for n, body in zip(names, parts[2::2])}


def load_runs(body, least):
    """Base operands of each run of at least `least` 16-byte loads that no branch, label or barrier interrupts."""
    runs, run = [], []
    for line in body.split("\n"):
        line = line.strip()
        m = re.match(r"global_load_dwordx4 v\[\d+:\d+\], \S+, (s\[\d+:\d+\]|off)", line)
        if m:
            run.append(m.group(1))
        elif re.match(r"(s_cbranch|s_branch|s_barrier|\.LBB|s_endpgm)", line):
            if len(run) >= least:
                runs.append(run)
            run = []
    return runs


@pytest.mark.parametrize("name,vectors", [("extract_kernel<16, true, -1, 0, 2>", 16), ("extract_kernel<16, false, -1, 0, 2>", 16)])
def test_one_stream_after_the_other(kernels, name, vectors):
    """A whole tile whose snapshot is left alone: all loads of one stream go out before the first of the other."""
    runs = load_runs(kernels[name], vectors)
    assert sum(map(len, runs)) >= 2 * vectors, runs
    for run in runs:
        assert sum(a != b for a, b in zip(run, run[1:])) <= 1, f"{name}: the streams alternate: {run}"


@pytest.mark.parametrize("name,waves", [("extract_kernel<8, false, 0, 1, 2>", 4), ("extract_kernel<8, false, 8, 1, 2>", 4),
                                        ("extract_kernel<16, true, 8, 1, 2>", 2), ("extract_kernel<16, false, 0, 1, 2>", 2),
                                        ("extract_kernel<4, true, 8, 0, 1>", 8), ("extract_kernel<4, true, -1, 0, 1>", 8)])
def test_resident_waves(kernels, name, waves):
    """The path of incomplete tiles must not take registers from the path of whole ones."""
    assert int(re.search(r"; Occupancy: (\d+)", kernels[name]).group(1)) >= waves


def test_no_extract_kernel_spills(kernels):
    """Occupancy that is reached by keeping registers in scratch memory is none."""
    spilled = {n: s for n, b in kernels.items() if "extract_" in n and (s := int(re.search(r"; ScratchSize: (\d+)", b).group(1)))}
    assert not spilled


@pytest.mark.parametrize("name", ["extract_whole_kernel<8>", "extract_whole_kernel<-1>"])
def test_whole_tiles_load_from_immediate_offsets(kernels, name):
    """The kernel for lists of whole aligned tiles: 16 loads of each stream with nothing but pauses and additions to their addresses
    between them, no choice of a position."""
    body = kernels[name]
    runs, run = [], []
    for line in body.split("\n"):
        op = line.strip().split(" ")[0]
        if op.startswith("global_load_dwordx4"):
            run.append(op)
        elif op and op[0] != ";" and not re.match(r"(s_sleep|s_nop|v_add_co_u32|v_addc_co_u32|v_lshl_add_u64|v_add_u32|s_mov|s_waitcnt)", op):
            if len(run) >= 4:
                runs.append(len(run))
            run = []
    assert 32 in runs or runs.count(16) >= 2, runs
