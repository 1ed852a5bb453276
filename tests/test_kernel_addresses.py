"""The copy kernels' addresses in long lines, on the CPU: csrc/kernels.h is
compiled for the host and its address computation run thread by thread, for
tiles around 2 GiB and just under 4 GiB into a line, against plain integer
arithmetic; and a KV block whose lines do not fit the kernels' 32-bit run is
refused before anything runs."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2511_11617_amd import atp

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_11617_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
ALIGNED, SRC_GRID = 1 << 7, 1 << 9


@pytest.fixture(scope="module")
def addresses(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("kernelhost") / "addresses")
    r = subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-w", "-I" + os.path.join(HERE, "kernelhost"),
                        "-I" + CSRC, os.path.join(HERE, "kernelhost", "addresses.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(kind, *args):
        r = subprocess.run([out, kind, *map(str, args)], capture_output=True, text=True, check=True)
        return [tuple(map(int, x.split())) for x in r.stdout.splitlines()]
    return run


BASE_S, BASE_D = 1 << 45, 3 << 45  # far from zero: an offset of the wrong sign shows


@pytest.mark.parametrize("kind", ["narrow", "wide"])
@pytest.mark.parametrize("cpl,col", [
    (140_000_001, (1 << 27) - 1), (140_000_001, 1 << 27), (140_000_001, 140_000_000),
    ((1 << 28) - 1, (1 << 28) - 2), (77, 76)])
def test_aligned_columns(addresses, kind, cpl, col):
    # two lines: the tile that holds column `col` of the first one, which crosses into the second near its end
    run, tile = cpl * 16, col // (1024 if kind == "wide" else 512)
    sp, dp = run + 4096, run + 64
    got = addresses(kind, BASE_S, BASE_D, 0, 0, sp, dp, 2, run, 1, ALIGNED, tile)
    n = 1024 if kind == "wide" else 512
    want = set()
    for c in range(tile * n, min((tile + 1) * n, 2 * cpl)):
        line, k = divmod(c, cpl)
        want.add((BASE_S + line * sp + k * 16, BASE_D + line * dp + k * 16))
    assert set(got) == want and len(got) == len(want)


@pytest.mark.parametrize("grid", ["src", "dst"])
@pytest.mark.parametrize("run", [(1 << 31) - 3, (1 << 31) + 5, (1 << 32) - 1, (1 << 32) - 16, 1000, 17])
@pytest.mark.parametrize("where", ["first", "half", "last"])
def test_unaligned_columns(addresses, grid, run, where):
    src, dst = BASE_S + 3, BASE_D + 9
    cpl = (run + 30) // 16
    tile = {"first": 0, "half": cpl // 2 // 512, "last": (cpl - 1) // 512}[where]
    got = addresses("any", src, dst, 0, 0, run, run, 1, run, 1, SRC_GRID if grid == "src" else 0, tile)
    head = (src if grid == "src" else dst) % 16
    want = []
    for c in range(tile * 512, min((tile + 1) * 512, cpl)):
        o = min(max(c * 16 - head, 0), run - 16)  # a chunk never leaves the line
        want.append((src + o, dst + o))
    assert sorted(got) == sorted(want)


def _kv_problem(heads, head_dim, block_tokens):
    """One session in one block per layer, TP 2 -> 1, old rank 0 left."""
    sp = atp.Space()
    sp.total_units, sp.old_tp, sp.new_tp = heads, 2, 1
    sp.old_rule = sp.new_rule = atp.RULE_CEIL_FIRST
    failed = (C.c_int32 * 1)(1)
    kv = atp.KV(0, 1, block_tokens, head_dim, 2, atp.KV_HEAD_MAJOR, 1, 1)
    t = atp.Tensor()
    t.space, t.kind, t.layer, t.elem_bytes = 0, atp.ROWS, 0, 2
    t.rows, t.cols, t.unit, t.old_offset = heads, 16, 1, atp.OFFSET_AUTO
    pb = atp.Problem()
    pb.n_spaces, pb.n_tensors, pb.n_failed = 1, 1, 1
    pb.spaces, pb.tensors, pb.kv = C.pointer(sp), C.pointer(t), C.pointer(kv)
    pb.failed = C.cast(failed, C.POINTER(C.c_int32))
    pb.self_old_rank = 0
    return atp.Plan(pb, keep=(sp, t, kv, failed))


def test_kv_lines_past_32_bits_are_refused():
    # 32 old heads of 128 x 2 bytes: a line is tokens * 8192 bytes
    plan = _kv_problem(64, 128, 1 << 19)  # exactly 4 GiB
    st = plan.stats()
    A, N, S, T, H = (i << 40 for i in range(1, 6))  # never dereferenced: the call is refused first
    with pytest.raises(atp.AtpError) as e:
        plan.reshard_kv(A, st.old_kv_bytes, N, st.new_kv_bytes, T, 1, 1, H, st.inflow_kv, None, 0, S, st.staging_kv,
                        0, 0)
    assert e.value.code == atp.EINVAL and "too large" in str(e.value)
