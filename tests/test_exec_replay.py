"""The executor's host logic on the CPU (no GPU): reshards of the workloads,
in and out of place, in both call orders, with and without atp_warmup, run
through libatp.so in a child process whose HIP runtime is the host-only
stand-in in tests/mockhip.  The stand-in aborts on any copy outside its
allocations or with the wrong host/device sides, and on any use of an
unknown event or stream; the executor must issue every call, sync it and
stay within the bounded side-stream search."""
import json
import os
import subprocess
import sys

import pytest

from tests.gpu_harness import late_gates_cfg

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def mockhip(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("mockhip") / "libmockhip.so")
    src = os.path.join(HERE, "mockhip")
    r = subprocess.run(["g++", "-O1", "-g", "-fPIC", "-shared", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", f"-Wl,--version-script={src}/mock.map", f"{src}/mock_hip.cpp",
                        "-o", out], capture_output=True, text=True)
    if r.returncode:
        pytest.skip("cannot build the HIP stand-in: " + r.stderr[-500:])
    return out


def _replay(mockhip, cases, tmp=None):
    env = dict(os.environ)
    if tmp is not None:
        env["ATP_REPLAY_TMP"] = str(tmp)
    # appended, so that anything already preloaded stays first
    env["LD_PRELOAD"] = ":".join(x for x in (env.get("LD_PRELOAD", ""), mockhip) if x)
    env["ATP_MOCKHIP"] = mockhip
    r = subprocess.run([sys.executable, os.path.join(HERE, "exec_replay.py"), json.dumps(cases)], env=env,
                       capture_output=True, text=True, timeout=600)
    assert "MOCKHIP FAULT" not in r.stderr, r.stderr[-3000:]
    assert r.returncode == 0 and "replay done" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])
    return [json.loads(x) for x in r.stdout.splitlines() if x.startswith("{")]


def test_out_of_place_both_orders(mockhip):
    cases = [{"w": w, "inplace": False, "order": o, "steps": 2, "warmup": wu}
             for w in (1, 2, 3, 4) for o in ("weights-first", "kv-first") for wu in (False, True)]
    res = _replay(mockhip, cases)
    assert len(res) == len(cases)
    for i, r in enumerate(res):
        assert r.get("ok"), r
        assert all(n > 0 for n in r["launches"])
        # two caller streams per case so far, plus at most eight side-stream candidates per device
        assert r["streams"] <= 2 * (i + 1) + 8


def test_in_place_weights_first_and_kv_first_refused(mockhip):
    cases = [{"w": 5, "inplace": True, "order": "weights-first", "steps": 2, "warmup": False},
             {"w": 2, "inplace": True, "order": "weights-first", "steps": 2, "warmup": True},
             {"w": 1, "inplace": True, "order": "weights-first", "steps": 3, "warmup": False},
             {"w": 1, "inplace": True, "order": "kv-first", "steps": 1, "warmup": False}]
    res = _replay(mockhip, cases)
    assert [r.get("ok") for r in res[:3]] == [True] * 3
    assert res[0]["launches"][0] > 100  # 22 weight and 25 KV levels, outbound reads, ring scatters
    assert res[3]["refused"] == -5 and "before" in res[3]["msg"]


def test_in_place_kv_inflow_pinned_at_both_ends_only(mockhip):
    """An in-place KV inflow buffer whose first and last page are pinned apart,
    with pageable memory between, takes the landing ring's copies: the copy
    kernel would fault on it."""
    case = {"w": 5, "inplace": True, "order": "weights-first", "steps": 1, "warmup": False}
    whole, = _replay(mockhip, [case])
    split, = _replay(mockhip, [dict(case, split_kv_inflow=True)])
    assert whole["ok"] and split["ok"]
    assert split["mock_copies"] > whole["mock_copies"]


@pytest.mark.parametrize("layout,head_dim,kernel,groups", [
    ("head", 128, "k_copy_linkILi4E", 10),   # items of 4096 bytes
    ("head", 80, "k_copy_linkILi2E", 24),    # 2560: waves cross items
    ("token", 128, "k_copy_linkILi4E", 10),  # 16 tokens of 256 bytes
    ("token", 72, "k_copy_linkILi2E", 24)])  # 16 of 144
def test_in_place_kv_reads_of_lines_that_cross_waves(mockhip, layout, head_dim, kernel, groups):
    """In-place KV lines whose items are not whole KiBs are read with narrow
    tiles on 24 workgroups: wide ones on 10 left the link idle."""
    case = {"w": 5, "inplace": True, "order": "weights-first", "steps": 1, "warmup": False, "layers": 2, "log": True,
            "shape": {"kv_layout": layout, "head_dim": head_dim, "n_seq": 16, "seq_tokens": 1024}}
    r, = _replay(mockhip, [case])
    reads = [(n, g) for n, g, stream in r["log"] if stream == "copy" and "k_copy" in n]
    assert reads and all(kernel in n and g == groups for n, g in reads), reads


def test_in_place_kv_inflow_with_late_gates_goes_to_its_slots(mockhip):
    """Where every read in place would wait for the preparation of thousands
    of descriptors and for a level, the first chunks are read into their slots
    at once and scattered after the levels; with few descriptors the reads go
    straight into place, and with one stream for both none holds up the
    levels."""
    late, few = late_gates_cfg(), late_gates_cfg(fragmented=False, pool_factor=1.0, n_seq=1, seq_tokens=64)
    r = {}
    for name, c in (("late", late), ("few", few), ("one-stream", late)):
        case = {"w": 1, "inplace": True, "order": "weights-first", "steps": 1, "warmup": False, "log": True,
                "shape": c, "one_stream": name == "one-stream"}
        r[name], = _replay(mockhip, [case])
        assert r[name]["ok"]
    kinds = {k: [n for n, g, s in v["log"] if n != "copy"] for k, v in r.items()}
    linear = [i for i, n in enumerate(kinds["late"]) if "k_copy_linear" in n]
    prepares = [i for i, n in enumerate(kinds["late"]) if "k_prepare" in n]
    assert linear and linear[0] < prepares[-1]  # before the KV call's own preparation
    assert not any("k_copy_linear" in n for n in kinds["few"] + kinds["one-stream"])


@pytest.mark.parametrize("order", ["kv-only", "weights-first"])
def test_in_place_kv_reads_beside_outbound_copies_are_held_back(mockhip, order):
    """An in-place KV call that copies bytes out reads as many bytes of its
    inflow with a grid that leaves the copies their share of the link, all of
    them with the weights call pending, and the rest with the usual one."""
    shape = dict(late_gates_cfg(n_q=16, n_kv=8, head_dim=80, layers=4, fragmented=False, pool_factor=1.0,
                                block_tokens=16), new_kv_widths=[4, 4], kv_rule="widths")
    r, = _replay(mockhip, [{"w": 1, "inplace": True, "order": order, "steps": 1, "warmup": False, "log": True,
                            "shape": shape}])
    log = [x for x in r["log"] if x[2] == "copy" or x[0] == "copy"]
    out = sum(g for n, g, s in log if n == "copy" and s == "side")
    reads = [(n, g) for n, g, s in log if s == "copy" and "k_copy" in n]
    assert out > 0 and not any("linear" in n for n, g in reads)
    held = [("k_copy16ILi2" in n and g == 20) for n, g in reads]
    assert held[0] and held == sorted(held, reverse=True)
    assert all(held) if order == "weights-first" else not held[-1]


def test_outbound_reads_of_a_weights_call_alone_get_their_whole_grid(mockhip):
    """The plan describes a KV cache whose inflow would outlast the weights'
    outbound reads, but whether the KV call is made is not known yet."""
    r, = _replay(mockhip, [{"w": 5, "inplace": True, "order": "weights-only", "steps": 1, "warmup": False, "layers": 2,
                            "log": True, "shape": {"n_seq": 32}}])
    side = [(n, g) for n, g, s in r["log"] if s == "side" and "k_copy" in n]
    assert {g for n, g in side if "k_copy_linkILi2" in n} == {4}, side


def test_awaited_reads_in_place_follow_the_buffer(mockhip, tmp_path):
    """While the inflow buffer is filled from files, the weight pieces of an
    in-place call go out in the order in which the buffer fills, each reading
    the buffer in about one place, not in the order their places get free."""
    r, = _replay(mockhip, [{"w": 5, "inplace": True, "order": "async-load", "steps": 1, "warmup": False, "layers": 24,
                            "log": True, "shape": {"hidden": 2048, "ffn": 5632, "n_q": 16, "n_kv": 8, "n_seq": 2,
                                                   "seq_tokens": 64}}], tmp_path)
    n = len(r["reads"])
    assert sum(b for _, _, b in r["reads"]) > 200e6
    spans = [tuple(map(int, k.split(":")[1:])) for k, g, s in r["log"] if s == "side" and "k_copy" in k]
    # the weights' reads are the last descriptors launched, and no others come after them on that stream
    d0 = max(d1 for _, d1 in spans) - n
    pieces = [(a - d0, b - d0) for a, b in spans if a >= d0]
    assert sorted(x for a, b in pieces for x in range(a, b)) == list(range(n))
    ends = [max(e for _, e, _ in r["reads"][a:b]) for a, b in pieces]
    assert ends == sorted(ends)
    for a, b in pieces:
        lo, hi = min(s for s, _, _ in r["reads"][a:b]), max(e for _, e, _ in r["reads"][a:b])
        assert hi - lo <= max(2 * sum(x for _, _, x in r["reads"][a:b]), 64 << 20)


@pytest.mark.parametrize("blocks", [65536, 65537, 300000])
def test_a_large_pool_is_marked_by_one_launch(mockhip, blocks):
    """One pass over the block table, whatever the number of windows."""
    r, = _replay(mockhip, [{"w": 1, "inplace": False, "order": "kv-only", "steps": 1, "warmup": False, "layers": 1,
                            "log": True, "shape": {"block_tokens": 1, "n_seq": 1, "seq_tokens": blocks}}])
    assert sum("k_mark_pool" in n for n, g, s in r["log"]) == int(blocks > 65536)


def test_many_descriptors_go_to_the_device_by_a_copy_command(mockhip):
    case = {"w": 1, "inplace": True, "order": "weights-first", "steps": 1, "warmup": False, "log": True}
    many, few = _replay(mockhip, [dict(case, shape=late_gates_cfg()), dict(case, shape=late_gates_cfg(
        fragmented=False, pool_factor=1.0, n_seq=1, seq_tokens=320))])
    copies = [g for n, g, s in many["log"] if n == "copy" and s == "compute"]
    assert len(copies) == 1 and copies[0] > 96 * 1024  # the KV call's 6358 descriptors; the weights call has few
    assert not [g for n, g, s in few["log"] if n == "copy" and s == "compute"]


def test_async_load_with_the_kv_call_between(mockhip, tmp_path):
    """atp_load_reshard_weights_async, the KV call while the reads run, then
    atp_sync issuing the weight pieces: in and out of place, fresh plans in
    a row, with the reads from a checkpoint of holes."""
    cases = [{"w": 1, "inplace": False, "order": "async-load", "steps": 2, "warmup": False},
             {"w": 1, "inplace": True, "order": "async-load", "steps": 2, "warmup": True},
             {"w": 2, "inplace": False, "order": "async-load", "steps": 2, "warmup": False, "layers": 1},
             {"w": 2, "inplace": True, "order": "async-load", "steps": 2, "warmup": False, "layers": 1}]
    res = _replay(mockhip, cases, tmp_path)
    assert [r.get("ok") for r in res] == [True] * 4, res
