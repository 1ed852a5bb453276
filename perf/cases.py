"""Timed cases of the reshard: what one surviving GPU does when a rank of its
tensor-parallel group dies.

A case is one decoder shape, one TP change N -> N-1 as one survivor sees it,
a paged KV cache, and the entry points a program calls for it:

  whole       plan, weights call, KV call, sync: a recovery's hot path
  weights     plan, weights call, sync
  kv          plan, KV call, sync
  kv_noalloc  a plan kept across calls, the no-allocation KV call, sync: the
              form a serving loop uses

A pass is one such sequence.  Its outputs are the arenas it leaves (and, in
place, the packed bytes it read out for its peers).  Bytes are only moved,
so outputs are compared exactly.  Plans are made inside the pass, as a
recovery makes them, except for kv_noalloc.
"""
import numpy as np
import torch

from paper_2511_11617_amd import atp, problem

# Decoder shapes per layer: the tiny one, the dense and mixture-of-experts
# decoders of the repository's workloads, and two generic mid-size ones.
TINY = dict(hidden=256, n_q=4, n_kv=2, head_dim=64, ffn=688, ffn_unit=1, experts=0, expert_ffn=0)
MID = dict(hidden=1024, n_q=16, n_kv=8, head_dim=64, ffn=2816, ffn_unit=1, experts=0, expert_ffn=0)
LARGE = dict(hidden=4096, n_q=32, n_kv=8, head_dim=128, ffn=11008, ffn_unit=16, experts=0, expert_ffn=0)
DENSE5120 = dict(hidden=5120, n_q=40, n_kv=8, head_dim=128, ffn=17408, ffn_unit=16, experts=0, expert_ffn=0)
DENSE8192 = dict(hidden=8192, n_q=64, n_kv=8, head_dim=128, ffn=28672, ffn_unit=16, experts=0, expert_ffn=0)
MOE = dict(hidden=2048, n_q=32, n_kv=4, head_dim=128, ffn=0, ffn_unit=16, experts=128, expert_ffn=768)

STAGING_CAP = 2 << 30  # in place, as the largest workload states it


def _case(shape, name=None, **kw):
    c = dict(call="whole", layers=2, old_tp=4, failed=1, self_old=0, kv_rule="gqa", kv_layout="head",
             block_tokens=16, n_seq=8, seq_tokens=128, pool_percent=100, in_place=False, keep_percent=100)
    c.update(shape)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest recovery: every launch and host call counts
        _case(TINY, "tiny_whole"),
        # the same in place with token-major KV: the shortest lines there are (128 B per token and head)
        _case(TINY, "tiny_token_in_place", kv_layout="token", in_place=True),
        # a serving loop with a few short sessions moves its KV without allocating
        _case(DENSE5120, "kv_noalloc_few_sessions", call="kv_noalloc", layers=40, self_old=3, kv_rule="even",
              n_seq=4, seq_tokens=512),
        # token-major KV pages (the layout attention kernels that gather by token use)
        _case(DENSE5120, "kv_token_major", call="kv", layers=8, self_old=3, kv_layout="token",
              n_seq=32, seq_tokens=2048),
        # half of the sessions survive the budget and are compacted, from a fragmented pool
        _case(DENSE5120, "kv_compact_after_evict", call="kv", layers=40, old_tp=8, self_old=7,
              n_seq=64, seq_tokens=4096, pool_percent=112, keep_percent=50),
        # FFN split by single columns: ragged row-parallel weight lines
        _case(DENSE5120, "weights_ragged_columns", call="weights", layers=8, old_tp=8, self_old=6, ffn_unit=1),
        # named share of the dense 4 -> 3 workload, a tenth of its layers
        _case(DENSE5120, "dense_4to3_4_layers", layers=4, self_old=2, kv_rule="even", n_seq=32, seq_tokens=4096),
        # the mixture-of-experts 4 -> 3 workload, a twelfth of its layers
        _case(MOE, "moe_4to3_4_layers", layers=4, self_old=2, n_seq=64, seq_tokens=4096),
        # the survivor with the most to keep: the dense 8 -> 7 workload, all 40 layers, fragmented pool
        _case(DENSE5120, "dense_8to7_last_rank", layers=40, old_tp=8, self_old=7, n_seq=64, seq_tokens=8192,
              pool_percent=112),
        # the in-place 8 -> 7 workload, four of its layers: levels, outbound reads and the landing ring
        _case(DENSE8192, "in_place_8to7_4_layers", layers=4, old_tp=8, self_old=2, n_seq=128, seq_tokens=8192,
              in_place=True),
        # one layer group of the state plane, in place, on the last rank
        _case(DENSE5120, "in_place_layer_group", layers=2, self_old=3, kv_rule="even", n_seq=32, seq_tokens=4096,
              in_place=True),
        # in place with little inflow: the chain of dependent levels
        _case(DENSE5120, "in_place_last_rank", layers=8, old_tp=8, self_old=7, n_seq=64, seq_tokens=8192,
              in_place=True),
    ]


def _built(c, n_live=None, pool=None):
    shape = dict(c, new_tp=c["old_tp"] - 1, failed=[c["failed"]], elem_bytes=2)
    if c["kv_rule"] == "even" and c["n_kv"] >= c["old_tp"] - 1:
        shape["kv_rule"] = "widths"
        shape["new_kv_widths"] = [b - a for a, b in atp.partition(c["n_kv"], c["old_tp"] - 1, atp.RULE_CEIL_FIRST)]
    else:
        shape["kv_rule"] = "gqa"
    flags = (atp.INPLACE if c["in_place"] else 0) | (atp.KV_COMPACT if c["keep_percent"] < 100 else 0)
    total, p = _blocks(c)
    return problem.build(shape, n_live=total if n_live is None else n_live, pool=p, flags=flags,
                         staging_cap=STAGING_CAP if c["in_place"] else 0, with_kv=c["call"] != "weights")


def _blocks(c):
    """(live blocks, pool) of the whole block table."""
    live = c["n_seq"] * -(-c["seq_tokens"] // c["block_tokens"])
    return live, -(-live * c["pool_percent"] // 100)


def _sessions_kept(c):
    return max(1, c["n_seq"] * c["keep_percent"] // 100)


def _stats(c):
    kept = _sessions_kept(c) * -(-c["seq_tokens"] // c["block_tokens"])
    return _built(c, n_live=kept).plan().stats()


def _parts(c):
    return c["call"] in ("whole", "weights"), c["call"] != "weights"


def work(case):
    """Every retained byte that moves is read once and written once, every
    inflow byte read from host memory and written, every outbound byte (in
    place) read and written to host memory."""
    st = _stats(case)
    w, k = _parts(case)
    moved = st.moved_w * w + st.moved_kv * k
    inflow = st.inflow_w * w + st.inflow_kv * k
    out = (st.outbound_w * w + st.outbound_kv * k) if case["in_place"] else 0
    return {"bytes": 2 * (moved + inflow + out), "flops": 0}


def tolerance(case):
    return "exact"


def draw(rng):
    """One more case: shapes, layers, sessions, ranks and options over the
    ranges of the listed ones, within the largest one's cost."""
    while True:
        shape = dict(rng.choice([TINY, MID, MID, LARGE, LARGE, DENSE5120, DENSE5120, DENSE8192, MOE]))
        n = rng.randint(3, 8)
        if n > shape["n_q"]:
            n = rng.choice([3, 4])
        failed = rng.randrange(n)
        c = _case(shape, call=rng.choice(["whole", "whole", "whole", "weights", "kv", "kv_noalloc"]),
                  layers=round(2 ** rng.uniform(0, 5.3)), old_tp=n, failed=failed,
                  self_old=rng.choice([r for r in range(n) if r != failed]), kv_rule=rng.choice(["gqa", "even"]),
                  kv_layout=rng.choice(["head", "head", "token"]), block_tokens=rng.choice([8, 16, 16, 32]),
                  n_seq=round(2 ** rng.uniform(1, 7)), seq_tokens=round(2 ** rng.uniform(6, 13)),
                  pool_percent=rng.choice([100, 100, 112, 130]))
        c["head_dim"] = rng.choice([c["head_dim"], c["head_dim"], 64, 80, 96, 128])
        if not c["experts"]:
            c["ffn_unit"] = rng.choice([c["ffn_unit"], 1, 8, 16])
        if c["call"] == "kv" and rng.random() < 0.5:
            c["keep_percent"] = rng.choice([25, 50, 75])
        elif c["call"] != "kv_noalloc":
            c["in_place"] = rng.random() < 0.35
        try:
            st = _stats(c)
        except atp.AtpError:  # a staging need over the cap
            continue
        b = work(c)["bytes"]
        inflow = st.inflow_w + st.inflow_kv
        arenas = st.old_arena_bytes + st.new_arena_bytes + st.old_kv_bytes + st.new_kv_bytes
        if c["call"] == "kv_noalloc" and st.staging_kv > atp.scratch_bytes():
            continue
        if 1 << 20 <= b <= 16e9 and inflow <= 1.4e9 and st.outbound_w + st.outbound_kv <= 0.3e9 and arenas <= 30e9:
            return c


_side = {}


def _streams():
    """The program's compute stream and its copy stream, and the library's
    one-time set-up for them."""
    if not _side:
        _side["copy"] = torch.cuda.Stream()
        atp.warmup(torch.cuda.current_stream().cuda_stream, _side["copy"].cuda_stream, 256)
    return torch.cuda.current_stream(), _side["copy"]


def _normal(n_bytes, sigma, gen):
    """n_bytes (a multiple of 8) of normal bfloat16 values, as bytes."""
    t = torch.empty(n_bytes // 2, dtype=torch.bfloat16, device="cuda")
    return t.normal_(0.0, sigma, generator=gen).view(torch.uint8)


def _up(n):
    return max(256, -(-n // 256) * 256)


def _pinned(n):
    return torch.empty(_up(n), dtype=torch.uint8, pin_memory=True)


def _filled_host(n, sigma, gen):
    t = _pinned(n)
    t.copy_(_normal(t.numel(), sigma, gen))
    return t


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    compute, copy = _streams()
    _, pool = _blocks(case)
    bps = -(-case["seq_tokens"] // case["block_tokens"])
    rng = np.random.Generator(np.random.PCG64(seed))
    live = case["n_seq"] * bps
    ids = rng.permutation(pool)[:live] if case["pool_percent"] > 100 else np.arange(live)
    table = ids.reshape(case["n_seq"], bps).astype(np.int32)
    if case["keep_percent"] < 100:
        # least recently used sessions go until the kept ones fit the budget
        keep, table, _ = atp.kv_evict_lru(table, rng.permutation(case["n_seq"]), pool, 1,
                                          _sessions_kept(case) * bps)
    n_live = int(np.count_nonzero(table >= 0))
    built = _built(case, n_live=n_live)
    plan = built.plan()
    st = plan.stats()
    w, k = _parts(case)
    s = dict(case=case, built=built, plan=plan if case["call"] == "kv_noalloc" else None,
             compute=compute.cuda_stream, copy=copy.cuda_stream, shape=table.shape,
             table=torch.from_numpy(np.ascontiguousarray(table)).cuda())
    for on, tag, old, new, inflow, out, staging, sigma in (
            (w, "w", st.old_arena_bytes, st.new_arena_bytes, st.inflow_w, st.outbound_w, st.staging_w, 0.02),
            (k, "k", st.old_kv_bytes, st.new_kv_bytes, st.inflow_kv, st.outbound_kv, st.staging_kv, 1.0)):
        if not on:
            continue
        if case["in_place"]:
            s["old_" + tag] = _normal(_up(max(old, new)), sigma, gen)
            s["new_" + tag] = None
            s["out_" + tag] = _pinned(out).zero_()
        else:
            s["old_" + tag] = _normal(_up(old), sigma, gen)
            s["new_" + tag] = torch.zeros(_up(new), dtype=torch.uint8, device="cuda")
            s["out_" + tag] = None
        s["in_" + tag] = _filled_host(inflow, sigma, gen)
        s["n_" + tag] = (inflow, out if case["in_place"] else 0)
        s["stage_" + tag] = torch.empty(_up(staging), dtype=torch.uint8, device="cuda")
    if s["plan"] is not None:
        # the loop's first call takes its events and buffers from the pool
        atp.warmup(s["compute"], s["copy"], 256)
        run(s)
        s["new_k"].zero_()
    return s


def _buffers(s, tag):
    old, new, out = s["old_" + tag], s["new_" + tag], s["out_" + tag]
    a = (old.data_ptr(), old.numel(), new.data_ptr() if new is not None else None,
         new.numel() if new is not None else 0)
    h = (s["in_" + tag].data_ptr(), s["n_" + tag][0], out.data_ptr() if out is not None else None, s["n_" + tag][1])
    g = (s["stage_" + tag].data_ptr(), s["stage_" + tag].numel())
    return a, h, g


def _words(t):
    return t.view(torch.int64)


def run(state):
    s = state
    w, k = _parts(s["case"])
    plan = s["plan"] or s["built"].plan()
    if w:
        a, h, g = _buffers(s, "w")
        plan.reshard_weights(*a, *h, *g, s["compute"], s["copy"])
    if k:
        a, h, g = _buffers(s, "k")
        table = (s["table"].data_ptr(), *s["shape"])
        if s["plan"] is not None:
            plan.reshard_kv_noalloc(*a, *table, *h, s["compute"], s["copy"])
        else:
            plan.reshard_kv(*a, *table, *h, *g, s["compute"], s["copy"])
    plan.sync()
    outs = []
    for tag in ("w" if w else "") + ("k" if k else ""):
        outs.append(_words(s["old_" + tag] if s["new_" + tag] is None else s["new_" + tag]))
        if s["out_" + tag] is not None:
            outs.append(_words(s["out_" + tag]))
    return outs
