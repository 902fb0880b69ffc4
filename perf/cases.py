"""The work that users of this library have it do, as cases to measure.

A case is one call, or the two or three calls that belong together, of the
restore path on one GPU: a donor's pack, a receiver's unpack, both in turn
(a restore), the exact compare of two replicas, a checksum, the repair of a
replica from two sets of chunk sums, and a donor's stripe of a restore.
Every output is whole numbers or bytes, so results have to be the same bit
for bit (and no 64-bit evaluation of them is needed).

State tables come from three sources: a decoder's tensors with bf16
parameters, fp32 masters and fp32 Adam moments, contiguous ("decoder"); the
same under ZeRO sharding, one rank's share ("zero"); tensors of log-uniform
sizes at random 16-byte offsets, shuffled differently at the two sides
("scatter").  Chunks run from 4 KiB to 1 MiB.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2509_03047_amd import flashrestore as F
from paper_2509_03047_amd import workloads as W

_DECODERS = {
    "toy": W.toy_decoder_tensors,
    "llama3-8b-tp8": W.llama3_8b_tp8_tensors,
    "llama3-70b-tp8-pp4-stage0": W.llama3_70b_tp8_pp4_stage0_tensors,
}


def listed():
    return [
        # a handful of small odd tensors (adapters, buffers, norms): the
        # smallest restore, where launches and the host count
        dict(name="tiny-restore", op="restore", layout="scatter", entries=48, lo=16, hi=4096, table_seed=5,
             chunk=4096),
        # a small model, restored and compared, 51 MB of state
        dict(name="toy-restore", op="restore", layout="decoder", model="toy", chunk=1 << 16),
        dict(name="toy-compare", op="verify_sums", layout="decoder", model="toy", chunk=1 << 16, flips=4),
        # one rank of an optimizer-sharded (ZeRO-1) model of odd sizes, smaller chunks
        dict(name="zero1-restore", op="restore", layout="zero", layers=12, hidden=1500, ffn=4001, vocab=32003,
             stage=1, shard=3, rank=1, chunk=1 << 14),
        # one rank's share of an 8B model: the donor and the receiver of a restore
        dict(name="8b-pack", op="pack", layout="decoder", model="llama3-8b-tp8", chunk=1 << 16),
        dict(name="8b-unpack", op="unpack", layout="decoder", model="llama3-8b-tp8", chunk=1 << 16),
        # the periodic check of two replicas on one GPU
        dict(name="8b-compare", op="verify", layout="decoder", model="llama3-8b-tp8", chunk=1 << 16, flips=64),
        # replicas on two GPUs: sums compared, the differing chunks sent again
        dict(name="8b-repair", op="repair", layout="decoder", model="llama3-8b-tp8", chunk=1 << 16, flips=4096),
        # one of seven donors of a striped restore
        dict(name="8b-stripe", op="stripe", layout="decoder", model="llama3-8b-tp8", chunk=1 << 16, parts=7,
             part=3),
        # many tensors of all sizes, none of them aligned to a cache line
        dict(name="scatter-restore", op="restore", layout="scatter", entries=20000, lo=256, hi=1 << 20,
             table_seed=2, chunk=1 << 14),
        dict(name="scatter-checksum", op="checksum", layout="scatter", entries=20000, lo=256, hi=1 << 20,
             table_seed=2, chunk=1 << 14),
        # the largest state: a stage of a 70B model, large chunks
        dict(name="70b-checksum", op="checksum", layout="decoder", model="llama3-70b-tp8-pp4-stage0",
             chunk=1 << 20),
    ]


def _log(rng, lo, hi):
    """A whole number, spread evenly over the logarithm of [lo, hi]."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    while True:
        c = dict(op=rng.choice(["restore", "pack", "unpack", "verify", "verify_sums", "checksum", "repair", "stripe"]),
                 layout=rng.choice(["decoder", "zero", "scatter"]), chunk=1 << rng.randint(12, 20))
        if c["layout"] == "scatter":
            lo = _log(rng, 16, 4096)
            c.update(entries=_log(rng, 8, 20000), lo=lo, hi=lo * _log(rng, 4, 8192), table_seed=rng.randrange(1 << 20))
        else:
            hidden = _log(rng, 32, 8192)
            c.update(layers=_log(rng, 1, 40), hidden=hidden, ffn=int(hidden * rng.uniform(0.4, 4)),
                     vocab=_log(rng, 100, 130000))
            if c["layout"] == "zero":
                shard = rng.randint(2, 8)
                c.update(stage=rng.randint(1, 3), shard=shard, rank=rng.randrange(shard))
        if c["op"] in ("verify", "verify_sums", "repair"):
            c["flips"] = _log(rng, 1, 4096)
        if c["op"] == "stripe":
            c["parts"] = rng.randint(2, 7)
            c["part"] = rng.randrange(c["parts"])
        state = _bytes(_table(c)[0]).sum()
        # 64 KiB of state to 6 GB
        if 1 << 16 <= state <= 6_000_000_000:
            return c


# ------------------------------------------------------------------ tables


def _decoder(case):
    """A decoder's logical tensors (name, numel)."""
    if "model" in case:
        return _DECODERS[case["model"]]()
    d, f = case["hidden"], case["ffn"]
    t = [("embed", case["vocab"] * d)]
    for l in range(case["layers"]):
        t += [(f"l{l}.attn_norm", d), (f"l{l}.wqkv", 3 * d * d), (f"l{l}.wo", d * d), (f"l{l}.ffn_norm", d),
              (f"l{l}.fc1", 2 * d * f), (f"l{l}.fc2", f * d)]
    return t + [("final_norm", d)]


def _table(case):
    """(descriptor table, sender arena bytes, receiver arena bytes)."""
    if case["layout"] == "scatter":
        w = W.stress_workload(case["table_seed"], case["entries"], case["lo"], case["hi"], case["chunk"])
        if case["op"] == "repair":  # in place: the replica has the donor's layout
            w.table["dst_offset"] = w.table["src_offset"]
            return w.table, w.src_arena_bytes, w.src_arena_bytes
        return w.table, w.src_arena_bytes, w.dst_arena_bytes
    tensors = _decoder(case)
    if case["layout"] == "decoder":
        t, nb = W.state_table(tensors)
    else:
        lay = F.Layout3D(dp=2 * case["shard"], shard=case["shard"], zero_stage=case["stage"])
        t, nb = lay.state_table(case["rank"], [n for _, n in tensors])
    return t, nb, nb


def _bytes(table):
    return (table["numel"] * np.where(table["dtype"] == F.FR_F32, 4, 2).astype(np.uint64)).astype(np.int64)


# ------------------------------------------------------------------ inputs


def _fill(table, arena, seed):
    """Values of a training state: parameters and masters N(0, 0.02), each
    derived parameter its rounded master, first moments N(0, 1e-3), second
    ones |N(0, 1e-6)|; N(0, 1) where the table has no such roles."""
    g = torch.Generator(device=arena.device)
    g.manual_seed(seed)
    der = table["derive_from"].tolist()
    master = set(d for d in der if d >= 0)
    roles = bool(master)
    nb = _bytes(table).tolist()
    off = table["src_offset"].tolist()
    dt = table["dtype"].tolist()

    def at(k):
        return arena[off[k]: off[k] + nb[k]].view(torch.float32 if dt[k] == F.FR_F32 else torch.bfloat16)

    moment = 0
    for k in range(len(table)):
        if der[k] >= 0 or nb[k] == 0:
            continue
        x = at(k)
        if not roles:
            x.normal_(generator=g)
        elif dt[k] == F.FR_BF16 or k in master:
            x.normal_(0.0, 0.02, generator=g)
            moment = 0
        else:
            x.normal_(0.0, 1e-6 if moment else 1e-3, generator=g)
            if moment:
                x.abs_()
            moment ^= 1
    for k in range(len(table)):
        if der[k] >= 0 and nb[k]:
            at(k).copy_(at(der[k]))


def _flip(table, arena, n, seed):
    """n distinct random bits of the table's tensors flipped."""
    nb = _bytes(table).astype(np.uint64)
    ends = np.cumsum(nb)
    bits = W.flip_positions(int(ends[-1]) * 8, n, seed)
    k = np.searchsorted(ends, bits >> 3, side="right")
    byte = table["src_offset"][k] + (bits >> 3) - (ends[k] - nb[k])
    masks = {}
    for b, q in zip(byte.tolist(), (bits & 7).tolist()):
        masks[b] = masks.get(b, 0) ^ (1 << q)
    i = torch.tensor(list(masks), dtype=torch.int64, device=arena.device)
    m = torch.tensor(list(masks.values()), dtype=torch.uint8, device=arena.device)
    arena[i] = arena[i] ^ m


def prepare(case, seed):
    table, src_bytes, dst_bytes = _table(case)
    op = case["op"]
    s = dict(op=op, plan=F.Plan(table, case["chunk"], src_bytes, dst_bytes))
    plan = s["plan"]
    src = torch.zeros(src_bytes, dtype=torch.uint8, device="cuda")
    _fill(table, src, seed)
    if op in ("pack", "restore", "unpack"):
        s["payload"], s["sums"] = plan.empty_payload(), plan.empty_sums()
    if op in ("restore", "unpack"):
        s["dst"] = torch.zeros(dst_bytes, dtype=torch.uint8, device="cuda")
        s["bad"], s["n_bad"] = plan.empty_bitmap(), plan.empty_counter()
    if op == "unpack":  # what has arrived from the donor
        plan.pack(src, s["payload"], s["sums"])
        return s
    s["src"] = src
    if op == "checksum":
        s["sums"] = plan.empty_sums()
    if op in ("verify", "verify_sums", "repair"):
        s["replica"] = src.clone()
        _flip(table, s["replica"], case["flips"], seed)
        s["diff"], s["n_diff"] = plan.empty_bitmap(), plan.empty_counter()
    if op in ("verify_sums", "repair"):
        s["sums_a"], s["sums_b"] = plan.empty_sums(), plan.empty_sums()
    if op == "repair":
        # each rank's sums have been exchanged; rows and bytes past the list stay as they are
        plan.checksum_state(src, s["sums_a"])
        plan.checksum_state(s["replica"], s["sums_b"])
        s["payload"], s["sums"] = plan.empty_delta_payload().zero_(), plan.empty_sums().zero_()
        s["counts"] = torch.zeros(2, dtype=torch.int64, device="cuda")
        s["bad"], s["n_bad"] = plan.empty_bitmap(), plan.empty_counter()
    if op == "stripe":
        k, n, c = case["part"], case["parts"], plan.n_chunks
        s["ids"] = np.arange(c * k // n, c * (k + 1) // n, dtype=np.uint32)
        s["payload"] = torch.empty(max(plan.delta_layout(s["ids"]), 16), dtype=torch.uint8, device="cuda").zero_()
        s["sums"] = torch.empty(max(len(s["ids"]), 1), 2, dtype=torch.int64, device="cuda").zero_()
    return s


# ------------------------------------------------------------------- calls


def _whole(x):
    """A buffer's bytes as 64-bit words."""
    return x.view(torch.int64)


def run(s):
    op, plan = s["op"], s["plan"]
    if op == "pack":
        plan.pack(s["src"], s["payload"], s["sums"])
        return [_whole(s["payload"]), s["sums"]]
    if op == "unpack":
        plan.unpack(s["payload"], s["sums"], s["dst"], s["bad"], s["n_bad"])
        return [_whole(s["dst"]), s["bad"], s["n_bad"]]
    if op == "restore":
        plan.pack(s["src"], s["payload"], s["sums"])
        plan.unpack(s["payload"], s["sums"], s["dst"], s["bad"], s["n_bad"])
        return [_whole(s["payload"]), s["sums"], _whole(s["dst"]), s["bad"], s["n_bad"]]
    if op == "verify":
        plan.verify_replicas(s["src"], s["replica"], s["diff"], s["n_diff"])
        return [s["diff"], s["n_diff"]]
    if op == "verify_sums":
        plan.verify_replicas(s["src"], s["replica"], s["diff"], s["n_diff"], s["sums_a"], s["sums_b"])
        return [s["diff"], s["n_diff"], s["sums_a"], s["sums_b"]]
    if op == "checksum":
        plan.checksum_state(s["src"], s["sums"])
        return [s["sums"]]
    if op == "repair":
        plan.compare_sums(s["sums_a"], s["sums_b"], s["diff"], s["n_diff"])
        plan.pack_flagged(s["src"], s["diff"], s["payload"], s["sums"], s["counts"])
        plan.unpack_flagged(s["payload"], s["sums"], s["diff"], s["replica"], s["bad"], s["n_bad"])
        return [s["diff"], s["n_diff"], _whole(s["payload"]), s["sums"], s["counts"], _whole(s["replica"]), s["bad"],
                s["n_bad"]]
    plan.pack_chunks(s["src"], s["ids"], s["payload"], s["sums"])
    return [_whole(s["payload"]), s["sums"]]


def work(case):
    table = _table(case)[0]
    nb = _bytes(table)
    state = int(nb.sum())
    sent = int(nb[table["derive_from"] < 0].sum())
    chunks = -(-nb // case["chunk"])
    n = int(chunks.sum())
    sums, bits = 16 * n, n // 8
    pack, unpack = state + sent + sums, sent + state + sums + bits
    op = case["op"]
    if op == "repair":
        # chunks hit by at least one flip, on average; each is read, sent and
        # written, and a listed parameter chunk read and written
        p = 1.0 - (1.0 - np.minimum(nb / np.maximum(chunks, 1), case["chunk"]) / state) ** case["flips"]
        listed_b = float((p * nb).sum())
        sent_b = float((p * nb)[table["derive_from"] < 0].sum())
        b = 2 * sums + 2 * bits + 2 * (listed_b + sent_b)
    else:
        b = {"pack": pack, "unpack": unpack, "restore": pack + unpack, "verify": 2 * state + bits,
             "verify_sums": 2 * state + bits + 2 * sums, "checksum": state + sums,
             "stripe": pack / case.get("parts", 1)}[op]
    # a checksum's two multiply-adds a word are no bound: bytes are
    return {"bytes": float(b), "flops": 0.0}


def tolerance(case):
    return "exact"
