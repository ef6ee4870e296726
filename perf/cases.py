"""The work a serving engine has this library do, as measurable cases.

Five kinds, each through the public calls of paper_2609_33762_amd.api:

  tier     store pages into host slots and load other slots into pages, on
           one stream or on two at once (an agent turn's write-back beside
           another request's restore);
  restore  a request's whole restore: chained keys of its prompt, lookup,
           load of the resident prefix, unpin;
  layered  a prefix loaded layer by layer, a consumer stream checksumming
           each layer behind its event;
  hbm      pages gathered into a device buffer and scattered from it into
           other pages (moving KV inside HBM);
  hash     chained block keys of a batch of sequences, from host tokens, from
           device tokens with host offsets, or with everything on the device.

All outputs are bytes and whole numbers, so every tolerance is "exact".
"""
import hashlib
import math

import numpy as np
import torch

from paper_2609_33762_amd import api

VOCAB = 32000


def listed():
    qwen3 = dict(layers=48, heads=4, head_dim=128, elem=2, page_tokens=16, scales=False)
    tp8 = dict(qwen3, heads=1)
    dense = dict(qwen3, layers=32, heads=8)
    return [
        # the smallest transfers: a tiny cache's 32 pages out and 32 others in,
        # where launches and latency are all there is
        dict(name="tiny_roundtrip", kind="tier", layers=2, heads=2, head_dim=64, elem=2,
             page_tokens=16, scales=False, pages=256, chunk=1, store=32, load=32, two=False),
        # a dense model's scattered calls of a few 2 MiB pages
        dict(name="dense_call", kind="tier", pages=2048, chunk=1, store=3, load=3, two=False,
             **dense),
        # one agent turn on a rank of TP8: 32k tokens written back beside the
        # restore of 24k tokens, each on its own stream
        dict(name="tp8_turn", kind="tier", pages=20000, chunk=1, store=2000, load=1500, two=True,
             **tp8),
        # a request's restore in 1,024-token host chunks on a rank of TP8: a
        # 24,576-token prompt whose first 23 chunks are in the tier
        dict(name="chunk_restore", kind="restore", pages=4096, chunk=64, tokens=24576, resident=23,
             **tp8),
        # the layer-pipelined fp8 prefix with its scales on a rank of TP8
        dict(name="layered_fp8", kind="layered", layers=48, heads=1, head_dim=128, elem=1,
             page_tokens=16, scales=True, pages=8192, chunk=1, load=4096),
        # a few dense pages moved inside HBM, and a whole 2,000-page refill
        dict(name="hbm_small", kind="hbm", pages=2048, moved=8, **dense),
        dict(name="hbm_refill", kind="hbm", pages=20000, moved=2000, **qwen3),
        # first lookups, host tokens in and host keys out: four short prompts,
        # and an agent's 56,000-token prompt as one chain
        dict(name="hash_tiny", kind="hash", entry="host", seqs=4, shortest=512, longest=512,
             block=16, parents=False),
        dict(name="hash_prompt", kind="hash", entry="host", seqs=1, shortest=56000, longest=56000,
             block=16, parents=False),
        # the agent pool's turns: 64 prompts' new tokens continued from their
        # cached parent keys, ragged
        dict(name="hash_agents", kind="hash", entry="device", seqs=64, shortest=500, longest=4300,
             block=16, parents=True),
        # large batches with everything on the device: ragged prompts, and the
        # even batch of many short ones
        dict(name="hash_ragged", kind="hash", entry="offsets", seqs=12000, shortest=40,
             longest=2000, block=16, parents=True),
        dict(name="hash_batch", kind="hash", entry="offsets", seqs=65536, shortest=256,
             longest=256, block=16, parents=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng):
    elem = rng.choice([1, 2])
    return dict(layers=rng.choice([24, 32, 40, 48]), heads=rng.choice([1, 2, 3, 4, 8]),
                head_dim=rng.choice([64, 80, 128]), elem=elem, page_tokens=rng.choice([16, 16, 32]),
                scales=elem == 1 and rng.random() < 0.7)


def draw(rng):
    kind = rng.choice(["tier", "restore", "layered", "hbm", "hash", "hash", "hash"])
    if kind == "hash":
        block = rng.choice([16, 16, 16, 32, 48, 64, 256, 1024])
        entry = rng.choice(["host", "device", "offsets", "noalloc"])
        most = 16 << 20 if entry != "host" else 1 << 20  # tokens of the batch
        seqs = _log(rng, 1, 66000 if entry != "host" else 600)
        longest = _log(rng, block, max(block, min(64000, most // seqs)))
        shortest = rng.choice([longest, max(1, longest // 2), max(1, longest // 40)])
        return dict(kind="hash", entry=entry, seqs=seqs, shortest=shortest, longest=longest,
                    block=block, parents=rng.random() < 0.5)
    sh = _draw_shape(rng)
    page = sh["layers"] * _piece(sh)
    if kind == "hbm":
        moved = _log(rng, 1, max(1, min(4500, (3 << 30) // page)))
        return dict(kind=kind, pages=2 * moved + rng.randrange(1, 2000), moved=moved, **sh)
    if kind == "layered":
        load = _log(rng, 1, max(1, min(4096, (800 << 20) // page)))
        return dict(kind=kind, pages=load + rng.randrange(1, 4096), chunk=1, load=load, **sh)
    chunk = rng.choice([1, 1, 16, 64])
    slots = (580 << 20) // (page * chunk)  # a side's most
    if kind == "restore":
        resident = _log(rng, 1, max(1, min(slots, 1500)))
        total = resident + max(1, resident // 50)
        return dict(kind=kind, pages=chunk * (total + 2) + rng.randrange(1, 500), chunk=chunk,
                    tokens=total * chunk * sh["page_tokens"] + rng.randrange(0, 16),
                    resident=resident, **sh)
    store, load = (_log(rng, 1, max(1, min(slots, 1800))) for _ in "sl")
    return dict(kind=kind, pages=chunk * (store + load) + rng.randrange(1, 2000), chunk=chunk,
                store=store, load=load, two=rng.random() < 0.5, **sh)


# ---------------------------------------------------------------- inputs

def _piece(c):
    return 2 * c["page_tokens"] * c["heads"] * c["head_dim"] * c["elem"]


def _slot_bytes(c, chunk):
    trailer = (c["layers"] * chunk * 8 + 255) // 256 * 256 if c["scales"] else 0
    return c["layers"] * chunk * _piece(c) + trailer


def _gen(seed, role):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * seed + role)
    return g


def _device_bytes(n, seed, role, bf16):
    """bf16 N(0,1) values, or uniform bytes (fp8 payloads and scales)."""
    t = torch.empty(n, dtype=torch.uint8, device="cuda")
    if bf16:
        t.view(torch.bfloat16).normal_(generator=_gen(seed, role))
    else:
        t.view(torch.int32).random_(-2**31, 2**31 - 1, generator=_gen(seed, role))
    return t


def _kv(c, seed):
    kv = _device_bytes(c["layers"] * c["pages"] * _piece(c), seed, 1, c["elem"] == 2)
    sc = _device_bytes(c["layers"] * c["pages"] * 8, seed, 2, False) if c["scales"] else None
    return kv, sc


def _page_ids(c, seed, n):
    return np.random.default_rng([seed, 3]).permutation(c["pages"])[:n].astype(np.int32)


def _host_slots(seed, n):
    """n slots in the tier's order of use: shuffled, as after evictions."""
    return np.random.default_rng([seed, 4]).permutation(n).astype(np.int64)


def _tier_image(c, seed, n):
    """What the first n host slots hold (device copy)."""
    return _device_bytes(n * _slot_bytes(c, c["chunk"]), seed, 5, c["elem"] == 2 and not c["scales"])


def _tier_slots(c):
    return c.get("store", 0) + c.get("load", 0) if c["kind"] != "restore" else c["resident"] + 1


def _tokens(seed, n):
    return np.random.default_rng([seed, 6]).integers(0, VOCAB, n, dtype=np.int32)


def _hash_inputs(c, seed):
    r = np.random.default_rng([seed, 7])
    n = c["seqs"]
    # a batch's lengths belong to the case, their order to the seed
    lens = r.permutation(np.random.default_rng(n).integers(c["shortest"], c["longest"] + 1, n))
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    par = r.integers(0, 256, (n, 32), dtype=np.uint8) if c["parents"] else None
    return _tokens(seed, int(offs[-1])), offs, par


# Streams as an engine keeps them: created once, after the default stream's
# first use.
_streams = []


def _two_streams():
    if not _streams:
        torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        _streams.extend(torch.cuda.Stream() for _ in range(2))
    return _streams


class _State:
    """What a user's program has in hand; the tier goes with it."""


def _make_cache(s, c, seed):
    s.kv, s.sc = _kv(c, seed)
    s.cache = api.Cache(s.kv, c["pages"], c["layers"], c["page_tokens"], c["heads"], c["head_dim"],
                        c["elem"], scales=s.sc)


def _make_tier(s, c):
    s.tier = api.Tier(s.cache, _tier_slots(c) * _slot_bytes(c, c["chunk"]), chunk_pages=c["chunk"])


def _fill_tier(s, image):
    torch.from_numpy(s.tier.host_view().reshape(-1)).copy_(image)


def prepare(case, seed):
    c = case
    s = _State()
    s.c = c
    if c["kind"] == "hash":
        s.tok, s.offs, s.par = _hash_inputs(c, seed)
        if c["entry"] == "host":
            return s
        n = len(s.offs) - 1
        total = int((np.diff(s.offs) // c["block"]).sum())
        s.d_tok = torch.from_numpy(s.tok).cuda()
        s.d_par = None if s.par is None else torch.from_numpy(s.par).cuda()
        s.d_keys = torch.zeros((max(total, 1), 32), dtype=torch.uint8, device="cuda")
        if c["entry"] != "device":
            s.d_offs = torch.from_numpy(s.offs).cuda()
            s.d_koff = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        return s
    _make_cache(s, c, seed)
    if c["kind"] == "hbm":
        ids = _page_ids(c, seed, 2 * c["moved"])
        s.src, s.dst = ids[:c["moved"]], ids[c["moved"]:]
        s.buf = torch.zeros(c["moved"] * s.cache.slot_bytes, dtype=torch.uint8, device="cuda")
        return s
    _make_tier(s, c)
    n = _tier_slots(c)
    if c["kind"] == "restore":
        s.prompt = _tokens(seed, c["tokens"])
        s.block = c["chunk"] * c["page_tokens"]
        s.ends = np.array([0, c["tokens"]], np.int64)
        s.tier.host_view()[:] = 0
        # an earlier turn stored the prefix from the pages it was computed in
        keys, _ = api.hash_blocks(s.prompt, s.ends, s.block)
        got, slots = s.tier.alloc(keys[:c["resident"]])
        assert got == c["resident"]
        s.tier.store(s.cache, _page_ids(c, seed, got * c["chunk"]), slots)
        torch.cuda.synchronize()
        s.tier.unpin(slots)
        s.free = np.random.default_rng([seed, 8]).permutation(c["pages"]).astype(np.int32)
        # the pages' contents change hands before the restore
        s.kv.copy_(_device_bytes(s.kv.numel(), seed, 9, c["elem"] == 2))
        if s.sc is not None:
            s.sc.copy_(_device_bytes(s.sc.numel(), seed, 10, False))
        return s
    _fill_tier(s, _tier_image(c, seed, n))
    slots = _host_slots(seed, n)
    st, ld, ck = c.get("store", 0), c["load"], c["chunk"]
    ids = _page_ids(c, seed, (st + ld) * ck)
    s.store_ids, s.load_ids = ids[:st * ck], ids[st * ck:]
    s.store_slots, s.load_slots = slots[:st], slots[st:]
    if c["kind"] == "layered":
        s.events = [torch.cuda.Event() for _ in range(c["layers"])]
        s.sums = torch.zeros((c["layers"], ld), dtype=torch.int64, device="cuda")
    s.streams = _two_streams()
    return s


# ------------------------------------------------------------------ passes

def _images(s):
    out = {"kv": s.kv.view(torch.int64)}
    if s.sc is not None:
        out["scales"] = s.sc.view(torch.int64)
    return out


def run(state):
    s, c = state, state.c
    if c["kind"] == "hash":
        if c["entry"] == "host":
            return api.hash_blocks(s.tok, s.offs, c["block"], parents=s.par)
        if c["entry"] == "device":
            koffs = api.hash_blocks_device(s.d_tok, s.offs, c["block"], s.d_keys, s.d_par)
            return s.d_keys, koffs
        api.hash_blocks_device_offsets(s.d_tok, s.d_offs, c["block"], s.d_keys, s.d_koff, s.d_par,
                                       noalloc=c["entry"] == "noalloc")
        return s.d_keys, s.d_koff
    if c["kind"] == "hbm":
        s.cache.gather(s.src, s.buf)
        s.cache.scatter(s.buf, s.dst)
        return dict(_images(s), buffer=s.buf.view(torch.int64))
    if c["kind"] == "restore":
        keys, _ = api.hash_blocks(s.prompt, s.ends, s.block)
        hit, slots = s.tier.lookup(keys)
        s.tier.load(s.cache, slots, s.free[:hit * c["chunk"]])
        s.tier.unpin(slots)
        return dict(_images(s), keys=keys, hit=hit)
    if c["kind"] == "layered":
        copy, consumer = s.streams
        s.tier.load_layered(s.cache, s.load_slots, s.load_ids, copy, s.events)
        for layer, event in enumerate(s.events):
            consumer.wait_event(event)
            s.cache.layer_checksum(layer, s.load_ids, s.sums[layer], stream=consumer)
        return dict(_images(s), sums=s.sums)
    a, b = s.streams if c["two"] else (None, None)
    s.tier.store(s.cache, s.store_ids, s.store_slots, stream=a)
    s.tier.load(s.cache, s.load_slots, s.load_ids, stream=b)
    slots = torch.from_numpy(s.tier.host_view().view(np.int64))
    slots.tier = s.tier  # the view is the tier's own pinned memory
    return dict(_images(s), tier=slots)


def work(case):
    c = case
    if c["kind"] == "hash":
        mean = (c["shortest"] + c["longest"]) / 2
        keys = c["seqs"] * max(0.0, mean / c["block"] - (0.5 if c["shortest"] < c["longest"] else 0))
        # 32-bit operations of one FIPS 180-4 compression: 64 rounds of 24
        # (rotations, logic, additions) and 48 schedule words of 13
        flops = keys * (c["block"] // 16 + 1) * (64 * 24 + 48 * 13)
        return {"bytes": keys * (4 * c["block"] + 32) + c["seqs"] * (48 if c["parents"] else 16),
                "flops": flops}
    if c["kind"] == "hbm":
        return {"bytes": 4 * c["moved"] * _slot_bytes(c, 1), "flops": 0}
    slots = c["resident"] if c["kind"] == "restore" else c.get("store", 0) + c["load"]
    moved = 2 * slots * _slot_bytes(c, c["chunk"])  # read once, written once
    if c["kind"] == "restore":
        keys = c["tokens"] // (c["chunk"] * c["page_tokens"])
        moved += 4 * c["tokens"] + 32 * keys
    if c["kind"] == "layered":  # the consumer reads every layer once
        moved += c["load"] * (c["layers"] * _piece(c) + 8 * c["layers"])
    return {"bytes": moved, "flops": 0}


def tolerance(case):
    return "exact"  # keys and copied bytes


# --------------------------------------------------- the same without the library

def _plain_keys(tok, offs, block, par):
    out, koff = [], np.zeros(len(offs), np.int64)
    raw = tok.astype("<i4").tobytes()
    for i in range(len(offs) - 1):
        key = bytes(32) if par is None else par[i].tobytes()
        n = int(offs[i + 1] - offs[i]) // block
        at = 4 * int(offs[i])
        for _ in range(n):
            key = hashlib.sha256(raw[at:at + 4 * block] + key).digest()
            out.append(key)
            at += 4 * block
        koff[i + 1] = koff[i] + n
    keys = np.frombuffer(b"".join(out), np.uint8).reshape(-1, 32) if out else \
        np.zeros((0, 32), np.uint8)
    return keys, koff


def _read_slots(c, kv, sc, ids, chunk):
    """uint8 [slots, slot bytes]: the slot images of the pages `ids`."""
    n, L = len(ids) // chunk, c["layers"]
    at = torch.as_tensor(ids.astype(np.int64), device="cuda")
    out = torch.zeros((n, _slot_bytes(c, chunk)), dtype=torch.uint8, device="cuda")
    data = kv.view(L, c["pages"], -1)[:, at].view(L, n, chunk, -1).permute(1, 0, 2, 3)
    out[:, :L * chunk * _piece(c)] = data.reshape(n, -1)
    if sc is not None:
        w = sc.view(L, c["pages"], 8)[:, at].view(L, n, chunk, 8).permute(1, 0, 2, 3)
        out[:, L * chunk * _piece(c):L * chunk * (_piece(c) + 8)] = w.reshape(n, -1)
    return out


def _write_pages(c, kv, sc, ids, images, chunk):
    n, L = len(ids) // chunk, c["layers"]
    at = torch.as_tensor(ids.astype(np.int64), device="cuda")
    end = L * chunk * _piece(c)
    data = images[:, :end].reshape(n, L, chunk, -1).permute(1, 0, 2, 3).reshape(L, n * chunk, -1)
    kv.view(L, c["pages"], -1)[:, at] = data
    if sc is not None:
        w = images[:, end:end + 8 * L * chunk].reshape(n, L, chunk, 8).permute(1, 0, 2, 3)
        sc.view(L, c["pages"], 8)[:, at] = w.reshape(L, n * chunk, 8)


def _plain_images(kv, sc):
    out = {"kv": kv.view(torch.int64)}
    if sc is not None:
        out["scales"] = sc.view(torch.int64)
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "hash":
        tok, offs, par = _hash_inputs(c, seed)
        keys, koff = _plain_keys(tok, offs, c["block"], par)
        if c["entry"] != "host" and len(keys) == 0:
            keys = np.zeros((1, 32), np.uint8)
        return keys, koff
    kv, sc = _kv(c, seed)
    if c["kind"] == "hbm":
        ids = _page_ids(c, seed, 2 * c["moved"])
        buf = _read_slots(c, kv, sc, ids[:c["moved"]], 1)
        _write_pages(c, kv, sc, ids[c["moved"]:], buf, 1)
        return dict(_plain_images(kv, sc), buffer=buf.view(-1).view(torch.int64))
    n, ck = _tier_slots(c), c["chunk"]
    if c["kind"] == "restore":
        tok = _tokens(seed, c["tokens"])
        keys, _ = _plain_keys(tok, [0, c["tokens"]], ck * c["page_tokens"], None)
        m = c["resident"]
        image = _read_slots(c, kv, sc, _page_ids(c, seed, m * ck), ck)
        kv.copy_(_device_bytes(kv.numel(), seed, 9, c["elem"] == 2))
        if sc is not None:
            sc.copy_(_device_bytes(sc.numel(), seed, 10, False))
        free = np.random.default_rng([seed, 8]).permutation(c["pages"]).astype(np.int32)
        _write_pages(c, kv, sc, free[:m * ck], image, ck)
        return dict(_plain_images(kv, sc), keys=keys, hit=m)
    image = _tier_image(c, seed, n).view(n, -1)
    slots = _host_slots(seed, n)
    st, ld = c.get("store", 0), c["load"]
    ids = _page_ids(c, seed, (st + ld) * ck)
    to = torch.as_tensor(slots, device="cuda")
    if st:
        image[to[:st]] = _read_slots(c, kv, sc, ids[:st * ck], ck)
    _write_pages(c, kv, sc, ids[st * ck:], image[to[st:]], ck)
    out = _plain_images(kv, sc)
    if c["kind"] != "layered":
        return dict(out, tier=image.view(torch.int64))
    at = torch.as_tensor(ids.astype(np.int64), device="cuda")
    words = kv.view(torch.int64).view(c["layers"], c["pages"], -1)[:, at]
    while words.shape[-1] > 1:  # XOR of the 64-bit words
        half = words.shape[-1] // 2
        odd = words[..., 2 * half:]
        words = words[..., :half] ^ words[..., half:2 * half]
        if odd.shape[-1]:
            words[..., :1] ^= odd
    sums = words[..., 0]
    if sc is not None:
        sums = sums ^ sc.view(torch.int64).view(c["layers"], c["pages"])[:, at]
    return dict(out, sums=sums.contiguous())
