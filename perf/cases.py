"""Timed workloads of the per-layer KV object path, through the entry points a serving engine calls.

A case is one call sequence on one batch of requests:
  restore   tutti_layer_restore for every layer: objects in a staging buffer -> paged pool blocks, with READ entries
  save      tutti_layer_save for every layer: paged pool blocks -> objects, with WRITE entries
  retrieve  tutti_retrieve_layer (several layers: the chained train and one tutti_complete_io): GPU files -> blocks
  store     tutti_store_layer (the same with blocks -> files)
  read      tutti_iocb_fill_direct + tutti_issue_io with READ contexts, per layer
  write     the same with WRITE contexts: deferred writes that are flushed
Everything a program keeps between calls (pool planes, rings, tables, extents, argument records) is made by
prepare(); run() is the calls alone.  All outputs are bytes and whole numbers.
"""
import weakref

import numpy as np
import torch

from paper_2605_03375_amd import binding as B
from paper_2605_03375_amd import placement
from paper_2605_03375_amd import workloads as W

DEV = "cuda:0"
GIB = 1 << 30
PLANE_BYTES = 2 * GIB          # buffer that holds the K planes (or the V planes) of all layers of a case
STAGE_ADDR, SGL_ADDR, SGL_ID = 1 << 40, 1 << 41, 3
FIRST_FILE = 1000

BASE = dict(op="restore", T=16, h=8, d=128, e=2, hnd=False, pool=65536, blocks=2048, reqs=1, lengths="long",
            table="random", layers=1, chunk=2 << 20, budget=0)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the smallest call an engine makes: one 512-token prefix of a tiny one-layer model (fp16, 2 heads x 64)
        _case("restore_tiny", h=2, d=64, pool=256, blocks=32),
        # a short prompt's 1K-token prefix: all 32 layers of the 8B shape, one call per layer
        _case("restore_1k_32layers", pool=1024, blocks=64, layers=32),
        # one layer of a 32K-token prefix, 8B shape: the headline size, both directions
        _case("restore_32k", ),
        _case("save_32k", op="save"),
        # a serving batch: 64 requests of Zipf-distributed lengths, one layer, 2.5 GiB of payload: the largest
        _case("restore_batch64", blocks=40719, reqs=64),
        # 70B shape, one layer of a 128K-token prefix whose blocks come from a churned free list
        _case("save_128k_churn", op="save", pool=38146, blocks=8192, table="churn"),
        # the same prefix as one rank of a tensor-parallel group of 8 holds it: one KV head, 4 KiB blocks
        _case("restore_128k_tp8", h=1, pool=38146, blocks=8192, table="churn"),
        # write-behind while decoding: 512 running sequences have each filled a few blocks (2 KV heads of a TP shard)
        _case("save_decode_512", op="save", h=2, blocks=1280, reqs=512, lengths="short", chunk=64 << 10),
        # a model whose block is no multiple of 4 KiB (5 heads x 80: 12,800 bytes), 24 requests
        _case("save_ragged_24", op="save", h=5, d=80, pool=49152, blocks=6007, reqs=24, chunk=256 << 10),
        # head-major pool of an 8-bit KV cache: a (token, head) row of 64 bytes
        _case("restore_hnd_fp8", h=16, d=64, e=1, hnd=True, blocks=4096, reqs=4),
        # the rings, 8B shape, one layer of a 32K-token prefix: GPU file -> blocks, completion included
        _case("retrieve_32k", op="retrieve"),
        # deferred writes flushed into a slack window with 32 compute units: 8 requests, 8K tokens in all
        _case("flush_writes_32cu", op="write", blocks=512, reqs=8, budget=32),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform over its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    ring = rng.random() < 0.4
    op = rng.choice(("retrieve", "store", "read", "write") if ring else ("restore", "save"))
    while True:
        T, h = rng.choice((16, 16, 32, 64)), rng.choice((1, 2, 4, 5, 8, 8, 10, 16))
        d, e = rng.choice((64, 80, 96, 128, 128, 192, 256)), rng.choice((1, 2, 2))
        block = T * h * d * e
        if block <= 128 << 10 and (not ring or block % 4096 == 0):
            break
    hnd = not ring and rng.random() < 0.3
    budget = rng.choice((8, 16, 32, 64)) if rng.random() < 0.2 else 0
    most = (48 << 20) if budget else (512 << 20)
    payload = _log(rng, 128 << 10, most)
    blocks = max(1, payload // (2 * block)) + rng.randrange(3)
    reqs = min(blocks, _log(rng, 1, 64 if ring else 1024))
    layers = rng.choice((2, 5, 16)) if payload < (4 << 20) else 1
    room = min(65536, PLANE_BYTES // (block * layers))
    pool = max(blocks, min(room, int(blocks * (1.2 + 8 * rng.random()))))
    table = "churn" if 4096 <= pool and blocks * 8 <= pool * 7 and rng.random() < 0.3 else "random"
    return dict(BASE, op=op, T=T, h=h, d=d, e=e, hnd=hnd, pool=pool, blocks=blocks, reqs=reqs,
                lengths=rng.choice(("long", "short")), table=table, layers=layers,
                chunk=rng.choice((128 << 10, 512 << 10, 2 << 20)), budget=budget)


def _geometry(case):
    block = case["T"] * case["h"] * case["d"] * case["e"]
    return block, 4096


def _lengths(case):
    """Blocks per request, the same for every seed (they decide the outputs' sizes): they add up to case["blocks"],
    every request has at least one."""
    n, total = case["reqs"], case["blocks"]
    rng = np.random.default_rng(W.seed_for(3))
    if case["lengths"] == "long":    # 1K..64K-token contexts, Zipf(1.1), of which a part was found
        ranks = np.arange(1, 65, dtype=np.float64)
        p = ranks ** -1.1
        w = rng.choice(ranks, size=n, p=p / p.sum()) * rng.uniform(0.3, 1.0, size=n)
    else:                            # a few blocks each
        w = rng.integers(1, 5, size=n).astype(np.float64)
    got = 1 + np.floor(w / w.sum() * (total - n)).astype(np.int64)
    got[np.argsort(-w, kind="stable")[:total - int(got.sum())]] += 1
    return got.astype(np.uint32)


class _Planes:
    """Buffers for pool planes, in pairs that lie in different HBM regions, found once per process as an engine does
    it when its pool is created; a pair goes back to the list when nothing refers to its lease any more."""

    def __init__(self):
        self.pairs = None

    def _make(self):
        cands, spacers = [], []
        try:
            for _ in range(6):
                cands += [torch.empty(PLANE_BYTES, dtype=torch.uint8, device=DEV) for _ in range(4)]
                spacers.append(torch.empty(28 * GIB, dtype=torch.uint8, device=DEV))
        except torch.cuda.OutOfMemoryError:
            pass
        want = min(4, len(cands) // 2)
        for last in (False, False, True):    # the classification is a timing: once more if it told too few apart
            classes, _ = placement.classify_planes(cands, DEV)
            try:
                pairs = placement.choose_pairs(classes, want, strict=not last)
                break
            except ValueError:
                pass
        self.pairs = [(cands[i], cands[j]) for i, j in pairs]
        del cands, spacers
        torch.cuda.empty_cache()

    def lease(self, need):
        if self.pairs is None:
            self._make()
        if need > PLANE_BYTES or not self.pairs:
            return [torch.empty(need, dtype=torch.uint8, device=DEV) for _ in range(2)], None
        pair = self.pairs.pop()
        lease = _Lease()
        weakref.finalize(lease, self.pairs.append, pair)
        return [p[:need] for p in pair], lease


class _Lease:
    pass


_PLANES = _Planes()


class _State:
    pass


def _fill(t, gen):
    t.view(torch.int64).random_(generator=gen)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(DEV)


def prepare(case, seed):
    block, align = _geometry(case)
    layers, reqs, blocks = case["layers"], case["reqs"], case["blocks"]
    op, budget = case["op"], case["budget"]
    rng = np.random.default_rng([seed, blocks])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    n_blocks = _lengths(case)
    if case["table"] == "churn":
        table = W.fragmented_table(rng, case["pool"], blocks, rounds=2000)
    else:
        table = rng.permutation(case["pool"])[:blocks].astype(np.uint32)

    st = _State()
    plane = case["pool"] * block
    (k, v), lease = _PLANES.lease(plane * layers)
    _fill(k, gen)
    _fill(v, gen)
    k.lease = v.lease = lease      # whoever holds the tensors holds the buffers
    pools = [B.make_pool(k[l * plane:(l + 1) * plane], v[l * plane:(l + 1) * plane], num_blocks=case["pool"],
                         block_tokens=case["T"], num_kv_heads=case["h"], head_dim=case["d"], elt_bytes=case["e"],
                         pool_layout=B.LAYOUT_HND if case["hnd"] else B.LAYOUT_NHD) for l in range(layers)]
    cfg = B.make_cfg(align, case["chunk"], layers)
    d_n, d_table, d_file = _dev(n_blocks), _dev(table), _dev(FIRST_FILE + np.arange(reqs, dtype=np.uint32))
    extents = torch.zeros(4 * reqs, dtype=torch.int64, device=DEV)
    totals = torch.zeros(2, dtype=torch.int64, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    st.out = {"extents": extents, "totals": totals, "status": status}
    objects = (n_blocks.astype(np.int64) * block + align - 1) // align * align
    st.calls = []
    if op in ("restore", "save"):
        payload = int(2 * objects.sum())
        stage = torch.empty(layers * payload, dtype=torch.uint8, device=DEV)
        _fill(stage, gen)
        entries = int(2 * ((objects + case["chunk"] - 1) // case["chunk"]).sum())
        sqe = torch.zeros(layers * 64 * entries, dtype=torch.uint8, device=DEV)
        call = B.tutti_layer_restore if op == "restore" else B.tutti_layer_save
        for l in range(layers):
            st.calls.append((call, (pools[l], cfg, d_n, reqs, d_table, blocks, d_file, l,
                                    stage[l * payload:(l + 1) * payload], payload, STAGE_ADDR, SGL_ID, extents, totals,
                                    sqe[l * 64 * entries:(l + 1) * 64 * entries], entries, budget, status)))
        st.out["entries"] = sqe.view(torch.int64)
        moved = stage
    else:
        slots = -(-2 * blocks // B.IOCB_SLOTS)
        depth = layers * slots
        sq_bytes, cq_bytes = B.ring_bytes(depth)
        sq = torch.zeros(sq_bytes, dtype=torch.uint8, device=DEV)
        cq = torch.zeros(cq_bytes, dtype=torch.uint8, device=DEV)
        ring = B.make_ring(sq, cq, depth)
        B.tutti_ring_init(ring)
        stride = int(2 * layers * objects.max())
        files = torch.empty(reqs * stride, dtype=torch.uint8, device=DEV)
        _fill(files, gen)
        store = B.make_filestore(files, stride, FIRST_FILE, reqs)
        if op in ("read", "write"):
            opcode = B.OP_READ if op == "read" else B.OP_WRITE
            B.tutti_obj_layout(pools[0], cfg, d_n, reqs, extents, totals)
            for l in range(layers):
                sgl = torch.zeros(16 * 2 * case["pool"], dtype=torch.uint8, device=DEV)
                B.tutti_sgl_table_build(pools[l], pools[l].k_base, pools[l].v_base, SGL_ID, sgl, 2 * case["pool"])
                st.calls.append((B.tutti_iocb_fill_direct, (ring, l * slots, slots, pools[l], cfg, extents, reqs,
                                                            d_table, blocks, d_file, l, opcode, SGL_ADDR, SGL_ID,
                                                            status)))
                st.calls.append((B.tutti_issue_io, (ring, l * slots, slots, sgl, 2 * case["pool"], SGL_ADDR, store,
                                                    block, budget, status)))
        elif layers == 1:
            call = B.tutti_retrieve_layer if op == "retrieve" else B.tutti_store_layer
            st.calls.append((call, (ring, 0, slots, pools[0], cfg, d_n, reqs, d_table, blocks, d_file, 0, SGL_ADDR,
                                    SGL_ID, store, extents, totals, budget, status)))
        else:
            call = B.tutti_retrieve_layer_chained if op == "retrieve" else B.tutti_store_layer_chained
            for l in range(layers):
                done = ((l - 1) * slots, slots) if l else (0, 0)
                st.calls.append((call, (ring, l * slots, slots) + done +
                                 (pools[l], cfg, d_n, reqs, d_table, blocks, d_file, l, SGL_ADDR, SGL_ID, store,
                                  extents, totals, budget, status)))
            st.calls.append((B.tutti_complete_io, (ring, (layers - 1) * slots, slots)))
        st.out["sq"], st.out["cq"] = sq.view(torch.int64), cq.view(torch.int32)
        moved = files
    if op in ("restore", "retrieve", "read"):
        st.out["k"], st.out["v"] = k.view(torch.int64), v.view(torch.int64)
        st.out["k"].lease = st.out["v"].lease = lease
        st.keep = (moved,)
    else:
        st.out["objects"] = moved.view(torch.int64)
        st.keep = (k, v)
    return st


def run(state):
    for call, args in state.calls:
        call(*args)
    return state.out


def work(case):
    block, _ = _geometry(case)
    units = 2 * case["blocks"] * case["layers"]                       # (block, K or V) moves
    moved = 2 * units * block + 4 * case["blocks"] * case["layers"]   # read once, written once; the table
    if case["op"] in ("restore", "save"):
        entries = 64 * max(units * block // case["chunk"], 2 * case["reqs"] * case["layers"])
    else:
        entries = 64 * units                                          # one recorded context per move
        if case["op"] in ("read", "write"):
            entries += (64 + 16) * units                              # the I/O kernel reads them and the descriptors
    return {"bytes": moved + entries + 36 * case["reqs"] * case["layers"], "flops": 0}


def tolerance(case):
    return "exact"
