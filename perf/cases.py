"""What a user of this framework has it do, as cases that can be timed and compared.

Every case goes through the public entry points of `paper_2410_07590_amd.binding`, in the order in which a serving or
an ingest program calls them, and returns everything that such a program would go on with: attention outputs, the
key/value cache rows that were formed, rotated keys, projected activations.  The sizes are those of the repository's
configurations (`synth.CONFIGS`), tests and benchmark; `draw` gives other sizes of the same ranges.

A case is a dict of plain values.  Its sizes (chunk lengths, query lengths, which chunks a request retrieves) follow
from the case alone, so `work` knows them; the seed decides the contents of the tensors and the order in which a
request's chunks were retrieved.

kind      "request"   one request: gather plan, cache formation with the query tokens' own rows, query prefill
          "batch"     several requests: batched cache formation, batched append, batched query prefill
          "gather"    one request whose attention reads the chunks in the store (no cache of the documents is formed)
          "decode"    one new token per request: append, then attention over everything before it
          "offline"   ingest: packed chunks, each attending only to itself; gives the keys the store keeps
          "sequence"  documents and query in one pass with the masks and position ids of inference
          "project"   query/key/value and output projections of the query tokens, layer after layer
shape     name in SHAPES, layout: pairs of the rotation ("interleaved" as Eq. 3 prints it, "half" as released weights)
chunks    chunks per request (or packed, or in front of the tail); lo, hi: their lengths, both ends included
store     chunks in the store; raw: the store keeps keys that were not rotated
mode      "reordered", "composite" or, for a batch, "mixed" (drawn per request)
q_lo,q_hi query tokens per request
mix       seed of the sizes
"""
import numpy as np
import torch

from paper_2410_07590_amd import binding as B
from paper_2410_07590_amd import synth

SHAPES = {"tiny": synth.CONFIGS[1].shape, "qwen2-7b": synth.QWEN2_7B, "llama3-8b": synth.LLAMA3_8B}
MODES = {"composite": B.TR_POS_COMPOSITE, "reordered": B.TR_POS_REORDERED}
LAYOUTS = {"interleaved": B.TR_ROPE_INTERLEAVED, "half": B.TR_ROPE_HALF}


def listed():
    return [
        # the smallest call: two short chunks and a short question, fp32; nothing but launches and host work
        dict(name="request-tiny-f32", kind="request", shape="tiny", layout="interleaved", raw=False, mode="reordered",
             store=2, chunks=2, lo=64, hi=64, q_lo=16, q_hi=16, mix=1),
        # one question over eight retrieved chunks: the ordinary interactive request
        dict(name="request-8x512-q64", kind="request", shape="qwen2-7b", layout="interleaved", raw=False, mode="reordered",
             store=256, chunks=8, lo=512, hi=512, q_lo=64, q_hi=64, mix=2),
        # a long context with a long question: the benchmark's workload
        dict(name="request-32x1024-q256", kind="request", shape="llama3-8b", layout="interleaved", raw=False, mode="reordered",
             store=32, chunks=32, lo=1024, hi=1024, q_lo=256, q_hi=256, mix=4),
        # the paper's own store (keys kept before rotation), chunks and question of odd lengths, released-weight layout
        dict(name="request-raw-ragged", kind="request", shape="qwen2-7b", layout="half", raw=True, mode="reordered",
             store=64, chunks=13, lo=100, hi=900, q_lo=37, q_hi=37, mix=6),
        # a question answered straight from the store, without keeping the assembled document rows
        dict(name="gather-ragged-q21", kind="gather", shape="llama3-8b", layout="half", mode="reordered",
             store=64, chunks=9, lo=200, hi=700, q_lo=21, q_hi=21, mix=7),
        # a serving batch: sixteen requests of ten popular chunks each, both position schemes
        dict(name="batch-16x10-mixed", kind="batch", shape="qwen2-7b", layout="interleaved", mode="mixed",
             store=1000, chunks=10, lo=256, hi=1024, n_req=16, q_lo=32, q_hi=128, mix=3),
        # a batch of short questions over long contexts (multi-document question answering)
        dict(name="batch-16x12-short", kind="batch", shape="qwen2-7b", layout="half", mode="composite",
             store=200, chunks=12, lo=1024, hi=1024, n_req=16, q_lo=16, q_hi=16, mix=8),
        # one answer token for a full batch of requests
        dict(name="decode-64x4096", kind="decode", shape="qwen2-7b", layout="interleaved", n_req=64, lo=4096, hi=4096, mix=9),
        # one answer token for the few requests of a quiet hour, each with its own length
        dict(name="decode-5-ragged", kind="decode", shape="llama3-8b", layout="half", n_req=5, lo=300, hi=3000, mix=10),
        # ingest of a document collection
        dict(name="offline-64x512", kind="offline", shape="llama3-8b", layout="interleaved", chunks=64, lo=512, hi=512, mix=5),
        # the whole context and its question prefilled in one pass
        dict(name="sequence-32x1024-q256", kind="sequence", shape="llama3-8b", layout="interleaved", mode="reordered",
             chunks=32, lo=1024, hi=1024, q_lo=256, q_hi=256, mix=11),
        # the projections around the attention for a question of 64 tokens, ten layers deep
        dict(name="project-10-layers-q64", kind="project", shape="qwen2-7b", layers=10, q_lo=64, q_hi=64, mix=12),
    ]


# ---- drawn cases ------------------------------------------------------------------------------------------------------


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """One more case of the listed ranges: context up to 32 k rows, up to 256 query tokens, batches up to 64 requests."""
    kind = rng.choice(["request", "request", "gather", "batch", "decode", "decode", "offline", "sequence", "project", "tiny"])
    c = dict(kind=kind, shape=rng.choice(["qwen2-7b", "llama3-8b"]), mix=rng.randrange(1, 1 << 30))
    if kind == "tiny":
        c.update(kind="request", shape="tiny", layout="interleaved", raw=rng.random() < 0.25, mode=rng.choice(["reordered", "composite"]),
                 store=8, chunks=rng.randint(1, 8), lo=rng.randint(16, 64), hi=rng.randint(64, 128))
        c["q_lo"] = c["q_hi"] = _log(rng, 1, 64)
        return c
    if kind == "project":
        c["layers"] = rng.randint(2, 10)
        c["q_lo"] = c["q_hi"] = _log(rng, 1, 128)
        return c
    c["layout"] = rng.choice(["interleaved", "half"])
    if kind == "decode":
        c["n_req"] = _log(rng, 1, 64)
        top = min(8192, 64 * 4096 // c["n_req"])
        c["lo"] = _log(rng, 128, top)
        c["hi"] = rng.randint(c["lo"], top)
        return c
    c["lo"] = _log(rng, 16 if kind == "offline" else 64, 1024)
    c["hi"] = c["lo"] if rng.random() < 0.3 else rng.randint(c["lo"], 1024)
    if kind == "offline":
        c["chunks"] = _log(rng, 1, min(256, 32768 // c["hi"]))
        return c
    c["mode"] = rng.choice(["reordered", "composite"])
    c["chunks"] = _log(rng, 1, 32)
    c["q_lo"] = c["q_hi"] = _log(rng, 1, 128 if kind == "gather" else 256)
    if kind == "request":
        c["raw"] = rng.random() < 0.25
    if kind == "batch":
        c["mode"] = rng.choice(["reordered", "composite", "mixed"])
        c["n_req"] = rng.randint(2, 16)
        c["chunks"] = rng.randint(2, 12)
        c["q_lo"] = _log(rng, 1, 64)
        c["q_hi"] = rng.randint(c["q_lo"], 128)
    if kind != "sequence":
        c["store"] = max(c["chunks"], rng.choice([40, 100, 200]))
    return c


# ---- sizes: functions of the case alone -------------------------------------------------------------------------------


def _shape(case):
    return SHAPES[case["shape"]]


def _sizes(case):
    """Lengths, retrieved ids, query lengths and position schemes of the case."""
    rng = np.random.Generator(np.random.PCG64([20241007, case["mix"]]))
    kind = case["kind"]
    s = {}
    if kind == "project":
        s["n_q"] = np.array([case["q_lo"]])
    elif kind == "decode":
        s["kv_len"] = rng.integers(case["lo"], case["hi"] + 1, case["n_req"])
    elif kind in ("offline", "sequence"):
        s["lens"] = rng.integers(case["lo"], case["hi"] + 1, case["chunks"])
        s["n_q"] = np.array([case.get("q_lo", 0)])
    else:
        n_req = case.get("n_req", 1)
        s["lens"] = rng.integers(case["lo"], case["hi"] + 1, case["store"])
        # popularity of the chunks: bounded Zipf for a batch over a large store, uniform otherwise; distinct in a request
        w = np.arange(1, case["store"] + 1) ** (-1.1 if kind == "batch" else 0.0)
        w = rng.permutation(w / w.sum())
        s["ids"] = [rng.choice(case["store"], case["chunks"], replace=False, p=w) for _ in range(n_req)]
        s["n_q"] = rng.integers(case["q_lo"], case["q_hi"] + 1, n_req)
        s["modes"] = [MODES[case["mode"]] if case["mode"] != "mixed" else int(rng.integers(2)) for _ in range(n_req)]
        s["n_doc"] = np.array([int(s["lens"][i].sum()) for i in s["ids"]])
    return s


# ---- inputs ---------------------------------------------------------------------------------------------------------------


def _starts(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


def prepare(case, seed):
    """The store, its handle, the request's tensors, cache, outputs and workspace.  Values are N(0, 1), as synth draws them."""
    sh, z = _shape(case), _sizes(case)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    order = np.random.Generator(np.random.PCG64([7, int(seed)]))
    dt, hq, hk, d = sh.torch_dtype, sh.n_q_heads, sh.n_kv_heads, sh.head_dim

    def normal(*size):
        return torch.randn(size, generator=g, device="cuda", dtype=dt)

    def empty(*size):
        return torch.zeros(size, device="cuda", dtype=dt)

    def ints(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()

    kind = case["kind"]
    if kind == "project":
        m, width, kv = int(z["n_q"][0]), hq * d, hk * d
        layers = []
        for _ in range(case["layers"]):
            w = [normal(n, width) / width ** 0.5 for n in (width, kv, kv, width)]
            layers.append(dict(x=normal(m, width), a=normal(m, width), qkv=w[:3], o=w[3],
                               y=[empty(m, n) for n in (width, kv, kv)], z=empty(m, width)))
        need = max(B.tr_linear_workspace_size(m, [width, kv, kv], width), B.tr_linear_workspace_size(m, [width], width))
        return dict(kind=kind, layers=layers, ws=B.workspace(need))

    gs = B.make_shape(hq, hk, d, sh.dtype, sh.rope_base, LAYOUTS[case["layout"]])
    st = dict(kind=kind, shape=gs)
    if kind == "decode":
        start = _starts(z["kv_len"])
        rows, n = int(start[-1]), case["n_req"]
        st.update(start=start, cu=np.arange(n + 1, dtype=np.int32), cache_k=normal(rows, hk, d), cache_v=normal(rows, hk, d),
                  k=normal(n, hk, d), v=normal(n, hk, d), q=normal(n, hq, d), out=empty(n, hq, d), pos=ints(z["kv_len"] - 1),
                  ws=B.workspace(B.tr_decode_attn_workspace_size(gs, start)))
        return st
    if kind == "offline":
        cu = _starts(z["lens"])
        t, longest = int(cu[-1]), int(z["lens"].max())
        st.update(q=normal(t, hq, d), k=normal(t, hk, d), v=normal(t, hk, d), out=empty(t, hq, d), k_rot=empty(t, hk, d), cu=ints(cu),
                  n=len(z["lens"]), longest=longest, ws=B.workspace(B.tr_chunk_prefill_attn_workspace_size(gs, t, longest)))
        return st
    if kind == "sequence":
        seg, pos = B.tr_sequence_plan(z["lens"].astype(np.int32), int(z["n_q"][0]), MODES[case["mode"]])
        t = len(seg)
        st.update(q=normal(t, hq, d), k=normal(t, hk, d), v=normal(t, hk, d), out=empty(t, hq, d), k_rot=empty(t, hk, d),
                  seg_host=seg, seg=ints(seg), pos=ints(pos),
                  ws=B.workspace(B.tr_sequence_prefill_attn_workspace_size(gs, seg, t)))
        return st

    row_start = _starts(z["lens"])
    rows = int(row_start[-1])
    store = B.Store(gs, normal(rows, hk, d), normal(rows, hk, d), row_start)
    ids = [order.permutation(i).astype(np.int32) for i in z["ids"]]
    n_q, n_doc = z["n_q"], z["n_doc"]
    total_q, cache_rows = int(n_q.sum()), int((n_doc + n_q).sum())
    q_pos = np.concatenate([synth.query_start(m, z["lens"][i]) + np.arange(n) for m, i, n in zip(z["modes"], ids, n_q)])
    st.update(store=store, q=normal(total_q, hq, d), k=normal(total_q, hk, d), v=normal(total_q, hk, d), q_pos=ints(q_pos),
              out=empty(total_q, hq, d), cache_k=empty(cache_rows, hk, d), cache_v=empty(cache_rows, hk, d))
    if kind == "batch":
        start, cu_q = _starts(n_doc + n_q), _starts(n_q).astype(np.int32)
        st.update(ids=np.concatenate(ids), cu_chunks=(np.arange(len(ids) + 1) * case["chunks"]).astype(np.int32), modes=z["modes"], start=start,
                  cu_q=cu_q, ws=B.workspace(B.tr_prefill_attn_batched_workspace_size(gs, cu_q, start)))
        return st
    st.update(ids=ids[0], mode=z["modes"][0], raw=case.get("raw", False), n_doc=int(n_doc[0]), kv_len=cache_rows)
    if kind == "gather":
        offsets, _ = B.tr_plan(store, ids[0], st["mode"], want_pos_ids=False)
        need = B.tr_prefill_attn_gather_workspace_size(store, ids[0], offsets, st["mode"], total_q)
    else:
        need = B.tr_prefill_attn_workspace_size(gs, total_q, cache_rows)
    st["ws"] = B.workspace(need)
    return st


# ---- one pass --------------------------------------------------------------------------------------------------------------


def run(st):
    kind = st["kind"]
    if kind == "project":
        for layer in st["layers"]:
            B.tr_linear(layer["x"], layer["qkv"], layer["y"], st["ws"])
            B.tr_linear(layer["a"], layer["o"], layer["z"], st["ws"])
        return [(layer["y"], layer["z"]) for layer in st["layers"]]
    gs, out = st["shape"], st["out"]
    if kind == "decode":
        B.tr_kv_append_batched(gs, st["k"], st["v"], st["pos"], st["cu"], st["start"], st["cache_k"], st["cache_v"])
        B.tr_decode_attn(gs, st["q"], st["cache_k"], st["cache_v"], st["pos"], st["start"], out, st["ws"])
        return out, st["cache_k"], st["cache_v"]
    if kind == "offline":
        B.tr_chunk_prefill_attn(gs, st["q"], st["k"], st["v"], st["cu"], st["n"], st["longest"], out, st["k_rot"], st["ws"])
        return out, st["k_rot"]
    if kind == "sequence":
        B.tr_sequence_prefill_attn(gs, st["q"], st["k"], st["v"], st["seg"], st["pos"], out, st["k_rot"],
                                   seg_start_host=st["seg_host"], workspace=st["ws"])
        return out, st["k_rot"]
    store, ck, cv = st["store"], st["cache_k"], st["cache_v"]
    if kind == "batch":
        B.tr_kv_assemble_batched(store, st["ids"], st["cu_chunks"], st["modes"], st["start"], ck, cv)
        B.tr_kv_append_batched(gs, st["k"], st["v"], st["q_pos"], st["cu_q"], st["start"], ck, cv)
        B.tr_prefill_attn_batched(gs, st["q"], ck, cv, st["q_pos"], st["cu_q"], st["start"], out, st["ws"])
        return out, ck, cv
    offsets, _ = B.tr_plan(store, st["ids"], st["mode"], want_pos_ids=False)
    if kind == "gather":
        n_doc = st["n_doc"]
        B.tr_kv_append(gs, st["k"], st["v"], st["q_pos"], ck, cv, n_doc)
        B.tr_prefill_attn_gather(store, st["ids"], offsets, st["mode"], st["q"], ck, cv, st["q_pos"], out, st["ws"])
        return out, ck[n_doc:], cv[n_doc:]
    if st["raw"]:
        B.tr_kv_assemble_raw(store, st["ids"], offsets, st["mode"], ck, cv)
        B.tr_kv_append(gs, st["k"], st["v"], st["q_pos"], ck, cv, st["n_doc"])
    else:
        B.tr_kv_assemble_append(store, st["ids"], offsets, st["mode"], st["k"], st["v"], st["q_pos"], ck, cv)
    B.tr_prefill_attn(gs, st["q"], ck, cv, st["q_pos"], st["kv_len"], out, st["ws"])
    return out, ck, cv


# ---- what a pass cannot do without, and how far correct results may lie apart ------------------------------------------


def work(case):
    """Inputs read once, outputs written once; 4 * head_dim flops per query head and visible (query, key) pair."""
    sh, z = _shape(case), _sizes(case)
    e, hq, hk, d = sh.elem_bytes, sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    kind = case["kind"]
    if kind == "project":
        m, width, feats = int(z["n_q"][0]), hq * d, 2 * hq * d + 2 * hk * d
        return {"bytes": case["layers"] * e * (width * feats + 2 * m * width + m * feats), "flops": case["layers"] * 2.0 * m * width * feats}
    row_q, row_kv = hq * d * e, hk * d * e
    if kind == "decode":
        n, rows = case["n_req"], int(z["kv_len"].sum())
        return {"bytes": 2 * n * row_q + 2 * rows * row_kv + 2 * n * row_kv, "flops": 4.0 * hq * d * rows}
    if kind in ("offline", "sequence"):
        lens, tail = z["lens"].astype(np.int64), int(z["n_q"][0])
        docs = int(lens.sum())
        pairs = int((lens * (lens + 1) // 2).sum()) + tail * docs + tail * (tail + 1) // 2
        return {"bytes": (docs + tail) * (2 * row_q + 3 * row_kv), "flops": 4.0 * hq * d * pairs}
    n_q, n_doc = z["n_q"].astype(np.int64), z["n_doc"].astype(np.int64)
    pairs = int((n_q * n_doc + n_q * (n_q + 1) // 2).sum())
    moved = (2 if kind == "gather" else 4) * int(n_doc.sum()) + 4 * int(n_q.sum())
    return {"bytes": moved * row_kv + 2 * int(n_q.sum()) * row_q, "flops": 4.0 * hq * d * pairs}


def tolerance(case):
    """About four times the error against fp64 sums over the same inputs (attention: fp32 3.2e-7, bf16 2.6e-3 .. 3.0e-3 with a
    largest of 0.04; projections, against the rounded fp64 product: 4.6e-5, and one bf16 step where a sum lies on the edge)."""
    if _shape(case).dtype == "f32":
        return {"rel": 1.5e-6, "max": 1e-5}
    if case["kind"] == "project":
        return {"rel": 2e-4, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 0.16}
