"""Performance cases of the NER + pseudonymize path.

Each case is one call (or one fixed chain of calls) through the package's
public entry points, on inputs that are already on the GPU, as a program that
serves or batch-processes scan records makes them.  The encoder runs with the
library's default tile choice.  Model shapes and record lengths are those of
the benchmark and the tests: "base" 12 layers h768, "large" 24 layers h1024,
"tiny" 2 layers h128, "modern" the ModernBERT-style encoder with h768;
lognormal record lengths around 180 tokens (scan records), 1100 tokens
(dataset-scale records, windowed at 512 every 448).  A case may cut the number
of layers: the layers are alike.

Paths
  forward     ner_forward of a packed batch: labels, logits, margins
  bucket      the same as a replay of a token-bucket HIP graph whose capacity
              is larger than the batch (what the server launches)
  windowed    ner_forward_windowed of records longer than one window
  layer       encoder_hidden: embedding and the first layers
  modern      the ModernBERT-style encoder's embedding and first layers
  decode      decode_spans of a labelled batch
  recognize   recognize_spans, merged with NER spans
  fields      field_spans of configured fields, then pseudonymize
  tail        decode_spans, recognize_spans, pseudonymize (all after the NER)

Lengths belong to the case (the seed only shuffles them), so a case's work is
the same for every seed; ids, weights and text come from the seed.
"""
from __future__ import annotations

import math
import random
from dataclasses import dataclass, replace

import numpy as np
import torch

from paper_2606_15650_amd import api


@dataclass(frozen=True)
class Shape:
    n_layers: int
    hidden: int
    n_heads: int
    ffn: int
    vocab: int
    n_labels: int
    max_pos: int = 512
    ln_eps: float = 1e-5


@dataclass(frozen=True)
class ModernShape:
    n_layers: int
    hidden: int
    n_heads: int
    intermediate: int
    vocab: int
    n_labels: int
    max_pos: int = 8192
    ln_eps: float = 1e-5
    local_window: int = 128
    global_every: int = 3
    theta_global: float = 160000.0
    theta_local: float = 10000.0


SHAPES = {
    "tiny": Shape(2, 128, 2, 512, 8192, 9),
    "base": Shape(12, 768, 12, 3072, 30522, 17),
    "large": Shape(24, 1024, 16, 4096, 30522, 17),
    "modern": ModernShape(22, 768, 12, 1152, 50368, 17),
}
TYPES = ["IP_ADDRESS", "HOSTNAME", "CVE_ID", "EMAIL_ADDRESS", "PORT", "URL", "MAC_ADDRESS", "HASH"]
FIELDS = {"Host": 1, "IP": 1, "Target": 1, "Hostname": 2, "FQDN": 2, "DNS Name": 2, "CVE": 3, "Reference": 3,
          "Contact": 4, "Owner": 4, "Port": 5, "See Also": 6, "MAC": 7, "Fingerprint": 8, "Hash": 8}
# static power-of-two scales of an FP8 layer's four GEMM inputs
FP8_SCALES = [2.0 ** -6, 2.0 ** -9, 2.0 ** -6, 2.0 ** -6]
ENCODER_PATHS = ("forward", "bucket", "windowed", "layer", "modern")
WINDOW, STRIDE = 512, 448
SLUG = 10
DEV = "cuda:0"


# ------------------------------------------------------------------- cases --
def _enc(path, size, precision, layers, records, center, spread, longest):
    """center, spread: median length (tokens) and sigma of the lognormal record lengths."""
    return {"path": path, "size": size, "precision": precision, "layers": layers, "records": records,
            "center": center, "spread": spread, "longest": longest}


def _text(path, records, kbytes):
    return {"path": path, "records": records, "kbytes": kbytes}


def listed():
    return [
        # one record typed in or arriving alone: the smallest call, latency and launches
        {"name": "forward_record", **_enc("forward", "base", "bf16", 12, 1, 137, 0.0, 512)},
        # one serving request of about 100 records, the mean of the serving benchmark
        {"name": "forward_request", **_enc("forward", "base", "bf16", 12, 100, 181, 0.6, 512)},
        # a small request replayed from the server's graph of a larger bucket
        {"name": "bucket_small", **_enc("bucket", "base", "bf16", 4, 11, 181, 0.6, 512)},
        # one encoder layer of the benchmark's batch of 4096 records, the bulk path
        {"name": "layer_batch_bf16", **_enc("layer", "base", "bf16", 1, 4096, 181, 0.6, 512)},
        # one layer of the large encoder in FP8
        {"name": "layer_batch_fp8", **_enc("layer", "large", "fp8", 1, 1500, 245, 0.7, 512)},
        # the plain FP32 path on a request
        {"name": "layer_request_fp32", **_enc("layer", "base", "fp32", 1, 100, 181, 0.6, 512)},
        # the ModernBERT-style encoder: one global and two local layers
        {"name": "modern_batch", **_enc("modern", "modern", "bf16", 3, 600, 181, 0.6, 512)},
        # dataset-scale records cut into overlapping windows
        {"name": "windowed_stream", **_enc("windowed", "base", "bf16", 1, 101, 1141, 0.6, 16384)},
        # span decoding of the bulk batch
        {"name": "decode_batch", **_text("decode", 4096, 4890)},
        # recognizers merged with the NER spans of the bulk batch
        {"name": "recognize_batch", **_text("recognize", 4096, 4890)},
        # everything after the NER for one request
        {"name": "tail_request", **_text("tail", 100, 120)},
        # configured fields of a dataset stream, no NER
        {"name": "fields_stream", **_text("fields", 16384, 128000)},
    ]


def _between(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    path = rng.choice(["forward", "forward", "bucket", "windowed", "layer", "layer", "modern", "decode", "recognize",
                       "fields", "tail"])
    if path == "decode" or path == "recognize":
        n = _between(rng, 1, 4096)
        return _text(path, n, max(1, n * _between(rng, 300, 2400) // 2000))
    if path == "tail":
        n = _between(rng, 1, 2000)
        return _text(path, n, max(1, n * _between(rng, 300, 2400) // 2000))
    if path == "fields":
        n = _between(rng, 1, 16384)
        return _text(path, n, max(1, n * _between(rng, 300, 12000) // 2000))
    if path == "windowed":
        return _enc(path, "base", rng.choice(["bf16", "bf16", "fp32"]), 1, _between(rng, 1, 60),
                    _between(rng, 300, 1500), 0.6, 16384)
    if path == "modern":
        return _enc(path, "modern", "bf16", rng.choice([1, 2, 3]), _between(rng, 1, 600),
                    _between(rng, 40, 220), 0.6, rng.choice([512, 1500]))
    if path == "layer":
        precision = rng.choice(["bf16", "bf16", "fp8", "fp32"])
        size = rng.choice(["tiny", "base", "base", "large"])
        return _enc(path, size, precision, 1, _between(rng, 1, 300 if precision == "fp32" else 1400),
                    _between(rng, 30, 260), rng.choice([0.0, 0.3, 0.6]), 512)
    return _enc(path, "base", "bf16", rng.choice([2, 4, 12]), _between(rng, 1, 120), _between(rng, 20, 200),
                rng.choice([0.0, 0.6]), 512)


# ----------------------------------------------------------------- helpers --
def _lengths(case) -> np.ndarray:
    rng = np.random.default_rng(case["records"] * 1009 + case["center"])
    x = np.exp(rng.normal(math.log(case["center"]), case["spread"], case["records"]))
    lo = 1 if case["center"] < 40 else 16
    return np.clip(np.round(x), lo, case["longest"]).astype(np.int64)


def _shape(case):
    return replace(SHAPES[case["size"]], n_layers=case["layers"])


def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + salt)


def _specs(cfg):
    """Weight tensors in the order the library takes them."""
    h, C = cfg.hidden, cfg.n_labels
    if isinstance(cfg, ModernShape):
        I = cfg.intermediate
        out = [("tok", (cfg.vocab, h)), ("eg", (h,))]
        for l in range(cfg.n_layers):
            out += ([(f"{l}.ag", (h,))] if l else []) + [
                (f"{l}.wqkv", (h, 3 * h)), (f"{l}.wo", (h, h)), (f"{l}.mg", (h,)), (f"{l}.wi", (h, 2 * I)),
                (f"{l}.wo2", (I, h))]
        return out + [("fg", (h,)), ("hw", (h, h)), ("hg", (h,)), ("wc", (h, C)), ("bc", (C,))]
    f = cfg.ffn
    out = [("tok", (cfg.vocab, h)), ("pos", (cfg.max_pos, h)), ("eg", (h,)), ("eb", (h,))]
    for l in range(cfg.n_layers):
        out += [(f"{l}.wqkv", (h, 3 * h)), (f"{l}.bqkv", (3 * h,)), (f"{l}.wo", (h, h)), (f"{l}.bo", (h,)),
                (f"{l}.g1", (h,)), (f"{l}.b1n", (h,)), (f"{l}.w1", (h, f)), (f"{l}.b1", (f,)), (f"{l}.w2", (f, h)),
                (f"{l}.b2", (h,)), (f"{l}.g2", (h,)), (f"{l}.b2n", (h,))]
    return out + [("wc", (h, C)), ("bc", (C,))]


def _weights(cfg, seed):
    """One flat N(0, 0.02) float32 tensor on the GPU (LayerNorm gains around 1,
    the O label favoured as in a real head) and the tensors as views of it."""
    specs = _specs(cfg)
    n = sum(math.prod(s) for _, s in specs)
    flat = torch.randn(n, generator=_gen(seed, 1), device=DEV, dtype=torch.float32).mul_(0.02)
    views, at = {}, 0
    for name, s in specs:
        k = math.prod(s)
        views[name] = flat[at:at + k].view(s)
        at += k
        if len(s) == 1 and name.split(".")[-1] in ("eg", "g1", "g2", "ag", "mg", "fg", "hg"):
            views[name].add_(1.0)
    views["bc"][0] += 2.0
    return flat, views


def _packed(case, seed):
    """Lengths shuffled by the seed, boundaries on the host and ids on the GPU."""
    cfg = _shape(case)
    L = np.random.default_rng(seed).permutation(_lengths(case))
    cu = np.concatenate([[0], np.cumsum(L)]).astype(np.int32)
    ids = torch.randint(0, cfg.vocab, (int(cu[-1]),), generator=_gen(seed, 2), device=DEV, dtype=torch.int32)
    return cfg, cu, ids


# lines of scan records: a few thousand rendered ones, sampled into a text
_WORDS = ("remote service version detected module banner listener daemon agent package handler request response "
          "session cipher protocol certificate option default enabled outdated patched vulnerable exposure upgrade "
          "vendor release build kernel driver socket channel worker memory buffer overflow injection bypass "
          "validation header cookie payload archive cluster replica gateway proxy subnet route policy scanner "
          "severity medium high low critical apply latest stable window observed attacker local message the a of on "
          "in to and with from for by is was").split()
_TEXT_FIELDS = ["Description", "Synopsis", "Solution", "Plugin Output", "Risk Factor", "Notes", "Summary", "Impact"]


def _entity(r, t):
    def label():
        return r.choice("abcdefghijklmnopqrstuvwxyz") + "".join(r.choices("abcdefghijklmnopqrstuvwxyz0123456789-", k=r.randint(2, 6))) + "x"

    def host():
        return ".".join(label() for _ in range(r.randint(1, 3))) + "." + r.choice(
            ["corp", "lan", "intra", "net", "org", "local", "example", "internal"])

    if t == 1:
        return ".".join(str(r.randrange(256)) for _ in range(4))
    if t == 2:
        return host()
    if t == 3:
        return "CVE-%d-%d" % (r.randint(1999, 2025), r.randint(1000, 99999))
    if t == 4:
        return label() + "@" + host()
    if t == 5:
        return str(r.randint(1, 65535))
    if t == 6:
        return "https://" + host() + "/" + "/".join(r.choices(["docs", "kb", "patch", "notes"], k=r.randint(1, 3)))
    if t == 7:
        return ":".join("%02x" % r.randrange(256) for _ in range(6))
    return "".join(r.choices("0123456789abcdef", k=r.choice([32, 40, 64])))


def _lines(seed, n=3000):
    """Rendered lines: bytes back to back, lengths, and one entity per line (offset, length, type; 0 = none)."""
    r = random.Random(int(seed) + 17)
    names = {}
    for k, t in FIELDS.items():
        names.setdefault(t, []).append(k)
    text, lens, ent = [], [], []
    for _ in range(n):
        u = r.random()
        if u < 0.12:
            t = r.randint(1, 8)
            e = _entity(r, t)
            head = r.choice(names[t]) + ": "
            s, at = head + e + ("/tcp" if t == 5 else "") + "\n", (len(head), len(e), t)
        else:
            s = r.choice(_TEXT_FIELDS) + ": " + " ".join(r.choices(_WORDS, k=r.randint(8, 22)))
            at = (0, 0, 0)
            if u < 0.20:
                t = r.randint(1, 8)
                e = _entity(r, t)
                at = (len(s) + 4, len(e), t)
                s += " on " + e + " " + " ".join(r.choices(_WORDS, k=r.randint(2, 8)))
            s += ".\n"
        text.append(s)
        lens.append(len(s))
        ent.append(at)
    return "".join(text).encode(), lens, ent


def _records_text(case, seed):
    """Records of sampled lines: text, boundaries and entity spans on the GPU."""
    n = case["kbytes"] * 1000
    B = case["records"]
    pool, lens, ent = _lines(seed)
    pool = torch.frombuffer(bytearray(pool), dtype=torch.uint8).to(DEV)
    lens = torch.tensor(lens, device=DEV)
    ent = torch.tensor(ent, device=DEV)
    starts = torch.cumsum(lens, 0) - lens
    g = _gen(seed, 3)
    k = int(n / lens.double().mean().item() * 1.1) + 200
    pick = torch.randint(0, lens.numel(), (k,), generator=g, device=DEV)
    ln = lens[pick]
    at = torch.cumsum(ln, 0) - ln
    assert int(at[-1] + ln[-1]) >= n
    src = torch.repeat_interleave(starts[pick] - at, ln, output_size=int(ln.sum()))[:n]
    text = pool[src + torch.arange(n, device=DEV)].contiguous()
    del src
    # record sizes are lognormal; a record begins at a line
    w = torch.exp(0.6 * torch.randn(B, generator=g, device=DEV, dtype=torch.float64))
    want = (torch.cumsum(w, 0) / w.sum() * n)[:-1].long()
    cut = at[torch.searchsorted(at, want).clamp(max=k - 1)].clamp(max=n)
    cu = torch.cat([torch.zeros(1, device=DEV, dtype=torch.int64), cut, torch.full((1,), n, device=DEV)]).contiguous()
    e = ent[pick]
    b, t = at + e[:, 0], e[:, 2]
    keep = (t > 0) & (b + e[:, 1] <= n)
    b, ln, t = b[keep], e[keep, 1], t[keep]
    rec = torch.searchsorted(cu, b, right=True) - 1
    return text, cu, rec, t, b, b + ln


def _span_rows(cu, rec, t, b, e):
    return torch.stack([rec | (t << 32), b - cu[rec], e - cu[rec]], 1).contiguous()


def _tokens(text, cu, rec, t, b, e, seed):
    """Tokens of 2-8 bytes over each record and the labels a good model gives: the entities, a tenth of
    them missed."""
    n = text.numel()
    g = _gen(seed, 4)
    step = torch.randint(2, 9, (n // 4 + 16,), generator=g, device=DEV)
    edge = torch.cumsum(step, 0)
    edge = torch.unique(torch.cat([torch.zeros(1, device=DEV, dtype=torch.int64), edge[edge < n], cu[:-1][cu[:-1] < n]]))
    end = torch.cat([edge[1:], torch.full((1,), n, device=DEV)])
    r = torch.searchsorted(cu, edge, right=True) - 1
    off = torch.stack([edge - cu[r], end - cu[r]], 1).to(torch.int32).contiguous()
    cu_tok = torch.searchsorted(edge, cu).to(torch.int32)
    lab = torch.zeros(edge.numel(), dtype=torch.uint8, device=DEV)
    if b.numel():
        kept = torch.rand(b.numel(), generator=g, device=DEV) < 0.9
        k = torch.searchsorted(b, edge, right=True) - 1
        inside = (k >= 0) & (edge < e[k.clamp(min=0)]) & kept[k.clamp(min=0)]
        k = k.clamp(min=0)
        first = inside & ~torch.cat([torch.zeros(1, dtype=torch.bool, device=DEV), inside[:-1] & (k[1:] == k[:-1])])
        lab = torch.where(inside, 2 * t[k] - first.long(), torch.zeros_like(k)).to(torch.uint8).contiguous()
    return off, cu_tok.contiguous(), lab


# ----------------------------------------------------------------- prepare --
def prepare(case, seed):
    s = {"case": case}
    path = case["path"]
    if path in ENCODER_PATHS:
        cfg, cu, ids = _packed(case, seed)
        flat, _ = _weights(cfg, seed)
        blob = flat.cpu().numpy()
        del flat
        T, B = int(cu[-1]), len(cu) - 1
        s.update(cfg=cfg, T=T, B=B, ids=ids, h_cu=cu, cu=torch.from_numpy(cu).to(DEV))
        if path == "modern":
            m = api.ModernModel(cfg, blob, case["precision"])
        else:
            sc = np.array([FP8_SCALES] * cfg.n_layers) if case["precision"] == "fp8" else None
            m = api.Model(cfg, blob, case["precision"], sc)
        s["model"] = m
        if path in ("layer", "modern"):
            s["hidden"] = torch.empty((T, cfg.hidden), dtype=torch.float32, device=DEV)
        else:
            s["labels"] = torch.empty(T, dtype=torch.uint8, device=DEV)
            s["logits"] = torch.empty((T, cfg.n_labels), dtype=torch.float32, device=DEV)
            s["margin"] = torch.empty(T, dtype=torch.float32, device=DEV)
        if path == "bucket":
            _prepare_bucket(s)
        else:
            n = m.windowed_workspace_size(cu, WINDOW, STRIDE) if path == "windowed" else m.workspace_size(T, B)
            s["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return s
    return _prepare_text(s, case, seed)


def _prepare_bucket(s):
    """The server's form: buffers of the bucket's capacity (the power of two at or above twice the batch)."""
    T_cap = 1 << (2 * s["T"] - 1).bit_length()
    m, cfg, B, T = s["model"], s["cfg"], s["B"], s["T"]
    ids = torch.zeros(T_cap, dtype=torch.int32, device=DEV)
    ids[:T] = s["ids"]
    cu = torch.full((T_cap + 1,), T, dtype=torch.int32, device=DEV)
    cu[:B + 1] = s["cu"]
    n_tok = torch.tensor([T], dtype=torch.int32, device=DEV)
    lab = torch.zeros(T_cap, dtype=torch.uint8, device=DEV)
    z = torch.zeros((T_cap, cfg.n_labels), dtype=torch.float32, device=DEV)
    mg = torch.zeros(T_cap, dtype=torch.float32, device=DEV)
    ws = torch.empty(m.workspace_size(T_cap, T_cap), dtype=torch.uint8, device=DEV)
    s["graph"] = api.ner_forward_capture_bucket(m, ids, cu, n_tok, T_cap, T_cap, lab, z, mg, ws, ws.numel())
    s.update(labels=lab[:T], logits=z[:T], margin=mg[:T])


def _prepare_text(s, case, seed):
    path = case["path"]
    text, cu, rec, t, b, e = _records_text(case, seed)
    n, B = text.numel(), cu.numel() - 1
    s.update(n=n, B=B, text=text, cu=cu)

    def zeros(k, dtype):
        return torch.zeros(max(k, 1), dtype=dtype, device=DEV)

    if path in ("decode", "tail"):
        s["off"], s["cu_tok"], s["labels"] = _tokens(text, cu, rec, t, b, e, seed)
        s["T"] = T = s["labels"].numel()
        s["span_cap"] = n // 4 + B + 64
        s["spans"] = zeros(3 * s["span_cap"], torch.int64).view(-1, 3)
        s["cu_spans"] = zeros(B + 1, torch.int32)
        s["ws_dec"] = zeros(api.decode_workspace_size(T, B), torch.uint8)
    if path == "recognize":  # a quarter of the NER spans end early
        short = torch.rand(b.numel(), generator=_gen(seed, 5), device=DEV) < 0.25
        e = torch.where(short & (e - b > 4), e - (e - b) // 3, e)
        s["ner"] = _span_rows(cu, rec, t, b, e)
        s["ner_cu"] = torch.searchsorted(b, cu).to(torch.int32).contiguous()
        s["ner_cap"] = s["ner"].shape[0]
        s["cap"] = n // 4 + 64
    if path in ("recognize", "tail"):
        s["types"] = api.recognizer_types(TYPES)
        if path == "tail":
            s["cap"] = s["span_cap"] + n // 5 + 1
        s["merged"] = zeros(3 * s["cap"], torch.int64).view(-1, 3)
        s["cu_merged"] = zeros(B + 1, torch.int32)
        s["ws_rec"] = zeros(api.recognize_workspace_size(n, B), torch.uint8)
    if path == "fields":
        s["cap"] = n // 16 + 64
        s["merged"] = zeros(3 * s["cap"], torch.int64).view(-1, 3)
        s["cu_merged"] = zeros(B + 1, torch.int32)
        s["ws_fd"] = zeros(api.field_workspace_size(n, B), torch.uint8)
    if path in ("fields", "tail"):
        s["cache"] = api.PseudonymCache(np.random.default_rng(seed).bytes(32), SLUG, TYPES, 1 << 20)
        s["out_cap"] = n + n // 4 + 4096
        s["out"] = zeros(s["out_cap"], torch.uint8)
        s["cu_out"] = zeros(B + 1, torch.int64)
        s["ws_ps"] = zeros(api.pseudonymize_workspace_size(B, s["cap"]), torch.uint8)
    return s


# --------------------------------------------------------------------- run --
def run(s):
    path = s["case"]["path"]
    if path == "bucket":
        s["graph"].launch()
        return {"labels": s["labels"], "logits": s["logits"], "margin": s["margin"]}
    if path == "forward":
        api.ner_forward(s["model"], s["ids"], s["cu"], s["B"], s["T"], s["labels"], s["logits"], s["margin"], s["ws"],
                        s["ws"].numel())
        return {"labels": s["labels"], "logits": s["logits"], "margin": s["margin"]}
    if path == "windowed":
        api.ner_forward_windowed(s["model"], s["ids"], s["cu"], s["h_cu"], s["B"], s["T"], WINDOW, STRIDE,
                                 s["labels"], s["logits"], s["margin"], s["ws"], s["ws"].numel())
        return {"labels": s["labels"], "logits": s["logits"], "margin": s["margin"]}
    if path == "layer":
        api.encoder_hidden(s["model"], s["ids"], s["cu"], s["B"], s["T"], s["cfg"].n_layers, s["hidden"], s["ws"],
                           s["ws"].numel())
        return {"hidden": s["hidden"]}
    if path == "modern":
        s["model"].hidden(s["ids"], s["cu"], s["B"], s["T"], s["cfg"].n_layers, s["hidden"], s["ws"],
                          s["ws"].numel())
        return {"hidden": s["hidden"]}
    if path in ("decode", "tail"):
        api.decode_spans(s["labels"], s["off"], s["cu_tok"], s["B"], s["T"], len(TYPES), s["spans"], s["span_cap"],
                         s["cu_spans"], s["ws_dec"], s["ws_dec"].numel())
        if path == "decode":
            return {"spans": s["spans"], "cu_spans": s["cu_spans"]}
        _recognize(s, s["spans"], s["cu_spans"], s["span_cap"])
    elif path == "recognize":
        _recognize(s, s["ner"], s["ner_cu"], s["ner_cap"])
        return {"spans": s["merged"], "cu_spans": s["cu_merged"]}
    else:
        api.field_spans(s["text"], s["cu"], s["B"], s["n"], FIELDS, len(TYPES), s["merged"], s["cap"],
                        s["cu_merged"], s["ws_fd"], s["ws_fd"].numel())
    api.pseudonymize(s["cache"], s["text"], s["cu"], s["B"], s["merged"], s["cu_merged"], s["cap"], s["out"],
                     s["out_cap"], s["cu_out"], s["ws_ps"], s["ws_ps"].numel())
    return {"spans": s["merged"], "cu_spans": s["cu_merged"], "out": s["out"], "cu_out": s["cu_out"]}


def _recognize(s, ner, ner_cu, ner_cap):
    api.recognize_spans(s["text"], s["cu"], s["B"], s["n"], s["types"], len(TYPES), ner, ner_cu, ner_cap, s["merged"],
                        s["cap"], s["cu_merged"], s["ws_rec"], s["ws_rec"].numel())


# -------------------------------------------------------------------- work --
def work(case):
    path = case["path"]
    if path not in ENCODER_PATHS:
        n, B = case["kbytes"] * 1000, case["records"]
        spans = 24 * n // 320  # about one entity per 320 bytes
        tokens = 9 * n // 5    # label and byte range of a token of about 5 bytes
        if path == "decode":
            return {"bytes": tokens + spans + 8 * B, "flops": 0}
        if path == "recognize":
            return {"bytes": n + 2 * spans + 16 * B, "flops": 0}
        return {"bytes": 2 * n + spans + 20 * B + (tokens if path == "tail" else 0), "flops": 0}
    cfg, L = _shape(case), _lengths(case)
    T, h, n = int(L.sum()), cfg.hidden, cfg.n_layers
    if path == "windowed":
        w = []
        for x in L.tolist():
            k = 1 if x <= WINDOW else 1 + -(-(x - WINDOW) // STRIDE)
            w += [min(WINDOW, x - i * STRIDE) for i in range(k)]
        L = np.array(w)
    rows = int(L.sum())
    es = {"fp32": 4, "bf16": 2, "fp8": 1}[case["precision"]]
    if path == "modern":
        per = 3 * h * h + h * h + 3 * cfg.intermediate * h
        keys = 0
        for l in range(n):
            if l % cfg.global_every == 0:
                keys += int((L * L).sum())
            else:  # a token sees itself and up to half a window on each side
                w = np.minimum(cfg.local_window // 2, L - 1)
                keys += int((L * (2 * w + 1) - w * (w + 1)).sum())
    else:
        per = 4 * h * h + 2 * h * cfg.ffn
        keys = n * int((L * L).sum())
    flops = 2 * rows * per * n + 4 * h * keys
    if path in ("layer", "modern"):
        out = 4 * T * h
    else:
        out = T * (4 * cfg.n_labels + 5)
        flops += 2 * rows * h * cfg.n_labels
    return {"bytes": per * n * es + 4 * T + min(rows, cfg.vocab) * 4 * h + out, "flops": flops}


# ------------------------------------------------------------------- exact --
def _ln(x, g, b, eps):
    m = x.mean(-1, keepdim=True)
    d = x - m
    y = d * torch.rsqrt((d * d).mean(-1, keepdim=True) + eps) * g
    return y if b is None else y + b


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _attention(q, k, v, L, window=None):
    """[T, H, 64] packed by the lengths L: softmax(q k^T / 8) v within each record."""
    out = torch.empty_like(q)
    start = np.concatenate([[0], np.cumsum(L)])
    order = np.argsort(L, kind="stable")
    i = 0
    while i < len(order):
        longest = int(L[order[min(len(order) - 1, i + 63)]])
        group = max(1, min(64, int(6e7 // (q.shape[1] * longest * longest))))
        recs = order[i:i + group]
        i += group
        longest = int(L[recs].max())
        pos = torch.arange(longest, device=DEV)
        n = torch.tensor(L[recs], device=DEV)
        idx = torch.tensor(start[recs], device=DEV)[:, None] + torch.minimum(pos[None], n[:, None] - 1)
        qq, kk, vv = (x[idx].permute(0, 2, 1, 3).contiguous() for x in (q, k, v))
        p = torch.matmul(qq, kk.transpose(2, 3).contiguous()) / 8.0
        dead = (pos[None] >= n[:, None])[:, None, None, :]
        if window is not None:
            dead = dead | ((pos[:, None] - pos[None, :]).abs() > window)[None, None]
        p = torch.softmax(p.masked_fill(dead, -math.inf), -1)
        o = torch.matmul(p, vv).permute(0, 2, 1, 3)
        live = pos[None] < n[:, None]
        out[idx[live]] = o[live]
    return out


def _rotate(x, pos, theta):
    inv = theta ** (-torch.arange(0, 64, 2, device=DEV, dtype=torch.float64) / 64.0)
    a = (pos[:, None] * inv[None])[:, None, :]
    c, s = torch.cos(a), torch.sin(a)
    x1, x2 = x[..., :32], x[..., 32:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _chunked(f, x, rows=65536):
    return torch.cat([f(x[i:i + rows]) for i in range(0, x.shape[0], rows)])


def _encode(cfg, W, ids, L):
    h, H = cfg.hidden, cfg.n_heads
    T = int(ids.numel())
    start = np.concatenate([[0], np.cumsum(L)])[:-1]
    pos = torch.arange(T, device=DEV) - torch.repeat_interleave(torch.tensor(start, device=DEV), torch.tensor(L, device=DEV))
    modern = isinstance(cfg, ModernShape)
    w = {k: v.double() for k, v in W.items() if k not in ("tok",)}
    x = W["tok"][ids.long()].double()
    if not modern:
        x = x + w["pos"][pos]
    x = _ln(x, w["eg"], None if modern else w["eb"], cfg.ln_eps)
    for l in range(cfg.n_layers):
        p = "%d." % l
        if modern:
            y = x if l == 0 else _ln(x, w[p + "ag"], None, cfg.ln_eps)
            qkv = y @ w[p + "wqkv"]
        else:
            qkv = x @ w[p + "wqkv"] + w[p + "bqkv"]
        q, k, v = (qkv[:, i * h:(i + 1) * h].reshape(T, H, 64) for i in range(3))
        del qkv
        win = None
        if modern:
            glob = l % cfg.global_every == 0
            theta = cfg.theta_global if glob else cfg.theta_local
            win = None if glob else cfg.local_window // 2
            q, k = _rotate(q, pos.double(), theta), _rotate(k, pos.double(), theta)
        a = _attention(q, k, v, L, win).reshape(T, h)
        del q, k, v
        if modern:
            x = x + a @ w[p + "wo"]
            I = cfg.intermediate

            def mlp(r):
                u = _ln(r, w[p + "mg"], None, cfg.ln_eps) @ w[p + "wi"]
                return r + (_gelu(u[:, :I]) * u[:, I:]) @ w[p + "wo2"]
        else:
            x = _ln(x + a @ w[p + "wo"] + w[p + "bo"], w[p + "g1"], w[p + "b1n"], cfg.ln_eps)

            def mlp(r):
                y = r + _gelu(r @ w[p + "w1"] + w[p + "b1"]) @ w[p + "w2"] + w[p + "b2"]
                return _ln(y, w[p + "g2"], w[p + "b2n"], cfg.ln_eps)
        del a
        x = _chunked(mlp, x)
    return x, w


def exact(case, seed):
    """The encoder in float64 (unrounded weights and activations); spans and bytes have no such value."""
    path = case["path"]
    if path not in ENCODER_PATHS:
        return None
    cfg, cu, ids = _packed(case, seed)
    _, W = _weights(cfg, seed)
    L = np.diff(cu).astype(np.int64)
    if path in ("layer", "modern"):
        return {"hidden": _encode(cfg, W, ids, L)[0]}
    if path == "windowed":
        src, wl, own = [], [], np.empty(int(cu[-1]), np.int64)
        half, n = (WINDOW - STRIDE) // 2, 0
        for b, x in enumerate(L.tolist()):
            k = 1 if x <= WINDOW else 1 + -(-(x - WINDOW) // STRIDE)
            for i in range(k):  # a token belongs to the later window from half the overlap on
                w = min(WINDOW, x - i * STRIDE)
                src.append(int(cu[b]) + i * STRIDE + np.arange(w))
                wl.append(w)
                lo = 0 if i == 0 else half
                own[int(cu[b]) + i * STRIDE + lo:int(cu[b]) + i * STRIDE + w] = n + np.arange(lo, w)
                n += w
        x, w = _encode(cfg, W, ids[torch.tensor(np.concatenate(src), device=DEV)], np.array(wl, np.int64))
        x = x[torch.tensor(own, device=DEV)]
    else:
        x, w = _encode(cfg, W, ids, L)
    z = x @ w["wc"] + w["bc"]
    top = torch.topk(z, 2, -1).values
    return {"labels": None, "logits": z, "margin": top[:, 0] - top[:, 1]}
