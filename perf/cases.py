"""Performance cases of the library: what users have it do, through the public
entry points of ``paper_2511_11337_amd``, from one small buffer to the batches
of the benchmark's models.

* ``compress`` / ``decompress``: host bytes to a container and back.
* ``encode`` / ``decode``: device-resident chunks with a workspace allocated
  once, as the benchmark and a serving loop do.
* ``logits``: teacher-forced logits of whole sequences.
* ``grad``: loss and gradient of a training batch.
* ``int8``: the integer-only pipeline, encode then decode.

Models: the shipped trained d_model 256 x 3 layers (containers always use it:
a chunk that an untrained model cannot shrink is stored raw), d_model 64 x 2
layers and, for the mixed streams in FP8, d_model 512 x 4 layers (both
seed-init).  Inputs are the repository's own synthetic records; a case fixes
its chunk lengths, the seed its bytes.
"""
import functools
import os

import numpy as np
import torch

import paper_2511_11337_amd as boa
from paper_2511_11337_amd import train
from synth import (ModelConfig, chunk_lengths_heavy, chunk_lengths_uniform, init_weights, mixed_chunks, param_layout,
                   records_f32_mix, records_structured64)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TRAINED = os.path.join(ROOT, "paper_2511_11337_amd", "models", "records64_d256x3.boam")
CONFIGS = {64: ModelConfig(64, 2), 256: ModelConfig(256, 3), 512: ModelConfig(512, 4)}


def listed():
    return [
        # one short buffer through the host API: launches, copies and the serial chain of a single stream
        dict(name="compress_small_f32", kind="compress", d_model=256, dtype="f32", chunks=1, chunk_len=4096, cut=0),
        dict(name="decompress_small_f32", kind="decompress", d_model=256, dtype="f32", chunks=1, chunk_len=1024, cut=0),
        # a file of a few MiB cut into 16 KiB chunks, the last one short
        dict(name="compress_file_bf16", kind="compress", d_model=256, dtype="bf16", chunks=256, chunk_len=16384,
             cut=5003),
        # one decoding stream per compute unit
        dict(name="decompress_file_bf16", kind="decompress", d_model=256, dtype="bf16", chunks=256, chunk_len=1024,
             cut=333),
        # the benchmark's batch: thousands of uneven chunks (its uniform length law, scaled down from KiB)
        dict(name="encode_batch_bf16", kind="encode", d_model=256, dtype="bf16", chunks=8192, lo=128, hi=1024),
        dict(name="decode_batch_bf16", kind="decode", d_model=256, dtype="bf16", chunks=8192, lo=128, hi=1024),
        # the mixed-stream workload: heavy-tailed lengths, three record types, the larger model in FP8
        dict(name="encode_mixed_fp8", kind="encode", d_model=512, dtype="fp8", chunks=3072, lo=16, hi=1024),
        dict(name="decode_mixed_fp8", kind="decode", d_model=512, dtype="fp8", chunks=3072, lo=16, hi=1024),
        # scoring a few sequences of odd length
        dict(name="logits_odd_f32", kind="logits", d_model=256, dtype="f32", batch=3, seq_len=333),
        # the training recipe's step, and a small odd batch in full precision
        dict(name="grad_recipe_bf16", kind="grad", d_model=256, dtype="bf16", batch=32, seq_len=8192, chunk_t=256),
        dict(name="grad_small_f32", kind="grad", d_model=64, dtype="f32", batch=5, seq_len=777, chunk_t=256),
        # containers that decode on any device
        dict(name="int8_round_trip", kind="int8", d_model=256, dtype="int8", chunks=1024, lo=128, hi=384),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["compress", "decompress", "encode", "decode", "encode", "decode", "logits", "grad", "grad",
                       "int8"])
    d = 256 if kind in ("encode", "decode") and rng.random() < 0.6 else rng.choice([64, 256, 512])
    dtype = rng.choice(["f32", "bf16", "fp8"])
    if kind in ("compress", "decompress"):
        d = 256
        n = _log_int(rng, 1, 256)
        length = _log_int(rng, 256, 16384 if kind == "compress" else 1024)
        if kind == "compress" and n < 16:
            length = min(length, 4096)
        return dict(kind=kind, d_model=d, dtype=dtype, chunks=n, chunk_len=length, cut=rng.randrange(0, length // 2))
    if kind in ("encode", "decode"):
        n = _log_int(rng, 256, 8192 if d < 512 else 3072)
        lo = _log_int(rng, 16, 128 if d < 512 else 16)
        return dict(kind=kind, d_model=d, dtype=dtype, chunks=n, lo=lo, hi=8 * lo if d < 512 else 64 * lo)
    if kind == "logits":
        return dict(kind=kind, d_model=d, dtype=dtype, batch=_log_int(rng, 1, 64), seq_len=_log_int(rng, 2, 2000))
    if kind == "grad":
        d = rng.choice([64, 256])
        return dict(kind=kind, d_model=d, dtype=rng.choice(["f32", "bf16"]), batch=_log_int(rng, 1, 32),
                    seq_len=_log_int(rng, 65, 4096), chunk_t=rng.choice([128, 256, 256]))
    lo = _log_int(rng, 16, 128)
    return dict(kind="int8", d_model=rng.choice([64, 256]), dtype="int8", chunks=_log_int(rng, 1, 1024), lo=lo,
                hi=3 * lo)


@functools.lru_cache(maxsize=None)
def _init(d_model):
    return init_weights(CONFIGS[d_model], 4242 + d_model)


def _model(d_model):
    return boa.Model.load(TRAINED) if d_model == 256 else boa.Model(CONFIGS[d_model], _init(d_model))


def _records(case, n, seed):
    return (records_structured64 if case["d_model"] == 256 else records_f32_mix)(n, seed)


def _chunks(case, seed):
    """(host bytes, chunk lengths) of an encode / decode / int8 case."""
    n = case["chunks"]
    if case["d_model"] == 512:
        lens = chunk_lengths_heavy(n, n, lo=case["lo"], ratio=case["hi"] / case["lo"])
        data = np.concatenate([c for _, c in mixed_chunks(lens, seed % 1000003)])
    else:
        lens = chunk_lengths_uniform(n, case["lo"], case["hi"], n)
        data = _records(case, int(lens.sum()), seed)
    return data, lens.astype(np.uint64)


def _sequences(case, seed):
    B, T = case["batch"], case["seq_len"]
    return torch.from_numpy(_records(case, B * T, seed).reshape(B, T)).cuda()


def _payload_index(chunk_lens):
    """Chunk of every byte of an encode call's payload buffer, and its place in that chunk's region."""
    cap = 2 * chunk_lens.astype(np.int64) + 64
    start = np.concatenate([[0], np.cumsum(cap)[:-1]])
    owner = np.repeat(np.arange(cap.size), cap)
    return (torch.from_numpy(owner.astype(np.int32)).cuda(),
            torch.from_numpy((np.arange(owner.size) - start[owner]).astype(np.int32)).cuda())


def _host_lens(pay_len):
    return pay_len.cpu().numpy().astype(np.uint32).astype(np.uint64)


def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    m = _model(case["d_model"])
    s = dict(case=case, model=m)
    if kind in ("compress", "decompress"):
        s["data"] = _records(case, case["chunks"] * case["chunk_len"] - case["cut"], seed)
        if kind == "compress":                         # raw storage bounds a container
            s["container"] = np.zeros(64 + 32 * case["chunks"] + s["data"].size, dtype=np.uint8)
        else:
            s["blob"] = boa.compress(m, s["data"], chunk_len=case["chunk_len"], dtype=dtype)
    elif kind in ("encode", "decode"):
        data, s["lens"] = _chunks(case, seed)
        s["data"] = torch.from_numpy(data).cuda()
        ws = boa.workspace_size(m, s["lens"], kind, dtype=dtype)
        s["workspace"] = torch.empty(max(ws, 1), dtype=torch.uint8, device="cuda")
        if kind == "encode":
            s["owner"], s["place"] = _payload_index(s["lens"])
        else:
            s["payload"], s["pay_off"], pl, _ = boa.encode_dev(m, s["data"], s["lens"], dtype=dtype, ideal=False)
            s["pay_len"] = _host_lens(pl)
            s["first"] = data[np.concatenate([[0], np.cumsum(s["lens"])[:-1]]).astype(np.int64)]
            s["out"] = torch.empty(data.size, dtype=torch.uint8, device="cuda")
    elif kind == "int8":
        data, s["lens"] = _chunks(case, seed)
        s["data"] = torch.from_numpy(data).cuda()
        s["qmodel"] = boa.QModel(m)
        s["owner"], s["place"] = _payload_index(s["lens"])
        s["first"] = data[np.concatenate([[0], np.cumsum(s["lens"])[:-1]]).astype(np.int64)]
    else:
        s["tokens"] = _sequences(case, seed)
    return s


def _coded(s, payload, pay_len):
    """The payload buffer with the bytes past each chunk's payload, which are not written, as zeros."""
    return torch.where(s["place"] < pay_len[s["owner"]], payload, torch.zeros((), dtype=torch.uint8, device="cuda"))


def run(s):
    case, m = s["case"], s["model"]
    kind, dtype = case["kind"], case["dtype"]
    if kind == "compress":
        blob = boa.compress(m, s["data"], chunk_len=case["chunk_len"], dtype=dtype)
        s["container"][:len(blob)] = np.frombuffer(blob, dtype=np.uint8)
        s["container"][len(blob):] = 0
        return s["container"], len(blob)
    if kind == "decompress":
        return np.frombuffer(boa.decompress(m, s["blob"]), dtype=np.uint8)
    if kind == "encode":
        payload, _, pay_len, _ = boa.encode_dev(m, s["data"], s["lens"], dtype=dtype, ideal=False,
                                                workspace=s["workspace"])
        return _coded(s, payload, pay_len), pay_len
    if kind == "decode":
        return boa.decode_dev(m, s["payload"], s["pay_off"], s["pay_len"], s["first"], s["lens"], dtype=dtype,
                              out=s["out"], workspace=s["workspace"])
    if kind == "int8":
        payload, off, pay_len = boa.int_encode_dev(s["qmodel"], s["data"], s["lens"])
        out = boa.int_decode_dev(s["qmodel"], payload, off, _host_lens(pay_len), s["first"], s["lens"])
        return _coded(s, payload, pay_len), pay_len, out
    if kind == "logits":
        return boa.logits(m, s["tokens"], dtype=dtype)
    return train.loss_and_grad(m, s["tokens"], chunk_t=case["chunk_t"], dtype=dtype)


def _positions(case):
    if case["kind"] in ("compress", "decompress"):
        return case["chunks"] * (case["chunk_len"] - 1) - case["cut"]
    if "batch" in case:
        return case["batch"] * (case["seq_len"] - 1)
    mean = 0.5 * (case["lo"] + case["hi"]) if case["d_model"] < 512 else 8.0 * case["lo"]
    return int(case["chunks"] * (mean - 1))


def work(case):
    cfg = CONFIGS[case["d_model"]]
    D, Di, N, R, L = cfg.d_model, cfg.d_inner, cfg.d_state, cfg.dt_rank, cfg.n_layers
    # per position: the projections of every layer and the head, conv, scan and gate
    flops = L * (2 * (2 * Di * D + (R + 2 * N) * Di + R * Di + D * Di) + 12 * Di + 6 * Di * N) + 2 * 256 * D
    params = sum(int(np.prod(shape)) for _, shape in param_layout(cfg))
    weights = params * {"f32": 4, "bf16": 2, "fp8": 1, "int8": 1}[case["dtype"]]
    n = _positions(case)
    if case["kind"] == "grad":
        return dict(bytes=n + 2 * 4 * params, flops=3 * flops * n)
    if case["kind"] == "logits":
        return dict(bytes=n + 4 * 256 * n + weights, flops=flops * n)
    passes = 2 if case["kind"] == "int8" else 1
    return dict(bytes=passes * (n + 0.25 * n + weights), flops=passes * flops * n)


# ---------------------------------------------------------------- 64-bit values
def _logits64(cfg, P, tokens):
    """Logits [B, T-1, 256] in float64 with plain torch operations, sequence form."""
    F = torch.nn.functional
    tok = tokens.long()
    B, T = tok.shape
    Tn, Di, N, R, K = T - 1, cfg.d_inner, cfg.d_state, cfg.dt_rank, cfg.d_conv
    r = P["embed"][tok[:, :Tn].reshape(-1)].reshape(B, Tn, cfg.d_model)
    for l in range(cfg.n_layers):
        p = {k.split(".")[-1]: v for k, v in P.items() if k.startswith(f"layers.{l}.")}
        a = F.layer_norm(r, (cfg.d_model,), p["norm_w"], p["norm_b"], 1e-5)
        xz = a @ p["in_proj_w"].T
        x, z = xz[..., :Di], xz[..., Di:]
        xp = torch.cat([x.new_zeros(B, K - 1, Di), x], dim=1)
        xs = F.silu(sum(xp[:, k:k + Tn] * p["conv_w"][:, k] for k in range(K)) + p["conv_b"])
        dbc = xs @ p["x_proj_w"].T
        dt = F.softplus(dbc[..., :R] @ p["dt_proj_w"].T + p["dt_proj_b"])
        A, Bm, Cm = -torch.exp(p["A_log"]), dbc[..., R:R + N], dbc[..., R + N:]
        h, ys = x.new_zeros(B, Di, N), []
        for t in range(Tn):
            h = torch.exp(dt[:, t, :, None] * A) * h + (dt[:, t] * xs[:, t])[..., None] * Bm[:, t, None, :]
            ys.append((h * Cm[:, t, None, :]).sum(-1))
        y = torch.stack(ys, dim=1) + p["D"] * xs
        r = r + (y * F.silu(z)) @ p["out_proj_w"].T
    r = F.layer_norm(r, (cfg.d_model,), P["norm_f_w"], P["norm_f_b"], 1e-5)
    return r @ P["head_w"].T + P["head_b"]


def exact(case, seed):
    if case["kind"] not in ("logits", "grad"):
        return None                                    # bytes
    cfg = CONFIGS[case["d_model"]]
    if case["batch"] * case["seq_len"] > 8192 and case["kind"] == "grad" or case["batch"] * case["seq_len"] > 65536:
        return None                                    # a sequential recurrence in float64 of that size is slow
    m = _model(case["d_model"])
    flat = torch.from_numpy(m.get_weights()).cuda().double()
    tokens = _sequences(case, seed)
    names, at = {}, 0
    for name, shape in param_layout(cfg):
        n = int(np.prod(shape))
        names[name] = flat[at:at + n].reshape(shape)
        at += n
    if case["kind"] == "logits":
        with torch.no_grad():
            return _logits64(cfg, names, tokens)
    P = {k: v.clone().requires_grad_(True) for k, v in names.items()}
    loss = torch.nn.functional.cross_entropy(_logits64(cfg, P, tokens).reshape(-1, 256),
                                             tokens[:, 1:].reshape(-1).long())
    grads = torch.autograd.grad(loss, list(P.values()))
    return float(loss), torch.cat([g.reshape(-1) for g in grads])
