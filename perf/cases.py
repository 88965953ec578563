"""Performance cases of the Comba operator library.

Each case is one call (or one forward + backward) that a program using this
library makes through its public entry points: decoding steps, prefill of one
prompt or of a batch, training steps of a layer (fixed length, packed, one long
row), and the layer's input prologue and output gate.  Sizes are those of the
repository's named workloads (340M and 1.3B layers: 8 or 16 heads of 128; the
merged heads of 256; the tiny fp32 workload), its benchmark, and ragged sizes
around them.

A case is a dict of plain values:
  kind   decode | prefill | train | train_direct | grad | layer_io   (see run)
  B, T, H, dk, dv          sizes (packed: B = 1, T the total)
  lens                     packed sequence lengths "n,n,..." or ""
  dtype                    bf16 | f32 (q, k, v, beta, beta~, dO)
  h0, bt                   initial states given; separate feedback strength given
"""
import math

import torch
import torch.nn.functional as F

import paper_2506_02475_amd as comba

CHUNK = 64


def _case(kind, B, T, H, dk, dv=None, *, lens=(), dtype="bf16", h0=True, bt=False, name=None):
    c = {"kind": kind, "B": B, "T": sum(lens) if lens else T, "H": H, "dk": dk,
         "dv": dk if dv is None else dv, "lens": ",".join(str(n) for n in lens), "dtype": dtype,
         "h0": h0, "bt": bt}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # One user's chat: one token of one sequence through one layer of 16 heads.
        _case("decode", 1, 1, 16, 128, bt=True, name="decode_b1"),
        # A serving batch's step: 64 sequences, one token each.
        _case("decode", 64, 1, 16, 128, bt=True, name="decode_b64"),
        # The tiny fp32 forward used to check a port or a model against references.
        _case("prefill", 1, 256, 1, 64, dtype="f32", h0=False, name="prefill_f32_tiny"),
        # Full-precision debugging run of a small model's layer, forward and gradients.
        _case("grad", 2, 1000, 8, 64, dtype="f32", name="grad_f32_b2_t1000"),
        # One prompt of ordinary length (not a multiple of the chunk) before decoding.
        _case("prefill", 1, 1000, 16, 128, h0=False, bt=True, name="prefill_b1_t1000"),
        # Batched prefill / evaluation at the merged heads of 256.
        _case("prefill", 4, 4096, 8, 256, name="prefill_b4_t4096_d256"),
        # Packed fine-tuning batch at the 340M layer's heads: unequal documents.
        _case("train", 1, 0, 8, 128, lens=(3001, 517, 64, 4096, 1250, 777, 2048, 1, 2900, 1730),
              h0=False, bt=True, name="train_packed_16k"),
        # Pretraining step of the 1.3B layer through autograd, as a model trains it.
        _case("train", 4, 4096, 16, 128, h0=False, bt=True, name="train_b4_t4096_h16"),
        # The same tokens with heads of 256, the training pair called by hand.
        _case("train_direct", 4, 4096, 8, 256, name="train_b4_t4096_d256"),
        # Long-context training: one row of 65,536 tokens.
        _case("train_direct", 1, 65536, 16, 128, name="train_b1_t65536"),
        # Long-context packed forward: 16 documents, 1 K to 65 K tokens.
        _case("prefill", 1, 0, 16, 128,
              lens=(50122, 17890, 64003, 9971, 41234, 2050, 65155, 30777, 58111, 12345, 1977, 36900,
                    47001, 21212, 5500, 61280), name="prefill_packed_512k"),
        # What surrounds the operator in the layer: prologue and gate, forward and backward.
        _case("layer_io", 4, 4096, 16, 128, name="layer_io_b4_t4096"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "train", "train",
                       "train_direct", "grad", "layer_io"])
    dtype = "f32" if (kind == "grad" and rng.random() < 0.5) or \
        (kind in ("prefill", "decode") and rng.random() < 0.15) else "bf16"
    dk = rng.choice([64, 128, 128, 128, 256])
    dv = dk
    if rng.random() < 0.15 and dk >= 128:
        dv = 384 - dk  # 128 with 256
    if dtype == "f32":
        dk = dv = 64 if kind != "decode" else min(dk, 128)
    H = rng.choice([4, 6, 8, 16])
    bt = rng.random() < 0.6
    h0 = rng.random() < 0.5
    if kind == "decode":  # T > 1: a short draft verified at once
        T = rng.choice([1, 1, 1, 3, 8])
        return _case(kind, _log_int(rng, 1, 200), T, H, dk, dv, dtype=dtype, h0=True, bt=bt)
    # tokens x heads x head size bounded by that of the 1.3B layer's training batch
    room = 4 * 4096 * 16 * 128 // (H * max(dk, dv))
    if dtype == "f32":
        room //= 16
    form = rng.choice(["batch", "batch", "one", "packed"])
    if form == "packed" and kind != "layer_io":
        n = rng.randint(2, 24)
        lens = [_log_int(rng, 1, max(2, room // n)) for _ in range(n)]
        return _case(kind, 1, 0, H, dk, dv, lens=lens, dtype=dtype, h0=h0, bt=bt)
    B = 1 if form == "one" else _log_int(rng, 1, 12)
    T = _log_int(rng, 48, max(64, room // B))
    return _case(kind, B, T, H, dk, dv, dtype=dtype, h0=h0, bt=bt)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _lens(case):
    return [int(x) for x in case["lens"].split(",")] if case["lens"] else []


def _inputs(case, seed):
    """Seeded inputs with the operator's distributions (q, k normalised per head,
    g = -softplus, beta = sigmoid, d in (0, 1)), in their storage types."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * int(seed) + 17)
    B, T, H, dk, dv = (case[n] for n in ("B", "T", "H", "dk", "dv"))
    dt, f32 = _dtype(case), torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=f32)

    s = {}
    if case["kind"] == "layer_io":
        for n, d in (("q", dk), ("k", dk), ("v", dv)):
            s["x" + n] = normal(B, T, H, d).to(dt)
            s["w" + n] = 0.5 * normal(H, d, 4)
            s["g" + n] = normal(B, T, H, d)
        s["o"], s["z"], s["dy"] = normal(B, T, H, dv), normal(B, T, H, dv).to(dt), \
            normal(B, T, H, dv)
        return s
    lens = _lens(case)
    N = len(lens) if lens else B
    s["q"] = F.normalize(normal(B, T, H, dk), dim=-1).to(dt)
    s["k"] = F.normalize(normal(B, T, H, dk), dim=-1).to(dt)
    s["v"] = normal(B, T, H, dv).to(dt)
    s["g"] = -F.softplus(normal(B, T, H))
    s["beta"] = torch.sigmoid(normal(B, T, H)).to(dt)
    s["bt"] = (s["beta"].float() * torch.sigmoid(normal(H))).to(dt) if case["bt"] else None
    s["d"] = torch.rand((H,), generator=gen, device=dev, dtype=f32)
    s["h0"] = 0.02 * normal(N, H, dk, dv) if case["h0"] else None
    if case["kind"] in ("train", "train_direct", "grad"):
        s["dO"] = normal(B, T, H, dv).to(dt)
        s["dht"] = 0.1 * normal(N, H, dk, dv) if case["h0"] else None
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    lens = _lens(case)
    s["packed"] = {}
    if lens:
        cu = torch.zeros(len(lens) + 1, dtype=torch.int32)
        cu[1:] = torch.cumsum(torch.tensor(lens), 0)
        s["packed"] = {"cu_seqlens": cu.cuda(), "cu_seqlens_host": cu.numpy()}
    if case["kind"] == "decode":
        s["ht"] = torch.empty_like(s["h0"])  # the cache's other half
    if case["kind"] == "train":
        # the gradient of o arrives in fp32, as from the output gate
        s["do"] = s["dO"].float()
        for n in ("q", "k", "v", "g", "beta", "d", "h0", "bt"):
            if s[n] is not None:
                s[n].requires_grad_()
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "layer_io":
        q, k, v = comba.comba_prologue_fwd(s["xq"], s["xk"], s["xv"], s["wq"], s["wk"], s["wv"])
        y = comba.comba_gate_fwd(s["o"], s["z"])
        do, dz = comba.comba_gate_bwd(s["o"], s["z"], s["dy"])
        out = comba.comba_prologue_bwd(s["xq"], s["xk"], s["xv"], s["wq"], s["wk"], s["wv"],
                                       s["gq"], s["gk"], s["gv"])
        out = dict(out)
        out.update(q=q, k=k, v=v, y=y, do=do, dz=dz)
        return out
    args = (s["q"], s["k"], s["v"], s["g"], s["beta"], s["d"], s["h0"])
    kws = dict(s["packed"], beta_tilde=s["bt"])
    if kind == "decode":
        o, ht = comba.comba_recurrent_fwd(*args, ht=s["ht"], **kws)
        return {"o": o, "ht": ht}
    if kind == "prefill":
        o, ht = comba.comba_chunk_fwd(*args, **kws)
        return {"o": o, "ht": ht}
    if kind == "train":
        o, ht = comba.comba_chunk(*args, **kws)
        names = [n for n in ("q", "k", "v", "g", "beta", "d", "h0", "bt") if s[n] is not None]
        outs, ups = [o], [s["do"]]
        if s["dht"] is not None:
            outs.append(ht)
            ups.append(s["dht"])
        grads = torch.autograd.grad(outs, [s[n] for n in names], ups)
        return dict({"d" + n: x for n, x in zip(names, grads)}, o=o.detach(), ht=ht.detach())
    if kind == "train_direct":
        o, ht, ws = comba.comba_chunk_fwd_save(*args, **kws)
        gr = comba.comba_chunk_bwd_saved(*args, s["dO"], s["dht"], workspace=ws, **kws)
    else:  # grad: forward, then the recomputing backward
        o, ht = comba.comba_chunk_fwd(*args, **kws)
        gr = comba.comba_chunk_bwd(*args, s["dO"], s["dht"], **kws)
    names = {"dq": "dq", "dk": "dk", "dv": "dv", "dg": "dg", "dbeta": "dbeta", "dd": "dd",
             "dh0": "dh0", "dbeta_tilde": "dbt"}
    out = {names[n]: x for n, x in gr.items() if x is not None}
    out.update(o=o, ht=ht)
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    B, T, H, dk, dv = (case[n] for n in ("B", "T", "H", "dk", "dv"))
    e = 2 if case["dtype"] == "bf16" else 4
    tok = B * T * H
    if case["kind"] == "layer_io":
        d = 2 * dk + dv
        io = tok * (d * (e + e) + d * (e + 4 + 4) + dv * (4 + e + e) + dv * (4 + e + 4 + 4 + 4))
        return {"bytes": io + 2 * H * d * 4 * 4, "flops": tok * (d * 60 + dv * 20)}
    lens = _lens(case) or [T] * B
    N, bt = len(lens), 1 if case["bt"] else 0
    states = N * H * dk * dv * 4
    inputs = tok * ((2 * dk + dv) * e + 4 + e * (1 + bt)) + (states if case["h0"] else 0)
    outputs = tok * dv * 4 + states
    if case["kind"] == "decode":
        return {"bytes": inputs + outputs, "flops": tok * 7 * dk * dv}
    chunks = sum(-(-n // CHUNK) for n in lens) * H
    fwd = chunks * (6 * CHUNK * dk * dv + 4 * CHUNK * CHUNK * dk + 4 * CHUNK * CHUNK * dv)
    if case["kind"] == "prefill":
        return {"bytes": inputs + outputs, "flops": fwd}
    g = e if case["kind"] == "train" else 4  # autograd hands gradients back in the inputs' types
    dout = tok * dv * (4 if case["kind"] == "train" else e)
    grads = tok * ((2 * dk + dv) * g + 4 + g * (1 + bt)) + (2 * states if case["h0"] else 0)
    bwd = chunks * (12 * CHUNK * dk * dv + 10 * CHUNK * CHUNK * dk + 8 * CHUNK * CHUNK * dv)
    # the inputs are read by the forward and by the backward
    return {"bytes": 2 * inputs + outputs + dout + grads, "flops": fwd + bwd}


def tolerance(case):
    # Four times the largest relative error against 64 bits over the outputs of
    # listed and drawn cases: bf16 outputs carry their own rounding; fp32 outputs
    # of the bf16 path carry about 16 bits per operand.
    if case["kind"] == "layer_io" or case["kind"] == "train":
        return {"rel": 1e-2, "max": 0.1}
    if case["kind"] == "decode":
        return {"rel": 1e-5, "max": 1e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-3, "max": 0.05}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _chunked(q, k, v, g, beta, bt, d, h0):
    """Comba over rows of equal length, [B,T,H,*] in float64: chunks of 64 with
    the triangular inverse as a product of squarings, states chunk by chunk."""
    B, T, H, dk = q.shape
    dv = v.shape[-1]
    n = -(-T // CHUNK)
    pad = n * CHUNK - T

    def split(x):
        x = F.pad(x, (0, 0) * (x.dim() - 2) + (0, pad)) if pad else x
        x = x.reshape((B, n, CHUNK) + x.shape[2:])
        return x.transpose(2, 3).transpose(1, 2).contiguous()  # [B,H,n,CHUNK,...]

    q, k, v, g, beta, bt = (split(x) for x in (q, k, v, g, beta, bt))
    qt = q - d.reshape(1, H, 1, 1, 1) * k
    G = g.cumsum(-1)
    Gm = G - g
    low = torch.ones(CHUNK, CHUNK, dtype=torch.bool, device=q.device).tril(-1)
    kT = k.transpose(-1, -2).contiguous()
    e = torch.exp((Gm.unsqueeze(-1) - G.unsqueeze(-2)).masked_fill(~low, -math.inf))
    L = -bt.unsqueeze(-1) * e * (k @ kT)
    eye = torch.eye(CHUNK, dtype=q.dtype, device=q.device)
    M = eye + L
    for _ in range(5):
        L = L @ L
        M = M + L @ M
    MV = M @ (beta.unsqueeze(-1) * v)
    MK = M @ ((bt * torch.exp(Gm)).unsqueeze(-1) * k)
    last = G[..., -1:]
    KtT = (torch.exp(last - G).unsqueeze(-1) * k).transpose(-1, -2).contiguous()
    decay = torch.exp(last).unsqueeze(-1)
    S = torch.zeros(B, H, dk, dv, dtype=q.dtype, device=q.device) if h0 is None else h0
    Xs, Us = [], []
    for c in range(n):
        U = MV[:, :, c] - MK[:, :, c] @ S
        Xs.append(S)
        Us.append(U)
        S = decay[:, :, c] * S + KtT[:, :, c] @ U
    X, U = torch.stack(Xs, 2), torch.stack(Us, 2)
    a = torch.exp((G.unsqueeze(-1) - G.unsqueeze(-2)).masked_fill(
        ~(low | eye.bool()), -math.inf)) * (qt @ kT)
    o = torch.exp(G).unsqueeze(-1) * (qt @ X) + a @ U
    o = o.transpose(1, 2).transpose(2, 3).reshape(B, n * CHUNK, H, dv)[:, :T]
    return o, S


def _exact_layer_io(s):
    x = {n: s[n].double() for n in ("o", "z", "dy")}
    sg = torch.sigmoid(x["z"])
    out = {"y": x["o"] * sg, "do": x["dy"] * sg, "dz": x["dy"] * x["o"] * sg * (1 - sg)}
    for n in ("q", "k", "v"):
        a = s["x" + n].double().requires_grad_()
        w = s["w" + n].double().requires_grad_()
        T = a.shape[1]
        p = F.pad(a, (0, 0, 0, 0, 3, 0))
        u = sum(p[:, j:j + T] * w[:, :, j] for j in range(4))
        y = F.silu(u)
        if n != "v":
            y = y / torch.sqrt((y * y).sum(-1, keepdim=True) + 1e-6)
        out[n] = y.detach()
        out["dx" + n], out["dw" + n] = torch.autograd.grad(y, [a, w], s["g" + n].double())
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "layer_io":
        return _exact_layer_io(s)
    lens = _lens(case) or [case["T"]] * case["B"]
    packed = bool(case["lens"])
    names = [n for n in ("q", "k", "v", "g", "beta", "d", "h0", "bt") if s[n] is not None]
    grads = kind in ("train", "train_direct", "grad")
    x = {n: s[n].double().requires_grad_(grads) for n in names}
    bt = x.get("bt", x["beta"])
    with torch.set_grad_enabled(grads):
        if packed:
            os, hts, a = [], [], 0
            for i, n in enumerate(lens):
                b = a + n
                h0 = x["h0"][i:i + 1] if "h0" in x else None
                o, ht = _chunked(x["q"][:, a:b], x["k"][:, a:b], x["v"][:, a:b], x["g"][:, a:b],
                                 x["beta"][:, a:b], bt[:, a:b], x["d"], h0)
                os.append(o)
                hts.append(ht)
                a = b
            o, ht = torch.cat(os, 1), torch.cat(hts, 0)
        else:
            o, ht = _chunked(x["q"], x["k"], x["v"], x["g"], x["beta"], bt, x["d"], x.get("h0"))
        out = {"o": o.detach(), "ht": ht.detach()}
        if grads:
            outs, ups = [o], [s["dO"].double()]
            if s["dht"] is not None:
                outs.append(ht)
                ups.append(s["dht"].double())
            gr = torch.autograd.grad(outs, [x[n] for n in names], ups)
            out.update({"d" + n: y for n, y in zip(names, gr)})
    if kind in ("train_direct", "grad") and "h0" not in x:
        out["dh0"] = None
    return out
