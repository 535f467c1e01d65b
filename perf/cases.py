"""The calls a user of this library makes, at the sizes they are made at.

A case is one pass through the public entry points (the Stage front end and the
loss helpers of the binding) on synthetic inputs drawn on the GPU from a seed:

* "step":    one training iteration of an initiator's stage: forward, loss (and
             head update), early-stopped backward, adapter update;
* "train":   forward and backward of a stage inside the ring: dY comes from the
             next client, and adapter gradients add up until the update;
* "forward": the forward of a frozen stage, which runs ahead on later batches;
* "head":    the initiator's classifier loss on a stage output;
* "mse":     the initiator's regression loss on a stage output.

The shapes are those of the library's workloads (workloads.py) and of its
tests; draw() spreads over the widths, lengths and batch sizes in between.
"""
import math

import torch
import torch.nn.functional as F

from paper_2502_19864_amd import binding as B
from paper_2502_19864_amd.stage import Stage
from paper_2502_19864_amd.workloads import Workload

DEV = "cuda:0"
LR = 1e-4


def _stage(name, kind, arch, n_blocks, d, heads, ffn, seq, batch, cut, dtype="bf16", m=64, placement="houlsby",
           loss="dy"):
    case = dict(kind=kind, arch=arch, dtype=dtype, n_blocks=n_blocks, d=d, heads=heads, ffn=ffn, m=m, seq=seq,
                batch=batch, cut=cut, placement=placement, loss=loss)
    return dict(case, name=name) if name else case


def _head(name, batch, seq, d, classes):
    case = dict(kind="head", dtype="bf16", batch=batch, seq=seq, d=d, classes=classes)
    return dict(case, name=name) if name else case


def _mse(name, batch, seq, d):
    case = dict(kind="mse", dtype="bf16", batch=batch, seq=seq, d=d)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the small fp32 stage: what a first experiment runs; all launches, no work
        _stage("tiny_f32_step", "step", "bert", 2, 128, 2, 512, 32, 4, 0, dtype="f32", m=16, loss="mse"),
        # the initiator's two losses on a BERT-base batch
        _head("head_ce", 32, 128, 768, 2),
        _mse("mse_loss", 32, 128, 768),
        # one short request through a frozen encoder block: latency
        _stage("bert_block_forward_short", "forward", "bert", 1, 768, 12, 3072, 37, 1, 1),
        # a frozen client of the ring on the BERT-base batch
        _stage("bert_block_forward", "forward", "bert", 1, 768, 12, 3072, 128, 32, 1),
        # a client above the cut-off: forward and full backward of a block
        _stage("bert_block_train", "train", "bert", 1, 768, 12, 3072, 128, 32, -1),
        # the terminator on batches that are not padded to a round length, with
        # the paper's own single adapter per block
        _stage("bert_ragged_train", "train", "bert", 2, 768, 12, 3072, 203, 9, 0, placement="ffn"),
        # a BERT-large client: longer sequences, attention in kernels of its own
        _stage("bert_large_block_train", "train", "bert", 1, 1024, 16, 4096, 256, 16, -1),
        # one short prompt through a frozen 7B decoder block: the weights' bytes
        _stage("llama_block_forward_short", "forward", "llama", 1, 4096, 32, 11008, 100, 1, 1),
        # a frozen client and a training client of the 7B share
        _stage("llama_block_forward", "forward", "llama", 1, 4096, 32, 11008, 512, 4, 1),
        _stage("llama_block_train", "train", "llama", 1, 4096, 32, 11008, 512, 4, -1),
        # the headline step: 12 BERT-base blocks, the top four unfrozen
        _stage("bert_base_step", "step", "bert", 12, 768, 12, 3072, 128, 32, 8, loss="cls_ce"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_FLOPS = 1.7e12  # of the largest listed case


def draw(rng):
    while True:
        kind = rng.choice(("step", "train", "train", "train", "forward", "forward", "head", "mse"))
        if kind in ("head", "mse"):
            batch, seq, d = _log(rng, 1, 128), _log(rng, 1, 512), 8 * _log(rng, 16, 512)
            if batch * seq * d > 1 << 23:
                continue
            return _head(None, batch, seq, d, rng.choice((2, 2, 3, 5, 16))) if kind == "head" else _mse(None, batch, seq, d)
        placement = rng.choice(("houlsby", "houlsby", "ffn"))
        n_blocks = rng.choice((1, 2))
        cut = n_blocks if kind == "forward" else rng.randrange(-1 if kind == "train" else 0, n_blocks)
        loss = rng.choice(("cls_ce", "mse")) if kind == "step" else "dy"
        if rng.random() < 0.15:  # fp32 stages are small
            heads = rng.choice((1, 2, 4))
            d = heads * 2 * _log(rng, 8, 32) if heads % 2 == 0 else 4 * _log(rng, 8, 32)
            if loss == "cls_ce" and d % 8:
                continue
            return _stage(None, kind, "bert", n_blocks, d, heads, 4 * d, _log(rng, 5, 64), _log(rng, 1, 8), cut,
                          dtype="f32", m=rng.choice((8, 16, 32)), placement=placement, loss=loss)
        arch = rng.choice(("bert", "bert", "llama"))
        d = rng.choice((256, 512, 768, 768, 1024, 1024, 2048, 3072, 4096))
        dh = rng.choice((64, 64, 128)) if arch == "bert" else rng.choice((64, 128, 128))
        ffn = 64 * round((4 * d if arch == "bert" else 2.6875 * d) * rng.choice((0.5, 1, 1, 1)) / 64)
        case = _stage(None, kind, arch, n_blocks, d, d // dh, ffn, rng.choice((128, _log(rng, 16, 1024))),
                      _log(rng, 1, 64), cut, placement=placement, loss=loss)
        if work(case)["flops"] <= MOST_FLOPS and case["seq"] * case["batch"] <= 8192:
            return case


# ---------------------------------------------------------------- inputs
def _weight_names(case):
    d, f = case["d"], case["ffn"]
    if case["arch"] == "bert":
        return (("w_qkv", (d, 3 * d)), ("b_qkv", (3 * d,)), ("w_o", (d, d)), ("b_o", (d,)), ("ln1_g", (d,)),
                ("ln1_b", (d,)), ("w_i", (d, f)), ("b_i", (f,)), ("w_f", (f, d)), ("b_f", (d,)), ("ln2_g", (d,)),
                ("ln2_b", (d,)))
    return (("rms1_g", (d,)), ("w_qkv", (d, 3 * d)), ("w_o", (d, d)), ("rms2_g", (d,)), ("w_gu", (d, 2 * f)),
            ("w_d", (f, d)))


def _inputs(case, seed):
    """Every input of one iteration on the GPU, drawn as workloads.py draws them:
    x and targets ~ N(0, 1), weights, biases and adapters ~ N(0, 0.02), gains
    1 + N(0, 0.02), dY ~ N(0, 1e-2)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    sd = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(shape, std, mean=0.0, dtype=sd):
        return (torch.randn(shape, generator=g, device=DEV) * std + mean).to(dtype)

    shape = (case["batch"], case["seq"], case["d"])
    inp = {"x": normal(shape, 1.0)}
    if case["kind"] in ("train", "step", "forward"):
        d, m = case["d"], case["m"]
        inp["weights"] = [{k: normal(s, 0.02, 1.0 if k.endswith("_g") else 0.0) for k, s in _weight_names(case)}
                          for _ in range(case["n_blocks"])]
        inp["adapters"] = [tuple({"w_down": normal((d, m), 0.02, dtype=torch.float32),
                                  "w_up": normal((m, d), 0.02, dtype=torch.float32)} for _ in range(2))
                           for _ in range(case["n_blocks"])]
    loss = case.get("loss", case["kind"])
    if loss == "dy":
        inp["dy"] = normal(shape, 1e-2)
    elif loss == "mse":
        inp["target"] = normal(shape, 1.0)
    else:
        classes = case.get("classes", 2)
        inp["wh"] = normal((case["d"], classes), 0.02, dtype=torch.float32)
        inp["bh"] = torch.zeros(classes, device=DEV)
        inp["labels"] = torch.randint(0, classes, (case["batch"],), generator=g, device=DEV, dtype=torch.int32)
    return inp


class _DeviceStage(Stage):
    """A stage whose weights are on the GPU already."""

    def upload(self, a):
        return a.to(self.sdtype).contiguous()

    def f32(self, a):
        return a.to(torch.float32).clone()


def prepare(case, seed):
    inp = _inputs(case, seed)
    kind, x = case["kind"], inp["x"]
    s = {"case": case, "x": x, "stream": torch.cuda.current_stream().cuda_stream,
         "dt": B.BF16 if case["dtype"] == "bf16" else B.F32}
    loss = case.get("loss", kind)
    s["loss"] = torch.zeros(1, device=DEV)
    s["dy"] = inp["dy"] if loss == "dy" else torch.empty_like(x)
    if loss == "mse":
        s["target"] = inp["target"]
    elif loss in ("cls_ce", "head"):
        # weight and bias in one buffer, their gradients in another: one update
        n = inp["wh"].numel()
        s["hp"] = torch.cat([inp["wh"].reshape(-1), inp["bh"]])
        s["hg"] = torch.zeros_like(s["hp"])
        s["wh"], s["bh"] = s["hp"][:n].view_as(inp["wh"]), s["hp"][n:]
        s["gwh"], s["gbh"] = s["hg"][:n].view_as(inp["wh"]), s["hg"][n:]
        s["labels"] = inp["labels"]
    if kind in ("step", "train", "forward"):
        w = Workload("case", case["arch"], case["dtype"], case["n_blocks"], case["d"], case["heads"], case["ffn"],
                     case["m"], case["seq"], case["batch"], case["cut"], case["loss"], int(seed),
                     placement=case["placement"])
        s["stage"] = _DeviceStage(w, inp)
        s["y"] = torch.empty_like(x)
        s["dx"] = torch.empty_like(x) if case["cut"] < 0 else None
        s["stage"].ensure_workspace(case["batch"], case["seq"], case["cut"])
    return s


# ---------------------------------------------------------------- one pass
def _ce(s, y):
    case = s["case"]
    B.ringada_head_ce(s["stream"], s["dt"], y, case["batch"], case["seq"], case["d"], s["wh"], s["bh"],
                      s["wh"].shape[1], s["labels"], s["dy"], s["gwh"], s["gbh"], s["loss"])


def _unfrozen(case):
    """(block, adapter) of the unfrozen adapters: 0 attention, 1 FFN."""
    return [(l, a) for l in range(max(case["cut"], 0), case["n_blocks"])
            for a in range(1 if case["placement"] == "ffn" else 0, 2)]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "head":
        _ce(s, s["x"])
        return {"loss": s["loss"], "dy": s["dy"], "g_wh": s["gwh"], "g_bh": s["gbh"]}
    if kind == "mse":
        B.ringada_loss_mse(s["stream"], s["dt"], s["x"], s["target"], s["x"].numel(), s["dy"], s["loss"])
        return {"loss": s["loss"], "dy": s["dy"]}
    st, c = s["stage"], case["cut"]
    st.forward(s["x"], s["y"], c)
    out = {"y": s["y"]}
    if kind == "forward":
        return out
    if kind == "step":
        if case["loss"] == "mse":
            B.ringada_loss_mse(st.sptr, s["dt"], s["y"], s["target"], s["y"].numel(), s["dy"], s["loss"])
        else:
            _ce(s, s["y"])
            B.ringada_sgd_f32(st.sptr, s["hp"], s["hg"], s["hp"].numel(), LR)
            out.update(w_h=s["wh"], b_h=s["bh"])
        out.update(loss=s["loss"], dy=s["dy"])
    st.backward(s["dy"], c, s["dx"])
    if kind == "step":
        st.step(c, LR)
        keys = ("w_down", "w_up")
    else:
        keys = ("g_down", "g_up")
        if c < 0:
            out["dx"] = s["dx"]
    for l, a in _unfrozen(case):
        for k in keys:
            out["%s_%d_%d" % (k, l, a)] = st.adapters[l][a][k]
    return out


# ---------------------------------------------------------------- work, tolerance
def work(case):
    """Each input and output once, and the contractions: projections forward,
    and back to the input only (they are frozen); attention; the adapters with
    their weight gradients.  Nothing below the cut-off goes back."""
    es = 2 if case["dtype"] == "bf16" else 4
    T, d = case["batch"] * case["seq"], case["d"]
    act = T * d * es
    if case["kind"] == "mse":
        return {"bytes": 3 * act, "flops": 4 * T * d}
    if case["kind"] == "head":
        # position 0 of every sequence is read, all of dY written
        rows, params = case["batch"] * d * es, d * case["classes"] * 4
        return {"bytes": act + rows + 3 * params, "flops": 6 * case["batch"] * d * case["classes"]}
    n, f, m, c = case["n_blocks"], case["ffn"], case["m"], case["cut"]
    llama, single = case["arch"] == "llama", case["placement"] == "ffn"
    per_block = 4 * d * d + (3 if llama else 2) * d * f
    adapters = 1 if single else 2
    attn = 4 * T * case["seq"] * d * (0.5 if llama else 1.0)
    flops = n * (2 * T * per_block + attn + adapters * 4 * T * d * m)
    bts = 2 * act + n * (per_block * es + adapters * 2 * d * m * 4)
    if case["kind"] != "forward":
        for l in range(max(c, 0), n):
            stop = l == c
            if stop and single:
                flops += 6 * T * d * m
                continue
            flops += 2 * T * (per_block - 4 * d * d) + adapters * 8 * T * d * m
            if not stop:
                flops += 2 * T * 4 * d * d + 2 * attn
        bts += act + (act if c < 0 else 0) + (n - max(c, 0)) * adapters * 2 * d * m * 4 * 2
        if case["loss"] != "dy":
            bts += 2 * act
    return {"bytes": bts, "flops": flops}


def tolerance(case):
    """Relative 2-norm of the worst output: about four times the distance from
    64 bits measured for the listed and some drawn cases (fp32 4e-7 at most,
    with room for longer sums; the rounding of dY alone 1.7e-3; the gradients
    of a bf16 block 5.8e-3 post-LN and 8.5e-3 pre-RMS)."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    if case["kind"] in ("head", "mse"):
        return {"rel": 7e-3}
    return {"rel": 3e-2 if case["arch"] == "llama" else 2e-2}


# ---------------------------------------------------------------- the same in 64 bits
def _adapter(z, ad):
    return z if ad is None else z + F.gelu(z @ ad["w_down"]) @ ad["w_up"]


def _attention(q, k, v, case):
    """[T, d] projections -> [T, d]."""
    n, S, h = case["batch"], case["seq"], case["heads"]
    dh = case["d"] // h
    q, k, v = (t.reshape(n, S, h, dh).transpose(1, 2).contiguous() for t in (q, k, v))
    if case["arch"] == "llama":
        inv = 10000.0 ** (-2.0 * torch.arange(dh // 2, dtype=torch.float64, device=DEV) / dh)
        ang = torch.arange(S, dtype=torch.float64, device=DEV)[:, None] * inv

        def rotate(t):
            a, b = t[..., : dh // 2], t[..., dh // 2:]
            return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

        q, k = rotate(q), rotate(k)
    sc = q @ k.transpose(-1, -2).contiguous() / math.sqrt(dh)
    if case["arch"] == "llama":
        sc = sc.masked_fill(torch.ones(S, S, dtype=torch.bool, device=DEV).triu(1), -math.inf)
    return (sc.softmax(-1) @ v).transpose(1, 2).reshape(n * S, h * dh)


def _block(x, w, ad, case):
    d, f = case["d"], case["ffn"]
    if case["arch"] == "bert":
        q, k, v = (x @ w["w_qkv"] + w["b_qkv"]).split(d, 1)
        a = _adapter(_attention(q, k, v, case) @ w["w_o"] + w["b_o"], ad[0])
        h = F.layer_norm(x + a, (d,), w["ln1_g"], w["ln1_b"], 1e-12)
        z = _adapter(F.gelu(h @ w["w_i"] + w["b_i"]) @ w["w_f"] + w["b_f"], ad[1])
        return F.layer_norm(h + z, (d,), w["ln2_g"], w["ln2_b"], 1e-12)

    def rms(t, g):
        return t * torch.rsqrt((t * t).mean(-1, keepdim=True) + 1e-6) * g

    q, k, v = (rms(x, w["rms1_g"]) @ w["w_qkv"]).split(d, 1)
    h = x + _adapter(_attention(q, k, v, case) @ w["w_o"], ad[0])
    gate, up = (rms(h, w["rms2_g"]) @ w["w_gu"]).split(f, 1)
    return h + _adapter((F.silu(gate) * up) @ w["w_d"], ad[1])


def _loss64(y, inp, case):
    """Loss and d loss / dy (and the head's gradients) for y [batch, seq, d]."""
    if case.get("loss", case["kind"]) == "mse":
        diff = y - inp["target"].double()
        return (diff * diff).mean(), 2 * diff / diff.numel(), None, None
    lab = inp["labels"].long()
    wh, bh = inp["wh"].double(), inp["bh"].double()
    logp = (y[:, 0] @ wh + bh).log_softmax(1)
    loss = -logp.gather(1, lab[:, None]).mean()
    dl = logp.exp()
    dl[torch.arange(len(lab), device=DEV), lab] -= 1
    dl /= len(lab)
    dy = torch.zeros_like(y)
    dy[:, 0] = dl @ wh.t()
    return loss, dy, y[:, 0].t() @ dl, dl.sum(0)


def exact(case, seed):
    inp = _inputs(case, seed)
    kind, x = case["kind"], inp["x"].double()
    if kind in ("head", "mse"):
        loss, dy, gwh, gbh = _loss64(x, inp, case)
        out = {"loss": loss.reshape(1), "dy": dy}
        return out if kind == "mse" else dict(out, g_wh=gwh, g_bh=gbh)
    single, bf = case["placement"] == "ffn", case["dtype"] == "bf16"

    def computed(t):  # a bf16 stage multiplies with the rounded adapter weights
        return (t.to(torch.bfloat16) if bf else t).double().requires_grad_(kind != "forward")

    weights = [{k: t.double() for k, t in w.items()} for w in inp["weights"]]
    ads = [[None if single and a == 0 else {k: computed(t) for k, t in pair[a].items()} for a in range(2)]
           for pair in inp["adapters"]]
    x.requires_grad_(kind != "forward")
    h = x.reshape(-1, case["d"])
    for w, ad in zip(weights, ads):
        h = _block(h, w, ad, case)
    y = h.reshape(x.shape)
    out = {"y": y.detach()}
    if kind == "forward":
        return out
    if kind == "step":
        loss, dy, gwh, gbh = _loss64(y.detach(), inp, case)
        out.update(loss=loss.reshape(1), dy=dy)
        if gwh is not None:
            out.update(w_h=inp["wh"].double() - LR * gwh, b_h=inp["bh"].double() - LR * gbh)
    else:
        dy = inp["dy"].double()
    want = [(l, a, k) for l, a in _unfrozen(case) for k in ("w_down", "w_up")]
    grads = torch.autograd.grad(y, [x] + [ads[l][a][k] for l, a, k in want], dy)
    if case["cut"] < 0 and kind == "train":
        out["dx"] = grads[0]
    for (l, a, k), g in zip(want, grads[1:]):
        if kind == "step":
            out["%s_%d_%d" % (k, l, a)] = inp["adapters"][l][a][k].double() - LR * g
        else:
            out["%s_%d_%d" % (k.replace("w_", "g_"), l, a)] = g
    return out
