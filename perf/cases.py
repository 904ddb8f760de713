"""Performance cases of the HDET step: the calls that a training program makes, at the sizes it makes them.

A case is one pass of a training loop's body through the public binding, on buffers laid out as such a program keeps them:
  kind "flat"  hdet_fanout_step on caller-made gradients, with the sync-step calls (converge, controller) where one is due
  kind "warm"  hdet_warm_init_noalloc: the N perturbed copies of a checkpoint, with the bfloat16 copy
  kind "mlp"   forward, backward and update of N replicas of an MLP
  kind "tf"    the same for N replicas of a decoder-only transformer
"call" says how a model step is made: "train" is hdet_train_step (one call), "two" is hdet_forward_backward and
hdet_fanout_step; "two" also returns the gradients.  A state starts in the middle of a run (update 100 is done), at a
constant base rate, so that a pass can be repeated.  exact() evaluates the first pass on a state in 64 bits.
"""
import math

import torch

import paper_2604_24708_amd as H

DEV = "cuda:0"
T0 = 100                 # updates done before the first pass
TOTAL = 1 << 40          # updates of the run: never reached
WD = 0.01
BETA1, BETA2, EPS, MOM = 0.9, 0.999, 1e-8, 0.9
DROP_BASE, DROP_ALPHA = 0.1, 1.0
WDCH_BASE, WDCH_ALPHA = 0.05, 0.5
LN_EPS = 1e-5


def listed():
    return [
        # the small fp32 study: a 40-step run is nothing but launches and latency
        dict(name="mlp_fp32_small", kind="mlp", n=4, widths="64-128-10", batch=32, bf16=False, opt="sgdm", shared=False, sync=4, call="two"),
        # the update of a large model whose gradients come from elsewhere: a pure memory stream
        dict(name="flat_adamw", kind="flat", n=8, p=96_000_000, opt="adamw", shared=False, one_state=False, sync=16),
        # the paper's gradient AllReduce with plain momentum on a model of odd size, every step a sync step
        dict(name="flat_sgdm_sync", kind="flat", n=5, p=1_000_003, opt="sgdm", shared=True, one_state=False, sync=1),
        # many replicas of a small model: more than fit one block, one set of moments
        dict(name="flat_shared_n32", kind="flat", n=32, p=2_000_000, opt="adamw", shared=True, one_state=True, sync=16),
        # start of a run from a checkpoint (Eq. 10), bfloat16 copy included
        dict(name="warm_init", kind="warm", n=8, p=64_000_000),
        # mixed precision, the update inside the weight-gradient products: small batch, so bound by the weights
        dict(name="mlp_bf16", kind="mlp", n=8, widths="1024-4096-4096-4096-1000", batch=256, bf16=True, opt="adamw", shared=False,
             sync=16, call="train"),
        # mixed precision on widths that are no multiples of the tiles (nor, one of them, of 8), shared gradients
        dict(name="mlp_bf16_ragged", kind="mlp", n=6, widths="784-1500-700-100", batch=96, bf16=True, opt="adamw", shared=True, sync=16,
             call="two"),
        # a whole training step of the 6-layer transformer: the head and the loss of a large vocabulary weigh most
        dict(name="tf_6l", kind="tf", n=8, blocks=6, d=512, heads=8, ff=2048, seq=256, vocab=32000, batch=16, bf16=True, channels=False,
             sync=32, call="two"),
        # the layers of the 12-layer transformer (two blocks of it under a small head), all three explored scalars on
        dict(name="tf_d1024_blocks", kind="tf", n=8, blocks=2, d=1024, heads=16, ff=4096, seq=512, vocab=2048, batch=16, bf16=True,
             channels=True, sync=64, call="train"),
        # one block over long sequences: attention weighs most
        dict(name="tf_long_seq", kind="tf", n=4, blocks=1, d=512, heads=8, ff=2048, seq=2048, vocab=4096, batch=2, bf16=True, channels=False,
             sync=32, call="two"),
        # the smallest transformer study, in fp32: launches and latency again
        dict(name="tf_fp32_small", kind="tf", n=4, blocks=2, d=64, heads=4, ff=256, seq=32, vocab=512, batch=4, bf16=False, channels=False,
             sync=4, call="train"),
        # full precision at a size where the products count
        dict(name="tf_fp32", kind="tf", n=4, blocks=2, d=256, heads=4, ff=1024, seq=128, vocab=4000, batch=4, bf16=False, channels=False,
             sync=16, call="two"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flat", "flat", "warm", "mlp32", "mlp16", "tf16", "tf32"])
    if kind == "flat":
        n = _log(rng, 1, 64)
        p = _log(rng, 1000, min(96_000_000, 400_000_000 // n))
        opt = rng.choice(["adamw", "adamw", "sgdm"])
        shared = rng.random() < 0.5
        return dict(kind="flat", n=n, p=p, opt=opt, shared=shared, one_state=bool(shared and opt == "adamw" and rng.random() < 0.5),
                    sync=rng.choice([1, 4, 16, 64]))
    if kind == "warm":
        n = _log(rng, 1, 16)
        return dict(kind="warm", n=n, p=_log(rng, 10_000, 400_000_000 // n if n > 6 else 64_000_000))
    if kind == "mlp32":
        widths = [_log(rng, 16, 784)] + [_log(rng, 16, 512) for _ in range(rng.randint(1, 3))] + [_log(rng, 2, 100)]
        return dict(kind="mlp", n=rng.randint(2, 8), widths="-".join(map(str, widths)), batch=_log(rng, 8, 128), bf16=False,
                    opt=rng.choice(["sgdm", "adamw"]), shared=rng.random() < 0.5, sync=4, call=rng.choice(["two", "train"]))
    if kind == "mlp16":
        step = rng.choice([1, 4, 8, 64])
        size = lambda lo, hi: max(step, _log(rng, lo, hi) // step * step)  # noqa: E731
        widths = [size(128, 1024)] + [size(256, 4096) for _ in range(rng.randint(1, 3))] + [size(10, 1000)]
        return dict(kind="mlp", n=rng.randint(2, 8), widths="-".join(map(str, widths)), batch=_log(rng, 32, 256), bf16=True, opt="adamw",
                    shared=rng.random() < 0.5, sync=16, call=rng.choice(["two", "train"]))
    if kind == "tf16":
        heads, dh = rng.choice([4, 6, 8, 12, 16]), rng.choice([32, 64, 64, 64])
        seq = rng.choice([64, 100, 128, 192, 256, 384, 512, 1024, 2048])
        d = heads * dh
        return dict(kind="tf", n=rng.randint(2, 8), blocks=rng.randint(1, 3), d=d, heads=heads, ff=4 * d, seq=seq, vocab=_log(rng, 500, 12000),
                    batch=max(1, min(16, 4096 // seq)), bf16=True, channels=rng.random() < 0.4, sync=32, call=rng.choice(["two", "train"]))
    heads, dh = rng.choice([2, 4, 8]), rng.choice([16, 32, 64])
    d = heads * dh
    return dict(kind="tf", n=rng.randint(2, 6), blocks=rng.randint(1, 3), d=d, heads=heads, ff=4 * d, seq=_log(rng, 16, 192), vocab=_log(rng, 64, 4000),
                batch=rng.randint(1, 6), bf16=False, channels=rng.random() < 0.3, sync=4, call=rng.choice(["two", "train"]))


# ---- sizes ------------------------------------------------------------------------------------------
def _widths(case):
    return [int(w) for w in case["widths"].split("-")]


def _shapes(case):
    """Tensors of a parameter plane in their order."""
    if case["kind"] in ("flat", "warm"):
        return [("p", (case["p"],))]
    if case["kind"] == "mlp":
        w = _widths(case)
        return [x for i in range(len(w) - 1) for x in (("w%d" % i, (w[i + 1], w[i])), ("b%d" % i, (w[i + 1],)))]
    d, ff, v, s = case["d"], case["ff"], case["vocab"], case["seq"]
    out = [("tok", (v, d)), ("pos", (s, d))]
    for l in range(case["blocks"]):
        out += [("g1.%d" % l, (d,)), ("c1.%d" % l, (d,)), ("qkv.%d" % l, (3 * d, d)), ("bqkv.%d" % l, (3 * d,)), ("o.%d" % l, (d, d)),
                ("bo.%d" % l, (d,)), ("g2.%d" % l, (d,)), ("c2.%d" % l, (d,)), ("w1.%d" % l, (ff, d)), ("b1.%d" % l, (ff,)),
                ("w2.%d" % l, (d, ff)), ("b2.%d" % l, (d,))]
    return out + [("gf", (d,)), ("cf", (d,)), ("head", (v, d)), ("bhead", (v,))]


def _count(case):
    return sum(math.prod(s) for _, s in _shapes(case))


def _split(case, flat):
    out, off = {}, 0
    for name, shape in _shapes(case):
        k = math.prod(shape)
        out[name] = flat[off:off + k].view(shape)
        off += k
    return out


def _rho(n, alpha):
    c = (n - 1) / 2.0
    return [1.0 + alpha * ((r - c) / max(c, 0.5)) for r in range(n)]


def _lr_max(case):
    return 0.02 if case["opt_"] == "sgdm" else 3e-4


def _opt(case):
    return case.get("opt", "adamw")


def _shared(case):
    return bool(case.get("shared", False))


def _one_state(case):
    """One set of moments: asked for on flat buffers, always taken by the mixed-precision models that share gradients."""
    return bool(case.get("one_state", case["kind"] != "flat" and _shared(case) and _opt(case) == "adamw"))


# ---- inputs -----------------------------------------------------------------------------------------
def _inputs(case, seed):
    """Everything a pass reads, made from the seed alone: [N, stride] planes (fp32) and the batch."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n, p = case["n"], _count(case)
    stride = (p + 63) // 64 * 64
    theta = torch.zeros((n, stride), device=DEV)
    one = theta[0, :p]
    for (name, shape), t in zip(_shapes(case), _split(case, one).values()):
        if case["kind"] == "mlp":
            bound = 1.0 / math.sqrt(shape[1] if len(shape) == 2 else shape[0])
            t.uniform_(-bound, bound, generator=g)
        else:
            # embeddings and vectors as initialised, matrices as training leaves them: their outputs are of the inputs' size
            emb = len(shape) == 1 or name in ("tok", "pos")
            t.normal_(0.0, 0.02 if emb else 1.0 / math.sqrt(shape[1]), generator=g)
            if name[0] == "g" and case["kind"] == "tf":
                t.add_(1.0)
    out = dict(theta=theta, p=p, stride=stride)
    if case["kind"] == "warm":
        out["theta0"] = one.clone()
        return out
    # the replicas have drifted apart since the last converge
    for r in range(1, n):
        theta[r, :p].normal_(0.0, 1e-4, generator=g).add_(one)
    planes = 1 if _one_state(case) else n
    m = torch.zeros((planes, stride), device=DEV)
    v = None
    if case["kind"] == "flat":
        m[:, :p].normal_(0.0, 3e-4, generator=g)
    if _opt(case) == "adamw":
        v = torch.zeros((planes, stride), device=DEV)
        v[:, :p].uniform_(2e-7, 2e-6, generator=g)
    grads = torch.zeros((n, stride), device=DEV)
    out.update(m=m, v=v, grads=grads)
    if case["kind"] == "flat":
        grads[:, :p].normal_(0.0, 1e-3, generator=g)
        out["losses"] = [1.0 + 0.01 * ((r + seed) % n) for r in range(n)]
    elif case["kind"] == "mlp":
        w, b = _widths(case), case["batch"]
        out["x"] = torch.randn((n, b, w[0]), device=DEV, generator=g)
        teacher = torch.randn((w[0], w[-1]), device=DEV, generator=g)
        out["y"] = torch.argmax(out["x"] @ teacher, dim=-1).to(torch.int32)
    else:
        s, b, vocab = case["seq"], case["batch"], case["vocab"]
        w = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64) ** -1.1      # Zipf(1.1) by inverse CDF
        u = torch.rand((n, b, s + 1), device=DEV, dtype=torch.float64, generator=g)
        tok = torch.searchsorted(torch.cumsum(w / w.sum(), 0), u, right=True).clamp_(max=vocab - 1).to(torch.int32)
        out["x"], out["y"] = tok[..., :-1].contiguous(), tok[..., 1:].contiguous()
    return out


class _State:
    """A handle and the buffers it borrows."""

    def __init__(self, case, inp):
        self.case, self.inp, self.t = case, inp, T0
        n, kind = case["n"], case["kind"]
        bf16 = bool(case.get("bf16", False))
        kw = dict(n_replicas=n, sync_interval=case["sync"], total_steps=TOTAL, warm_steps=0, lr_max=_lr_max(dict(opt_=_opt(case))),
                  constant_lr=1, alpha=0.1, autolr_enabled=1, optimizer=H.HDET_SGDM if _opt(case) == "sgdm" else H.HDET_ADAMW,
                  momentum=MOM, beta1=BETA1, beta2=BETA2, eps=EPS, weight_decay=WD, seed=7, lambda_=1e-3,
                  grad_mode=H.HDET_GRAD_SHARED if _shared(case) else H.HDET_GRAD_PER_REPLICA, shared_opt_state=int(_one_state(case)),
                  precision=H.HDET_BF16_GEMM_FP32_MASTER if bf16 else H.HDET_FP32, stream=torch.cuda.current_stream().cuda_stream)
        if kind == "flat":
            kw.update(model_kind=H.HDET_FLAT, n_params=case["p"])
        elif kind == "mlp":
            kw.update(model_kind=H.HDET_MLP, widths=_widths(case), batch=case["batch"])
        else:
            kw.update(model_kind=H.HDET_TRANSFORMER, batch=case["batch"], n_blocks=case["blocks"], d_model=case["d"], n_heads=case["heads"],
                      d_ff=case["ff"], seq_len=case["seq"], vocab=case["vocab"])
            if case["channels"]:
                kw["extra"] = [(H.HDET_CH_DROPOUT, DROP_BASE, DROP_ALPHA, 1e-3, 0.0, 0.45), (H.HDET_CH_WD, WDCH_BASE, WDCH_ALPHA, 1e-3, 0.0, 1.0)]
        cfg = H.make_config(**kw)
        _, _, ws = H.hdet_workspace_bytes(cfg, inp["stride"])
        self.shadow = torch.empty((n, inp["stride"]), dtype=torch.bfloat16, device=DEV) if bf16 else None
        self.ws = torch.empty(max(ws, 16), dtype=torch.uint8, device=DEV)
        self.h = H.hdet_create(cfg, inp["theta"], inp["m"], inp["v"], grads=inp["grads"], params_bf16=self.shadow, workspace=self.ws,
                               plane_stride=inp["stride"])
        st = H.hdet_get_state(self.h)
        st.t = T0
        H.hdet_set_state(self.h, st)

    def __del__(self):
        if getattr(self, "h", None):
            H.hdet_destroy(self.h)
            self.h = None


def prepare(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "warm":
        inp["case"] = case
        inp["shadow"] = torch.zeros((case["n"], inp["stride"]), dtype=torch.bfloat16, device=DEV)
        inp["seed"] = seed
        return inp
    return _State(case, inp)


def _tensors(case, planes):
    """The planes tensor by tensor, [N][elements] each: small and large gradients side by side."""
    out, off = {}, 0
    for name, shape in _shapes(case):
        out[name] = planes[:, off:off + math.prod(shape)]
        off += math.prod(shape)
    return out


def _outputs(case, p, theta, m, v, grads):
    """Everything the pass wrote.  A model's gradients -- or, where they are no output, the first moments, a tenth of them --
    come tensor by tensor (a model of many blocks: as whole planes)."""
    out = dict(params=theta[:, :p], m=m[:, :p])
    if v is not None:
        out["v"] = v[:, :p]
    if case["kind"] == "flat":
        return out
    key = "m"
    if case["call"] == "two" and not _shared(case):
        out["grads"], key = grads[:, :p], "grads"
    if len(_shapes(case)) <= 48:
        out[key] = _tensors(case, out[key])
    return out


def run(s):
    if isinstance(s, dict):
        H.hdet_warm_init_noalloc(s["theta0"], s["theta"], s["shadow"], s["p"], s["stride"], s["case"]["n"], 0.01, s["seed"],
                                 torch.cuda.current_stream().cuda_stream)
        return dict(params=s["theta"][:, :s["p"]], copy=s["shadow"][:, :s["p"]].view(torch.int16))
    c, i = s.case, s.inp
    if c["kind"] == "flat":
        H.hdet_fanout_step(s.h, i["grads"], H.HDET_FUSE_CONVERGE)
    elif c["call"] == "train":
        H.hdet_train_step(s.h, i["x"], i["y"], H.HDET_FUSE_CONVERGE)
    else:
        H.hdet_forward_backward(s.h, i["x"], i["y"])
        H.hdet_fanout_step(s.h, None, H.HDET_FUSE_CONVERGE)
    s.t += 1
    if s.t % c["sync"] == 0:
        H.hdet_converge(s.h)
        H.hdet_autolr_update(s.h, i.get("losses"), c["n"])
    return _outputs(c, i["p"], i["theta"], i["m"], i["v"], i["grads"])


# ---- what a pass cannot do without --------------------------------------------------------------------
def work(case):
    n, p = case["n"], _count(case)
    if case["kind"] == "warm":
        return dict(bytes=4.0 * p + 6.0 * n * p, flops=0.0)
    planes = 1 if _one_state(case) else n
    moments = 1 if _opt(case) == "sgdm" else 2
    update = 8.0 * n * p + 8.0 * moments * planes * p              # theta, moments: read and written
    if case["kind"] == "flat":
        return dict(bytes=update + 4.0 * n * p, flops=0.0)
    if case.get("bf16"):
        update += 2.0 * n * p + 2.0 * n * p                        # the bfloat16 copy: read by the products, written by the update
    if case["call"] == "two" and not _shared(case):
        update += 4.0 * n * p                                      # the gradients, an output of their own
    if case["kind"] == "mlp":
        w, b = _widths(case), case["batch"]
        mm = sum(w[i] * w[i + 1] for i in range(len(w) - 1))
        return dict(bytes=update + 4.0 * n * b * (w[0] + 1), flops=2.0 * n * b * (3 * mm - w[0] * w[1]))
    m, d, ff = case["batch"] * case["seq"], case["d"], case["ff"]
    mm = case["blocks"] * (4 * d * d + 2 * d * ff) + case["vocab"] * d
    attn = case["blocks"] * 2.0 * m * d * (case["seq"] + 1)          # q k and p v under the causal mask: S + 1 over 2 keys a query
    return dict(bytes=update + 8.0 * n * m, flops=n * 3.0 * (2.0 * m * mm + attn))


def tolerance(case):
    if case["kind"] == "warm":
        return dict(rel=1e-6, max=1e-5, differ=1e-3)                 # one fp32 rounding; a copy may round the other way next to a tie
    if case["kind"] == "flat":
        return dict(rel=1e-6, max=1e-5)
    if not case["bf16"]:
        return dict(rel=1e-5, max=4e-4)                              # sums in another order
    # values next to a rounding boundary of bfloat16 may round the other way where they are stored; behind a ReLU that also
    # moves units across zero (64 bits with nothing rounded differ by up to 0.05 in norm there, and by 0.003 without a ReLU)
    return dict(rel=0.02 if case["kind"] == "mlp" else 0.012, max=0.9)


# ---- the same in 64 bits -------------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, k0, k1):
    """Philox-4x32-10 on int64 tensors holding 32-bit words."""
    mask = 0xFFFFFFFF

    def mul(a, b):                                                    # high and low words of a 32 x 32-bit product
        lo = (a & 0xFFFF) * b
        hi = (a >> 16) * b + (lo >> 16)
        return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)

    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        h0, l0 = mul(c0, 0xD2511F53)
        h1, l1 = mul(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
    return c0, c1, c2, c3


def _normals(seed, replica, n):
    b = torch.arange((n + 3) // 4, device=DEV, dtype=torch.int64)
    z = torch.zeros_like(b)
    w = _philox(b, z + replica, z, z + 0x5741524D, seed & 0xFFFFFFFF, seed >> 32)
    out = []
    for u, t in ((w[0], w[1]), (w[2], w[3])):
        rad = torch.sqrt(-2.0 * torch.log((u.double() + 1.0) / 4294967296.0))
        ang = t.double() * (2.0 * math.pi / 4294967296.0)
        out += [rad * torch.cos(ang), rad * torch.sin(ang)]
    return torch.stack(out, 1).reshape(-1)[:n]


def _keep(case, replica, site, count, p):
    b = torch.arange((count + 3) // 4, device=DEV, dtype=torch.int64)
    z = torch.zeros_like(b)
    w = _philox(b, z + T0 + 1, z + replica * 65536 + site, z + 0x44524F50, 7, 0)
    return torch.stack(w, 1).reshape(-1)[:count] >= int(math.floor(p * 4294967296.0))


def _as_used(case, t):
    """The operand as the products see it: rounded to bfloat16 in mixed precision."""
    return (t.to(torch.bfloat16) if case["bf16"] else t).double()


def _mlp_grad(case, flat, x, y):
    par = {k: (_as_used(case, t) if t.dim() == 2 else t.double()).requires_grad_() for k, t in _split(case, flat).items()}
    a = _as_used(case, x)
    layers = len(_widths(case)) - 1
    for i in range(layers):
        a = a @ par["w%d" % i].T + par["b%d" % i]
        if i + 1 < layers:
            a = torch.relu(a)
    torch.nn.functional.cross_entropy(a, y.long()).backward()
    return torch.cat([t.grad.reshape(-1) for t in par.values()])


def _tf_grad(case, flat, ids, tgt, replica):
    matrices = ("qkv", "o", "w1", "w2", "head")
    par = {k: (_as_used(case, t) if k.split(".")[0] in matrices else t.double()).requires_grad_() for k, t in _split(case, flat).items()}
    b, s, d, nh = case["batch"], case["seq"], case["d"], case["heads"]
    dh, m = d // nh, b * s
    p = 0.0
    if case["channels"]:
        p = torch.tensor(DROP_BASE * _rho(case["n"], DROP_ALPHA)[replica], dtype=torch.float64).float().double().item()

    def drop(t, site):
        if p == 0.0:
            return t
        return torch.where(_keep(case, replica, site, m * d, p).view(m, d), t / (1.0 - p), torch.zeros((), dtype=t.dtype, device=DEV))

    def ln(t, g, c):
        return torch.nn.functional.layer_norm(t, (d,), par[g], par[c], LN_EPS)

    x = par["tok"][ids.reshape(-1).long()] + par["pos"].repeat(b, 1)
    causal = torch.ones((s, s), dtype=torch.bool, device=DEV).tril()
    for l in range(case["blocks"]):
        k = ".%d" % l
        qkv = ln(x, "g1" + k, "c1" + k) @ par["qkv" + k].T + par["bqkv" + k]
        q, kk, v = (t.reshape(b, s, nh, dh).transpose(1, 2).contiguous() for t in qkv.split(d, dim=1))
        a = []
        for i in range(b):                                            # one sequence at a time: bounded memory
            sc = torch.matmul(q[i], kk[i].transpose(1, 2).contiguous()) / math.sqrt(dh)
            a.append(torch.matmul(torch.softmax(sc.masked_fill(~causal, -math.inf), -1), v[i]).transpose(0, 1).reshape(s, d))
        x = x + drop(torch.cat(a) @ par["o" + k].T + par["bo" + k], 2 * l)
        f = torch.nn.functional.gelu(ln(x, "g2" + k, "c2" + k) @ par["w1" + k].T + par["b1" + k], approximate="tanh")
        x = x + drop(f @ par["w2" + k].T + par["b2" + k], 2 * l + 1)
    logits = ln(x, "gf", "cf") @ par["head"].T + par["bhead"]
    torch.nn.functional.cross_entropy(logits, tgt.reshape(-1).long()).backward()
    return torch.cat([t.grad.reshape(-1) for t in par.values()])


def exact(case, seed):
    i = _inputs(case, seed)
    n, p = case["n"], i["p"]
    if case["kind"] == "warm":
        t0 = i["theta0"].double()
        sigma = 0.01 * torch.sqrt((t0 * t0).sum() / p)
        return dict(params=torch.stack([t0 + sigma * _normals(seed, r, p) for r in range(n)]), copy=None)
    theta, m, v = i["theta"][:, :p].double(), i["m"][:, :p].double(), None if i["v"] is None else i["v"][:, :p].double()
    if case["kind"] == "flat":
        g = i["grads"][:, :p].double()
    elif case["kind"] == "mlp":
        g = torch.stack([_mlp_grad(case, i["theta"][r, :p], i["x"][r], i["y"][r]) for r in range(n)])
    else:
        g = torch.stack([_tf_grad(case, i["theta"][r, :p], i["x"][r], i["y"][r], r) for r in range(n)])
    own = g
    if _shared(case):
        g = g.mean(0, keepdim=True)
    opt = _opt(case)
    col = lambda v: torch.tensor(v, dtype=torch.float64, device=DEV).view(-1, 1)  # noqa: E731
    lr = col([_lr_max(dict(opt_=opt)) * r for r in _rho(n, 0.1)])
    wd = col([WDCH_BASE * r for r in _rho(n, WDCH_ALPHA)] if case.get("channels") else [WD] * n)
    t = T0 + 1
    if opt == "sgdm":
        m = MOM * m + g + wd * theta
        theta = theta - lr * m
    else:
        m = BETA1 * m + (1 - BETA1) * g
        v = BETA2 * v + (1 - BETA2) * g * g
        theta = theta * (1 - lr * wd) - lr / (1 - BETA1 ** t) * m / (torch.sqrt(v) / math.sqrt(1 - BETA2 ** t) + EPS)
    if t % case["sync"] == 0:
        theta = theta.mean(0, keepdim=True).expand(n, p)
    return _outputs(case, p, theta, m, v, own)
