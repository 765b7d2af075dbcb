"""What this framework is timed on: its calls as a user's program makes them, from one 64 x 64 product to a whole network.

Every case is a call (or the few calls of one training step of one layer) of paper_2401_14110_amd.binding on device tensors.
Operands are E4M3 codes (M4E3 where a case says so) of the distributions the layers meet: ReLU(N(0,1)) or N(0,1) activations,
He-initialised or N(0, 0.02^2) weights, scaled per tensor by a power of two that is folded into the quantizers' biases.
"""
import torch

from paper_2401_14110_amd import binding, inputs

FLOOR, RNE = binding.ROUND_FLOOR, binding.ROUND_RNE
SEQ, CHUNK16 = binding.ORDER_SEQ, binding.ORDER_CHUNK16


def _case(kind, name=None, **kw):
    """One case: the call it times and its sizes.  qp / qa: exponent bits, mantissa bits and bias (real units) of Q_prod and Q_acc."""
    c = {"kind": kind, "round": FLOOR, "order": SEQ, "acts": "relu", "qpe": 5, "qpm": 7, "qpb": 15, "qae": 4, "qam": 7, "qab": 7}
    if name is not None:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: configuration 1 of the benchmark, where launches and latency are what counts
        _case("gemm", "gemm_64x64x256_rne", M=64, N=64, K=256, acts="normal", round=RNE),
        # a classifier head: few outputs, a long chain
        _case("gemm", "fc_64x1000x2048", M=64, N=1000, K=2048),
        # attention scores of a transformer: 32 x 12 heads of 128 x 128 x 64
        _case("batched", "attention_384x128x128x64", batch=384, M=128, N=128, K=64, acts="normal"),
        # a 3 x 3 convolution in the middle of a ResNet-50, from the NHWC tensor
        _case("conv", "conv3x3_28x28x128", n=64, h=28, w=28, c=128, cout=128, k=3, stride=1, pad=1),
        # the first convolution of a ResNet on images of an odd size and an odd batch: 3 channels, K = 147
        _case("conv", "stem_37x225x223x3", n=37, h=225, w=223, c=3, cout=64, k=7, stride=2, pad=3, acts="normal"),
        # a linear layer of BERT-base, nearest-even accumulation
        _case("gemm", "bert_ffn_4096x3072x768_rne", M=4096, N=3072, K=768, acts="normal", std=0.02, round=RNE),
        # the paper's own setting: M4E3 operands with flex bias, chunks of 16, biases 10 and 12; a late ResNet-50 layer
        _case("gemm_in", "m4e3_chunk16_3136x512x4608", M=3136, N=512, K=4608, order=CHUNK16, qab=10, qpb=12),
        # one point of the accumulator-width sweep: a wide accumulator on a large square product
        _case("gemm", "wide_acc_4096x4096x4096", M=4096, N=4096, K=4096, acts="normal", std=1.0, qae=5, qam=10, qab=15),
        # the recompute call with both event planes of a linear layer
        _case("planes", "planes_4096x768x3072", M=4096, N=768, K=3072, acts="normal", std=0.02),
        # one training step of a convolution layer as a matrix product: forward, recompute, immediate / OF estimator
        _case("train_immediate", "train_immediate_12544x256x2304", M=12544, N=256, K=2304),
        # one training step of a linear layer of ragged sizes in the chunked order: forward, recompute, recursive / OF estimator
        _case("train_recursive", "train_recursive_3985x770x771", M=3985, N=770, K=771, acts="normal", std=0.02, order=CHUNK16),
        # the whole network: every convolution and the classifier of a ResNet-50 at batch 64, the headline benchmark
        _case("resnet50", "resnet50_forward_b64", batch=64),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case: any call, its sizes over the logarithm of their ranges, at most 6e10 multiply-adds (2e10 where planes are written)."""
    kind = rng.choice(["gemm", "gemm", "gemm", "conv", "conv", "gemm_in", "batched", "planes", "train_immediate", "train_recursive"])
    opt = {"acts": rng.choice(["relu", "normal"])}
    opt["round"] = rng.choice([FLOOR, FLOOR, FLOOR, RNE]) if kind in ("gemm", "gemm_in", "conv", "planes") else FLOOR
    if kind in ("gemm", "gemm_in", "conv", "batched"):
        opt["order"] = rng.choice([SEQ, SEQ, CHUNK16])
    if kind == "train_recursive":
        opt["order"] = CHUNK16
    fmt = rng.choice(["12-bit", "12-bit", "paper", "sweep"])
    if fmt == "paper":
        opt.update(qab=10, qpb=12)
    elif fmt == "sweep" and kind in ("gemm", "conv", "batched"):
        e = rng.choice([4, 5, 6])
        opt.update(qae=e, qam=rng.randint(3, 10), qab=2 ** (e - 1) - 1)
    most = 6e10 if kind in ("gemm", "gemm_in", "conv", "batched") else 2e10
    while True:
        if kind == "conv":
            k = rng.choice([1, 3, 3, 7])
            h = _log_uniform(rng, 7, 112)
            d = dict(n=_log_uniform(rng, 1, 64), h=h, w=h + rng.choice([0, 0, 1, 3]), c=rng.choice([3, 16, 64, 96, 128, 200, 256, 512]),
                     cout=rng.choice([24, 64, 100, 128, 256, 512]), k=k, stride=rng.choice([1, 1, 2]), pad=k // 2)
            size = d["n"] * d["h"] * d["w"] * d["cout"] * k * k * d["c"]
        elif kind == "batched":
            s = rng.choice([32, 64, 100, 128, 197, 256])
            d = dict(batch=_log_uniform(rng, 2, 400), M=s, N=rng.choice([s, 64]), K=rng.choice([s, 64, 80]))
            size = d["batch"] * d["M"] * d["N"] * d["K"]
        else:
            d = dict(M=_log_uniform(rng, 32, 60000), N=_log_uniform(rng, 32, 4096), K=_log_uniform(rng, 48, 4608))
            if rng.random() < 0.6:      # most layers have round sizes
                d.update(M=-(-d["M"] // 32) * 32, N=-(-d["N"] // 32) * 32, K=-(-d["K"] // 16) * 16)
            size = d["M"] * d["N"] * d["K"]
        if 2e5 <= size <= most:
            return _case(kind, **opt, **d)


# ---- inputs ---------------------------------------------------------------------------------

class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) + 1)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)


def _codes(x, in_fmt):
    """Codes and the power of two (E4M3) or the flex bias (M4E3) of a tensor."""
    x = x.double()
    return inputs.quantize_tensor_fp8(x, *in_fmt) if in_fmt else inputs.quantize_tensor(x)


def _operands(case, r, shape_a, shape_b, k, in_fmt=None):
    a = r.normal(*shape_a)
    if case["acts"] == "relu":
        a = a.clamp(min=0.0)
    b = r.normal(*shape_b) * case.get("std", (2.0 / k) ** 0.5)
    A, ta = _codes(a, in_fmt)
    B, tb = _codes(b, in_fmt)
    return A.contiguous(), ta, B.contiguous(), tb


def _formats(case, ta, tb):
    qp, qa, _ = inputs.folded_formats(ta, tb, (case["qpe"], case["qpm"], case["qpb"]), (case["qae"], case["qam"], case["qab"]), case["round"])
    return qp, qa


def prepare(case, seed):
    r, kind = _Rand(seed), case["kind"]
    if kind == "resnet50":
        acts, weights, layers = {}, {}, []
        for name, M, N, K in inputs.resnet50_gemms(batch=case["batch"], image=224):
            if (M, K) not in acts:
                a = r.normal(M, K)
                acts[M, K] = _codes(a if name == "conv1" else a.clamp(min=0.0), None)
            if (N, K) not in weights:
                weights[N, K] = _codes(r.normal(N, K) * (2.0 / K) ** 0.5, None)
            (A, ta), (B, tb) = acts[M, K], weights[N, K]
            layers.append((A, B) + _formats(case, ta, tb))
        return {"case": case, "layers": layers}
    if kind == "conv":
        k = case["k"] * case["k"] * case["c"]
        X, ta, W, tb = _operands(case, r, (case["n"], case["h"], case["w"], case["c"]), (case["cout"], case["k"], case["k"], case["c"]), k)
        qp, qa = _formats(case, ta, tb)
        return {"case": case, "A": X, "B": W, "qp": qp, "qa": qa}
    M, N, K = case["M"], case["N"], case["K"]
    if kind == "batched":
        A, ta, B, tb = _operands({**case, "std": 1.0}, r, (case["batch"], M, K), (case["batch"], N, K), K)
    elif kind == "gemm_in":
        A, fa, B, fb = _operands(case, r, (M, K), (N, K), K, in_fmt=(3, 4))
        qp, qa = (case["qpe"], case["qpm"], case["qpb"], case["round"]), (case["qae"], case["qam"], case["qab"], case["round"])
        return {"case": case, "A": A, "B": B, "qp": qp, "qa": qa, "fa": (3, 4, fa), "fb": (3, 4, fb)}
    else:
        A, ta, B, tb = _operands(case, r, (M, K), (N, K), K)
    qp, qa = _formats(case, ta, tb)
    s = {"case": case, "A": A, "B": B, "qp": qp, "qa": qa}
    if kind.startswith("train"):
        s["G"] = r.normal(M, N) * 2.0 ** -10
        s["workspace"] = torch.empty(max(256, binding.lba_grad_workspace_bytes_fast(M, N, K)), dtype=torch.uint8, device="cuda")
    return s


# ---- the calls ------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "resnet50":
        return [binding.gemm(A, B, qp, qa, order=case["order"]) for A, B, qp, qa in s["layers"]]
    A, B, qp, qa = s["A"], s["B"], s["qp"], s["qa"]
    if kind == "gemm":
        return binding.gemm(A, B, qp, qa, order=case["order"])
    if kind == "batched":
        return binding.gemm_batched(A, B, qp, qa, order=case["order"])
    if kind == "gemm_in":
        return binding.gemm_in(A, B, s["fa"], s["fb"], qp, qa, order=case["order"])
    if kind == "conv":
        return binding.conv2d(A, B, qp, qa, stride=case["stride"], pad=case["pad"], order=case["order"])
    if kind == "planes":
        return binding.gemm_bwd(A, B, qp, qa)
    if kind == "train_immediate":
        y = binding.gemm(A, B, qp, qa)
        _, of, _, ws = binding.gemm_bwd_ws(A, B, qp, qa, workspace=s["workspace"], want_c=False, want_uf=False)
        dx, dw = binding.grad_premapped(s["G"], A, B, of, ws)
        return {"y": y, "dx": dx, "dw": dw}
    if kind == "train_recursive":
        y = binding.gemm(A, B, qp, qa, order=CHUNK16)
        _, of, _, of2, _ = binding.gemm_bwd_chunked(A, B, qp, qa, want_c=False, want_uf=False)
        coef = binding.ste_plane(of, case["K"], binding.STE_RECURSIVE_OF, order=CHUNK16, of_plane2=of2)
        dx, dw = binding.grad(s["G"], A, B, binding.STE_COEF_PLANE, of_plane=coef, workspace=s["workspace"])
        return {"y": y, "dx": dx, "dw": dw}
    raise ValueError(kind)


def _conv_shape(case):
    o = lambda n: (n + 2 * case["pad"] - case["k"]) // case["stride"] + 1  # noqa: E731
    return case["n"] * o(case["h"]) * o(case["w"]), case["cout"], case["k"] * case["k"] * case["c"]


def work(case):
    """Codes read once, results written once; a multiply-add of the simulated chain and one of a gradient product are two operations each."""
    kind = case["kind"]
    if kind == "resnet50":
        g = inputs.resnet50_gemms(batch=case["batch"], image=224)
        return {"bytes": sum(M * K + N * K + 4 * M * N for _, M, N, K in g), "flops": 2 * sum(M * N * K for _, M, N, K in g)}
    M, N, K = _conv_shape(case) if kind == "conv" else (case["M"], case["N"], case["K"])
    b = case.get("batch", 1)
    read = case["n"] * case["h"] * case["w"] * case["c"] if kind == "conv" else b * M * K
    total, macs = read + b * N * K + 4 * b * M * N, b * M * N * K
    words = -(-K // 32) * M * N
    if kind == "planes":
        total += 2 * 4 * words
    if kind.startswith("train"):
        total += 4 * M * N + 4 * M * K + 4 * N * K   # G read, dX and dW written
        macs *= 4                                    # forward, recompute, dX, dW
    return {"bytes": total, "flops": 2 * macs}


def tolerance(case):
    """The chain and its event planes are defined bit for bit.  Gradients are 32-bit sums in an unspecified order: against 64 bits they
    are off by 1.2e-7 to 6e-7 (2-norm), four times that is stated."""
    return {"rel": 2.4e-6, "max": 1e-4} if case["kind"].startswith("train") else "exact"


# ---- the same results in 64 bits, in plain torch --------------------------------------------

def _values(codes, e_bits, bias):
    m_bits = 7 - e_bits
    c = torch.arange(256, dtype=torch.float64)
    s, e, m = (c >= 128), (c.long() >> m_bits) & ((1 << e_bits) - 1), c.long() & ((1 << m_bits) - 1)
    v = torch.where(e == 0, m.double() * 2.0 ** (1 - bias - m_bits), (1 + m.double() / 2 ** m_bits) * torch.exp2(e.double() - bias))
    return torch.where(s, -v, v).to(codes.device)[codes.long()]


def _quantize(x, fmt):
    """Q_{M,E,b} of a float64 tensor whose values are exact; also where it saturates and where it flushes a non-zero value."""
    e_bits, m_bits, bias, rnd = fmt
    top, low = 2.0 ** (2 ** e_bits - bias - 1) * (2 - 2.0 ** -m_bits), 2.0 ** -bias
    ax = x.abs()
    of, uf = ax >= top, ax < low
    if rnd == FLOOR:
        q = (x.view(torch.int64) & -(1 << (52 - m_bits))).view(torch.float64)
    else:
        unit = (x.view(torch.int64) & (0x7FF << 52)).view(torch.float64) * 2.0 ** -m_bits
        q = torch.where(uf, 0.0, torch.round(x / unit) * unit)
    q = q.clamp(-top, top)
    return q.masked_fill(uf, 0.0), of, uf & (x != 0)


def _chain(a, b, qp, qa, order, each=None, second=None):
    """S_K of every pair of rows of a [M, K] and b [N, K] (float64).  each(k, of, uf) / second(j, of): the event bits of a step."""
    K = a.shape[1]
    at, bt = a.t().contiguous(), b.t().contiguous()
    s = torch.zeros(a.shape[0], b.shape[0], dtype=torch.float64, device=a.device)
    t = torch.zeros_like(s)
    for k in range(K):
        p, _, pu = _quantize(at[k][:, None] * bt[k][None, :], qp)
        s, of, uf = _quantize(s + p, qa)
        if each is not None:
            each(k, of, uf | pu)
        if order == CHUNK16 and (k % 16 == 15 or k == K - 1):
            t, of, _ = _quantize(t + s, qa)
            if second is not None:
                second(k // 16, of)
            s = torch.zeros_like(s)
    return t if order == CHUNK16 else s


def _product(A, B, qp, qa, order, fa=(4, 3, 7), fb=(4, 3, 7)):
    """The chain, by blocks of rows whose intermediate tensors stay near the chip."""
    if fa == (4, 3, 7):
        a, b = _values(A, 4, 7), _values(B, 4, 7)
    else:
        a, b = _values(A, fa[0], fa[2]), _values(B, fb[0], fb[2])
    rows = max(1, (1 << 22) // b.shape[0])
    return torch.cat([_chain(x, b, qp, qa, order) for x in a.split(rows)]).float()


def exact(case, seed):
    s, kind, order = prepare(case, seed), case["kind"], case["order"]
    if kind == "resnet50":
        return None     # 54 layers in 64 bits: over 20 seconds
    A, B, qp, qa = s["A"], s["B"], s["qp"], s["qa"]
    if kind == "gemm":
        return _product(A, B, qp, qa, order)
    if kind == "batched":
        return torch.stack([_product(x, y, qp, qa, order) for x, y in zip(A, B)]) if case["batch"] * case["K"] <= 30000 else None
    if kind == "gemm_in":
        return _product(A, B, qp, qa, order, s["fa"], s["fb"])
    if kind == "conv":
        k, st, pad = case["k"], case["stride"], case["pad"]
        x = torch.nn.functional.pad(A, (0, 0, pad, pad, pad, pad))
        rows = x.unfold(1, k, st).unfold(2, k, st).permute(0, 1, 2, 4, 5, 3)        # n, oh, ow, kh, kw, c
        y = _product(rows.reshape(-1, k * k * case["c"]), B.reshape(B.shape[0], -1), qp, qa, order)
        return y.view(rows.shape[0], rows.shape[1], rows.shape[2], -1)
    M, N, K = case["M"], case["N"], case["K"]
    a, b = _values(A, 4, 7), _values(B, 4, 7)
    if kind == "planes":
        of_w, uf_w = (torch.zeros(-(-K // 32), M, N, dtype=torch.int32, device="cuda") for _ in range(2))

        def bits(k, of, uf):
            bit = 1 << (k % 32) if k % 32 < 31 else -(1 << 31)
            of_w[k // 32].bitwise_or_(of.int() * bit)
            uf_w[k // 32].bitwise_or_(uf.int() * bit)

        return _chain(a, b, qp, qa, order, bits).float(), of_w, uf_w
    g = s["G"].double()
    dx, dw = torch.zeros(K, M, dtype=torch.float64, device="cuda"), torch.zeros(K, N, dtype=torch.float64, device="cuda")

    def add(k, blocked):
        gc = g.masked_fill(blocked, 0.0)
        dx[k], dw[k] = gc @ b[:, k], gc.t() @ a[:, k]

    if kind == "train_immediate":
        y = _chain(a, b, qp, qa, order, lambda k, of, uf: add(k, of))
    else:
        first, later = [None] * K, {}
        y = _chain(a, b, qp, qa, order, lambda k, of, uf: first.__setitem__(k, of), later.__setitem__)
        blocked2 = torch.zeros(M, N, dtype=torch.bool, device="cuda")
        for k in range(K - 1, -1, -1):
            if k == K - 1 or k % 16 == 15:
                blocked2 = blocked2 | later[k // 16]
                blocked = blocked2
            blocked = blocked | first[k]
            add(k, blocked)
    return {"y": y.float(), "dx": dx.t(), "dw": dw.t()}
