"""Performance cases of the W4A4 SVDQuant-style linear layer and of its offline calibration.

A case is a dict of plain values.  `kind` says what a pass does, always through the package's public entry points:

  layer    one quantised linear: quantise pass (smoothing, clipped 4-bit codes, low-rank down-projection) and GEMM
  ffn      feed-forward block: up-projection, GELU, down-projection; `fused` runs the GEMM epilogue that emits the
           down-projection's operands, otherwise the down-projection's quantise pass applies the GELU
  block    the six linears of one DiT block (q, k, v on one input, attention output, feed-forward up and down)
  hessian  calibration: the Hessian of the layer-wise objective over a batch of tokens
  gptq     calibration: the residual's 4-bit codes and scales by GPTQ
  search   calibration: clipping-ratio search over the timestep bins

Inputs are synthetic with the distributions of the workloads that bench.py times: Gaussian activations with a few
outlier channels, N(0, 0.02^2) weights, a smoothing vector from both, a low-rank pair that takes the outlier channels,
and the remainder rounded to the container's 4-bit format.  Everything is made on the GPU from the seed.
"""
import math

import torch

import paper_2605_27003_amd as svdq

DEVICE = "cuda:0"
HIDDEN, FFN = 5120, 13824                       # widths of the DiT block that bench.py times
RATIOS = (0.6, 0.7, 0.8, 0.9, 1.0)              # candidate clipping ratios of the search
TABLE = (0.8, 0.8, 0.9, 0.8, 0.7, 0.8, 0.9, 0.8)  # clipping ratio per timestep bin
BLOCK = (("q", "x_qkv", HIDDEN, HIDDEN), ("k", "x_qkv", HIDDEN, HIDDEN), ("v", "x_qkv", HIDDEN, HIDDEN),
         ("o", "x_o", HIDDEN, HIDDEN), ("up", "x_up", HIDDEN, FFN), ("down", "x_down", FFN, HIDDEN))


def listed():
    return [
        # a single small linear: what is left when the chip has nearly nothing to do (launches, host path)
        dict(name="tiny_e3m2", kind="layer", container="e3m2", M=256, K=512, N=512, r=16, step=3),
        # key / value projection of a 512-token conditioning sequence: few token tiles, weights dominate
        dict(name="cond512_e3m2", kind="layer", container="e3m2", M=512, K=HIDDEN, N=HIDDEN, r=32, step=7),
        # a short clip with a ragged token count through the widest layer, paper's MXFP4 format
        dict(name="ragged2305_mxfp4", kind="layer", container="mxfp4", M=2305, K=HIDDEN, N=FFN, r=16, step=12),
        # attention output projection of a 480p, 81-frame clip (21 x 30 x 52 tokens) in each container
        dict(name="attn480p_e3m2", kind="layer", container="e3m2", M=32760, K=HIDDEN, N=HIDDEN, r=32, step=5),
        dict(name="attn480p_nibble", kind="layer", container="nibble", M=32760, K=HIDDEN, N=HIDDEN, r=32, step=5),
        dict(name="attn480p_mxfp4", kind="layer", container="mxfp4", M=32760, K=HIDDEN, N=HIDDEN, r=32, step=5),
        # feed-forward block at 480p: GELU in the down-projection's quantise pass; and emitted by the GEMM epilogue
        dict(name="ffn480p_e3m2", kind="ffn", container="e3m2", fused=False, M=32760, K=HIDDEN, N=FFN, r=32, step=9),
        dict(name="ffn480p_mxfp4_fused", kind="ffn", container="mxfp4", fused=True, M=32760, K=HIDDEN, N=FFN, r=32, step=9),
        # one denoising step of a whole block at 720p (21 x 45 x 80 tokens), the default container: the headline workload
        dict(name="block720p_e3m2", kind="block", container="e3m2", M=75600, r=32, step=19),
        # calibration of a hidden-width layer: Hessian of one batch of tokens, GPTQ, clipping-ratio search
        dict(name="hessian_5120", kind="hessian", M=8192, K=HIDDEN),
        dict(name="gptq_5120", kind="gptq", K=HIDDEN, N=HIDDEN),
        dict(name="search_2048", kind="search", container="e3m2", M=2048, K=HIDDEN, N=HIDDEN, r=32, steps=8),
    ]


def _log(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // multiple * multiple, max(multiple, int(round(v / multiple)) * multiple))


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["ffn", "ffn", "block", "hessian", "gptq", "search"])
    step = rng.randrange(20)
    container = rng.choice(["e3m2", "e3m2", "nibble", "mxfp4", "mxfp4"])
    if kind == "layer":
        return dict(kind=kind, container=container, M=_log(rng, 1, 75600), K=_log(rng, 512, FFN, 64),
                    N=_log(rng, 512, FFN, 128), r=rng.choice([0, 16, 32, 32]), step=step)
    if kind == "ffn":
        fused = rng.random() < 0.5 and container != "nibble"
        return dict(kind=kind, container=container, fused=fused, M=_log(rng, 64, 32760), K=_log(rng, 1024, HIDDEN, 128),
                    N=_log(rng, 2048, FFN, 128), r=rng.choice([16, 32]), step=step)
    if kind == "block":
        return dict(kind=kind, container=container, M=_log(rng, 512, 32760), r=32, step=step)
    if kind == "hessian":
        return dict(kind=kind, M=_log(rng, 256, 8192), K=_log(rng, 256, HIDDEN, 64))
    if kind == "gptq":
        return dict(kind=kind, K=_log(rng, 256, HIDDEN, 64), N=_log(rng, 256, HIDDEN, 128))
    return dict(kind=kind, container=container, M=_log(rng, 256, 2048), K=_log(rng, 512, HIDDEN, 64),
                N=_log(rng, 512, HIDDEN, 128), r=rng.choice([16, 32]), steps=rng.randrange(4, 9))


# ---- inputs ------------------------------------------------------------------------------------
def _activations(g, M, K, gelu=False, outliers=True):
    """[M, K] bf16 on the GPU: N(0, 1) with 0.5 % outlier channels x 50, or the spread of a pre-GELU tensor."""
    x = torch.randn((M, K), generator=g, device=DEVICE, dtype=torch.bfloat16)
    n_out = max(1, round(0.005 * K))
    channels = torch.randperm(K, generator=g, device=DEVICE)[:n_out]
    if gelu:
        x = torch.nn.functional.gelu(x * 1.5)
    elif outliers:
        x[:, channels] *= 50.0
    return x, channels


def _int4(R):
    """[K, N] f32 -> canonical (codes [N, K/2], scales [K/64, N] f32), round to nearest per output channel and 64-group."""
    K, N = R.shape
    Rg = R.view(K // 64, 64, N)
    sw = Rg.abs().amax(dim=1) / 7.0
    q = (Rg / sw.clamp_min(1e-30)[:, None, :]).round_().clamp_(-8, 7).to(torch.int8).view(K, N).t().contiguous()
    u = q.view(torch.uint8) & 15
    return (u[:, 0::2] | (u[:, 1::2] << 4)).contiguous(), sw.contiguous()


def _mxfp4(R):
    """[K, N] f32 -> (E2M1 codes [N, K/2], E8M0 bytes [K/32, N]), blocks of 32 along K."""
    K, N = R.shape
    Rb = R.view(K // 32, 32, N)
    shared = torch.frexp(Rb.abs().amax(dim=1).clamp_min(1e-30))[1] - 3
    v = torch.ldexp(Rb, -shared[:, None, :])
    edges = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], device=R.device)
    code = torch.bucketize(v.abs(), edges).to(torch.uint8) | ((v < 0).to(torch.uint8) << 3)
    code = code.view(K, N).t().contiguous()
    return (code[:, 0::2] | (code[:, 1::2] << 4)).contiguous(), (shared + 127).to(torch.uint8).contiguous()


def _weight(g, K, N):
    return torch.randn((K, N), generator=g, device=DEVICE) * 0.02


def _linear(g, x, channels, W, r, container, colmax=None):
    """W [K, N] (overwritten) as a calibrated layer for inputs like x: smoothing vector, low-rank pair on the outlier
    channels, 4-bit residual."""
    K, N = W.shape
    if colmax is None:
        colmax = x.abs().amax(dim=0).float()
    lam = (colmax.clamp_min(1e-3) / W.abs().amax(dim=1)).sqrt()
    R = W.mul_(lam[:, None])
    L1 = L2 = None
    if r:
        L2 = torch.randn((r, N), generator=g, device=DEVICE) * 0.1
        L1 = torch.randn((K, r), generator=g, device=DEVICE) * 0.02
        n = min(r, channels.numel())
        L2[:n] = R[channels[:n]]
        L1[channels[:n], torch.arange(n, device=DEVICE)] = 1.0
        L1, L2 = L1.to(torch.bfloat16), L2.to(torch.bfloat16)
        R.addmm_(L1.float(), L2.float(), alpha=-1.0)
    qw, sw = (_mxfp4 if container == "mxfp4" else _int4)(R)
    bias = torch.randn(N, generator=g, device=DEVICE) * 0.01
    return svdq.W4A4Linear((1.0 / lam).contiguous(), L1, L2, qw, sw, bias, container=container)


def prepare(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    kind, M, K, N = case["kind"], case.get("M"), case.get("K"), case.get("N")
    s = dict(case)
    if kind == "layer":
        s["x"], ch = _activations(g, M, K)
        s["lin"] = _linear(g, s["x"], ch, _weight(g, K, N), case["r"], case["container"])
    elif kind == "ffn":
        s["x"], ch = _activations(g, M, K)
        s["up"] = _linear(g, s["x"], ch, _weight(g, K, N), case["r"], case["container"])
        # the down-projection was calibrated on activated tensors: GELU of values up to about 6
        colmax = 2.0 + 4.0 * torch.rand(N, generator=g, device=DEVICE)
        few = torch.randperm(N, generator=g, device=DEVICE)[:8]
        s["down"] = _linear(g, None, few, _weight(g, N, K), case["r"], case["container"], colmax)
    elif kind == "block":
        made = {n: _activations(g, M, k, gelu=n == "x_down") for n, k in
                (("x_qkv", HIDDEN), ("x_o", HIDDEN), ("x_up", HIDDEN), ("x_down", FFN))}
        s["x"] = {n: v[0] for n, v in made.items()}
        s["lin"] = {n: _linear(g, *made[inp], _weight(g, k, o), case["r"], case["container"]) for n, inp, k, o in BLOCK}
    elif kind == "hessian":
        s["x"], _ = _activations(g, M, K)
        s["inv_lambda"] = 0.5 + torch.rand(K, generator=g, device=DEVICE)
    elif kind == "gptq":
        # neighbouring channels share a component, so rounding errors have somewhere to go; the values are small whole
        # numbers, which makes every sum of the Hessian exact
        T = 2 * K
        z = torch.randn((T, K), generator=g, device=DEVICE)
        z += torch.randn((T, K // 8), generator=g, device=DEVICE).repeat_interleave(8, dim=1)
        X = (z * 8.0).round_().double()
        s["H"] = (X.t() @ X) / 64.0
        s["R"] = torch.randn((K, N), generator=g, device=DEVICE) * 0.02
    elif kind == "search":
        W = _weight(g, K, N)
        Wb = W.to(torch.bfloat16)
        x, ch = _activations(g, M, K)
        s["lin"] = _linear(g, x, ch, W, case["r"], case["container"])
        # the outlier channels fade along the trajectory; the reference is the full-precision layer
        s["xs"] = [x]
        for i in range(1, case["steps"]):
            x = torch.randn((M, K), generator=g, device=DEVICE, dtype=torch.bfloat16)
            x[:, ch] *= 50.0 * (1.0 - 0.8 * i / case["steps"])
            s["xs"].append(x)
        s["refs"] = [x @ Wb for x in s["xs"]]
        s["bins"] = [i * 4 // case["steps"] for i in range(case["steps"])]
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "hessian":
        return svdq.gptq_hessian(s["x"], s["inv_lambda"])
    if kind == "gptq":
        return svdq.gptq_quantize(s["R"], s["H"])
    if kind == "search":
        table, err = svdq.search_clipping_ratios(s["lin"].forward, s["xs"], s["refs"], s["bins"], 4, RATIOS)
        return err, table
    rho = svdq.alpha_lookup(TABLE, s["step"], 0, 20)
    if kind == "layer":
        return s["lin"].forward(s["x"], rho)
    if kind == "block":
        return [s["lin"][n].forward(s["x"][inp], rho) for n, inp, _, _ in BLOCK]
    up, down = s["up"], s["down"]
    if not s["fused"]:
        return down.forward(up.forward(s["x"], rho), rho, gelu=True)
    q = up.quantize(s["x"], rho)
    buffers = down.buffers(s["M"], s["x"].device)[:3]
    if s["container"] == "mxfp4":
        nq = svdq.linear_mxfp4_next(q[0], q[1], up.weights(), up.N, down.inv_lambda, rho, q[2], up.L2, up.bias,
                                    next_l1_packed=down.l1_packed, next_r=down.r, out=buffers)
    else:
        nq = svdq.linear_w4a4_e3m2_next(q[0], up.weights(), up.N, down.inv_lambda, rho, q[2], up.L2, up.bias,
                                        next_l1_packed=down.l1_packed, next_r=down.r, out=buffers)
    return down.gemm(*nq)


# ---- what a pass cannot do without -------------------------------------------------------------
def _layer_work(M, K, N, r, container, read_x=True, write_y=True):
    weight = K * N / 2 + (K * N / 32 if container == "mxfp4" else 4 * K * N / 64)
    b = weight + 2 * r * (K + N) + 4 * (K + N) + (2 * M * K if read_x else 0) + (2 * M * N if write_y else 0)
    return b, 2.0 * M * N * K + 2.0 * M * r * (K + N)


def work(case):
    kind, M, K, N = case["kind"], case.get("M"), case.get("K"), case.get("N")
    if kind == "layer":
        parts = [_layer_work(M, K, N, case["r"], case["container"])]
    elif kind == "ffn":
        parts = [_layer_work(M, K, N, case["r"], case["container"], write_y=False),
                 _layer_work(M, N, K, case["r"], case["container"], read_x=False)]
    elif kind == "block":
        parts = [_layer_work(M, k, o, case["r"], case["container"], read_x=n not in ("k", "v")) for n, _, k, o in BLOCK]
    elif kind == "hessian":
        parts = [(2 * M * K + 4 * K + 8 * K * K, float(M) * K * (K + 1))]      # one triangle
    elif kind == "gptq":
        # an inverse of a symmetric matrix, then each weight's error over the channels after it
        parts = [(4 * K * N + 8 * K * K + K * N / 2 + 4 * K * N / 64, float(K) ** 3 + float(K) * K * N)]
    else:
        b, f = _layer_work(M, K, N, case["r"], case["container"], write_y=False)
        n = len(RATIOS)
        parts = [(b + 2 * M * N, n * (f + 3.0 * M * N))] * case["steps"]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    kind = case["kind"]
    if kind == "hessian":
        return {"rel": 1e-12}                       # binary64 sums in any order
    if kind == "gptq":
        return "exact"                              # defined operation by operation
    if kind == "ffn":
        return {"rel": 1e-2}                        # a bf16 step of the hidden tensor can move a group's scale and codes
    if kind == "search":
        return {"rel": 1e-3, "max": 1e-2}           # sums of squares over bf16 outputs
    return {"rel": 2e-3, "max": 1e-2}               # bf16 outputs: half a step at random, one step at most
