"""The work that users of this package have it do, as cases that can be timed and compared.

Kinds of case (the sizes are those of the layers this repository names: the 784-300-100-10 MLP, LeNet-5,
the 4096 x 4096 layer over its densities and the 9216 -> 4096 layer; `draw` takes other sizes of the same ranges):

l1      one l1-phase training step of a CSR layer, `l1_step`: forward product, CSC copy, backward product,
        dense weight gradient, proximal step and recompression
debias  one debiasing step on a fixed pattern: forward and backward products, gradient sampled on the
        pattern, values-only step, refresh of the CSC copy's values
update  the proximal update from a stored dense gradient (plain, Prox-RMSProp or Prox-ADAM) with recompression
conv    the l1-phase step of a convolution layer from its maps
lenet   forward pass of the compressed LeNet-5

The weight matrix is drawn with independent entries (or power-law row lengths), values N(0, w_std); inputs are
U[0, 1) like scaled pixels, upstream gradients N(0, 1) times the loss scale, as the repository's own generators do.
"""
import math

import torch

import paper_1905_07931_amd as L1
from paper_1905_07931_amd import synth

PRECISION = {"f32": L1.F32, "bf16x3": L1.BF16X3}
SOLVER = {"rmsprop": L1.SOLVER_RMSPROP, "adam": L1.SOLVER_ADAM}
LENET_G1 = (1, 28, 28, 5, 5)
LENET_P1 = (20, 24, 24, 2, 2, 2, 2)
LENET_G2 = (20, 12, 12, 5, 5)
LENET_P2 = (50, 8, 8, 2, 2, 2, 2)
# layers of the compressed LeNet-5: outputs, inputs, stored weights
LENET = {"conv1": (20, 25, synth.LENET5_NNZ["conv1"]), "conv2": (50, 500, synth.LENET5_NNZ["conv2"]),
         "fc1": (500, 800, synth.LENET5_NNZ["fc1"]), "fc2": (10, 500, synth.LENET5_NNZ["fc2"])}


def listed():
    return [
        # first layer of the small MLP: launches and host calls decide
        dict(name="l1_784x300_b64_d10", kind="l1", N=300, K=784, B=64, density=0.10, pattern="uniform",
             precision="f32", dy_scale=1.0, lam=1e-4, w_std=0.05),
        # a large square layer late in training, few survivors per step
        dict(name="l1_4096_b512_d5", kind="l1", N=4096, K=4096, B=512, density=0.05, pattern="uniform",
             precision="f32", dy_scale=1.0 / 512, lam=0.0865, w_std=0.1),
        # the same layer early in training, half dense, with the split-bf16 gradient
        dict(name="l1_4096_b512_d50_bf16x3", kind="l1", N=4096, K=4096, B=512, density=0.50, pattern="uniform",
             precision="bf16x3", dy_scale=1.0 / 512, lam=0.0618, w_std=0.1),
        # the largest step: 9216 -> 4096, power-law rows (the benchmark's own workload)
        dict(name="l1_9216x4096_b1024_zipf9", kind="l1", N=4096, K=9216, B=1024, density=0.09, pattern="zipf",
             precision="f32", dy_scale=1.0, lam=1e-4, w_std=0.01),
        # sizes that no tile divides, an odd batch
        dict(name="l1_3001x2049_b333_d10", kind="l1", N=2049, K=3001, B=333, density=0.10, pattern="uniform",
             precision="f32", dy_scale=1.0 / 333, lam=3e-3, w_std=0.05),
        # the proximal update with Prox-ADAM over all weights of the largest layer
        dict(name="update_adam_9216x4096", kind="update", N=4096, K=9216, density=0.09, pattern="zipf",
             solver="adam", lam=1e-4, w_std=0.01),
        # retraining on the pattern, very sparse and moderately sparse
        dict(name="debias_4096_b512_d1", kind="debias", N=4096, K=4096, B=512, density=0.01, pattern="uniform",
             dy_scale=1.0 / 512, w_std=0.1),
        dict(name="debias_4096_b512_d20", kind="debias", N=4096, K=4096, B=512, density=0.20, pattern="uniform",
             dy_scale=1.0 / 512, w_std=0.1),
        # a lowered convolution layer: few short rows, a long batch
        dict(name="debias_50x500_b16384_d10", kind="debias", N=50, K=500, B=16384, density=0.10, pattern="uniform",
             dy_scale=1.0, w_std=0.05),
        # LeNet-5's second convolution from its maps
        dict(name="conv2_l1_b256_d10", kind="conv", n_out=50, C=20, H=12, W=12, KH=5, KW=5, P=0, B=256, density=0.10),
        # inference of the compressed network: one image, and a large batch
        dict(name="lenet5_b1", kind="lenet", B=1),
        dict(name="lenet5_b1024", kind="lenet", B=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: sizes and densities over their logarithm, odd ones among them."""
    kind = rng.choice(["l1", "l1", "l1", "debias", "debias", "update", "conv", "lenet"])
    if kind == "lenet":
        return dict(kind=kind, B=_log(rng, 2, 4096))
    if kind == "conv":
        side = rng.randint(8, 24)
        k = rng.choice([3, 5])
        return dict(kind=kind, n_out=_log(rng, 16, 128), C=_log(rng, 3, 40), H=side, W=side, KH=k, KW=k,
                    P=rng.choice([0, k // 2]), B=_log(rng, 16, 256),
                    density=math.exp(rng.uniform(math.log(0.03), math.log(0.5))))
    N, K = _log(rng, 100, 4096), _log(rng, 100, 9216)
    density = math.exp(rng.uniform(math.log(0.01), math.log(0.5)))
    pattern = rng.choice(["uniform", "uniform", "zipf"])
    B = _log(rng, 32, 1024)
    if rng.random() < 0.5:  # half of the drawn batches are the even ones that loaders hand out
        B = max(32, B // 32 * 32)
    # no more products than the largest listed step has
    density = min(density, 0.09 * 4096 * 9216 * 1024 / (N * K * B))
    if kind == "update":
        return dict(kind=kind, N=N, K=K, density=density, pattern=pattern, solver=rng.choice(["plain", "rmsprop", "adam"]),
                    lam=1e-4, w_std=0.05)
    c = dict(kind=kind, N=N, K=K, B=B, density=density, pattern=pattern, dy_scale=1.0 / B, w_std=0.05)
    if kind == "l1":
        # thresholds of 0 to 3 standard deviations of the gradient: from nearly all weights kept to few
        c["lam"] = rng.choice([0.0, 1.0, 2.0, 3.0]) * math.sqrt(B / 3.0) / B
        c["precision"] = rng.choice(["f32", "f32", "bf16x3"])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _mask(g, N, K, density, pattern, nnz=None):
    """Which weights are stored: as many for every seed."""
    r = _rand(g, N, K)
    total = max(1, int(round(density * N * K))) if nnz is None else nnz
    mask = torch.zeros(N, K, dtype=torch.bool, device="cuda")
    if pattern == "uniform":
        mask.view(-1)[r.view(-1).argsort()[:total]] = True
        return mask
    lengths = torch.from_numpy(synth.zipf_row_lengths(N, K, total, 1.1)).cuda()
    lengths = lengths[torch.randperm(N, generator=g, device="cuda")]
    chosen = torch.arange(K, device="cuda").view(1, K) < lengths.view(N, 1)
    return mask.scatter_(1, r.argsort(dim=1), chosen)


def _csr(mask, dense):
    """The CSR of the weights at the mask, and the dense weights themselves."""
    N, K = mask.shape
    row_ptr = torch.zeros(N + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = mask.sum(dim=1).cumsum(0).to(torch.int32)
    at = mask.nonzero()
    nnz = at.shape[0]
    col, val = at[:, 1].to(torch.int32).contiguous(), dense[mask].contiguous()
    if nnz == 0:
        col, val = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
    return L1.CSR(N, K, row_ptr, col, val, nnz)


def _weights(g, c, N, K, nnz=None, w_std=None):
    mask = _mask(g, N, K, c.get("density"), c.get("pattern", "uniform"), nnz)
    w = _randn(g, N, K) * (c.get("w_std", 0.05) if w_std is None else w_std)
    w = torch.where(w == 0, torch.full_like(w, 1e-3), w)
    return _csr(mask, w), torch.where(mask, w, torch.zeros_like(w))


def _out(N, K):
    return L1.CSR(N, K, torch.zeros(N + 1, dtype=torch.int32, device="cuda"),
                  torch.zeros(N * K, dtype=torch.int32, device="cuda"), torch.zeros(N * K, device="cuda"), None)


def _inputs(c, seed):
    """The random inputs of a case: what prepare() hands to the package and exact() computes from."""
    g = _gen(seed)
    k = c["kind"]
    if k in ("l1", "debias"):
        W, dense = _weights(g, c, c["N"], c["K"])
        X = _rand(g, c["K"], c["B"])
        dY = _randn(g, c["N"], c["B"]) * c["dy_scale"]
        return dict(W=W, dense=dense, X=X, dY=dY)
    if k == "update":
        W, dense = _weights(g, c, c["N"], c["K"])
        G = _randn(g, c["N"], c["K"])
        s = dict(W=W, dense=dense, G=G)
        if c["solver"] != "plain":  # the state some steps into training
            s["v"] = (_randn(g, c["N"], c["K"]).square() * 0.01)
            if c["solver"] == "adam":
                s["m"] = _randn(g, c["N"], c["K"]) * 0.3
        return s
    if k == "conv":
        W, dense = _weights(g, c, c["n_out"], c["C"] * c["KH"] * c["KW"])
        geom = L1.ConvGeom(c["C"], c["H"], c["W"], c["KH"], c["KW"], 1, 1, c["P"], c["P"])
        OH, OW = geom.out_hw
        X = _rand(g, geom.in_rows, c["B"])
        dY = _randn(g, c["n_out"] * OH * OW, c["B"])
        return dict(W=W, dense=dense, X=X, dY=dY, geom=geom)
    Ws, dense = {}, {}
    for name, (n, fan_in, nnz) in LENET.items():
        Ws[name], dense[name] = _weights(g, c, n, fan_in, nnz, math.sqrt(2.0 / fan_in))
    return dict(W=Ws, dense=dense, X=_rand(g, 784, c["B"]))


ADAPTIVE_ETA = 1e-3  # the usual step of the adaptive solvers
ETA = 0.01
ADAPTIVE_T = 10      # the state's step number


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    del s["dense"]
    s["case"] = c
    new = lambda *shape: torch.zeros(*shape, device="cuda")  # noqa: E731
    if c["kind"] in ("l1", "debias"):
        N, K, B, nnz = c["N"], c["K"], c["B"], s["W"].nnz
        s["Y"], s["dX"] = new(N, B), new(K, B)
        s["csc"] = L1.CSC.empty(K, nnz, s["X"].device)
        if c["kind"] == "l1":
            s["Z"], s["out"] = new(N, K), _out(N, K)
            s["bitmap"] = L1.Bitmap.empty(N, K, s["X"].device)
        else:
            s["gv"] = new(max(nnz, 1))
            L1.csc_build(s["W"], s["csc"])  # the pattern is fixed while debiasing
    elif c["kind"] == "update":
        s["out"] = _out(c["N"], c["K"])
        if c["solver"] != "plain":
            s["state"] = L1.AdaptiveState(SOLVER[c["solver"]], s["v"], s.get("m"), t=ADAPTIVE_T)
    elif c["kind"] == "conv":
        g, n, B, nnz = s["geom"], c["n_out"], c["B"], s["W"].nnz
        OH, OW = g.out_hw
        s["Y"], s["dX"] = new(n * OH * OW, B), new(g.in_rows, B)
        s["Xcol"], s["dW"] = new(g.filter_cols, OH * OW * B), new(n, g.filter_cols)
        s["csc"], s["out"] = L1.CSC.empty(g.filter_cols, nnz, s["X"].device), _out(n, g.filter_cols)
    else:
        B = c["B"]
        s["g"] = [L1.ConvGeom(*v) for v in (LENET_G1, LENET_P1, LENET_G2, LENET_P2)]
        s["y1"], s["q1"], s["y2"], s["q2"] = new(20 * 576, B), new(20 * 144, B), new(50 * 64, B), new(800, B)
        s["h1"], s["r1"], s["z"] = new(500, B), new(500, B), new(10, B)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _row_lengths(csr):
    # the stored weights per row, which a training loop watches.  Where Z is computed by a sum, a weight at the
    # threshold may be kept by one order of summation and dropped by another, and row_ptr past it would then
    # differ throughout: the lengths say the same and differ in one place
    return csr.row_ptr[1:] - csr.row_ptr[:-1]


def run(state):
    s, c = state, state["case"]
    k = c["kind"]
    if k == "l1":
        L1.l1_step(s["W"], s["X"], s["dY"], ETA, c["lam"], Y=s["Y"], dX=s["dX"], dW=s["Z"], csc=s["csc"], out=s["out"],
                   precision=PRECISION[c["precision"]], bitmap=s["bitmap"])
        return {"Y": s["Y"], "dX": s["dX"], "Z": s["Z"], "row_lengths": _row_lengths(s["out"])}
    if k == "debias":
        W, csc = s["W"], s["csc"]
        L1.csr_spmm_fwd(W, s["X"], s["Y"])
        L1.csr_spmm_bwd_t(W, s["dY"], csc, s["dX"])
        L1.sddmm_masked_wgrad(W, s["dY"], s["X"], s["gv"])
        L1.prox_l1_step(L1.PROX_CSR, W, s["gv"], ETA, 0.0)
        L1.csc_update_vals(W, csc)
        return {"Y": s["Y"], "dX": s["dX"], "gv": s["gv"], "vals": W.vals, "vals_t": csc.vals_t}
    if k == "update":
        out = s["out"]
        if c["solver"] == "plain":
            L1.prox_l1_recompress(s["W"], s["G"], ETA, c["lam"], out=out)
            return {"row_ptr": out.row_ptr, "col_idx": out.col_idx, "vals": out.vals}
        L1.prox_adaptive_recompress(s["W"], s["G"], s["state"], ADAPTIVE_ETA, c["lam"], out=out)
        got = {"row_ptr": out.row_ptr, "col_idx": out.col_idx, "vals": out.vals, "v": s["v"]}
        if c["solver"] == "adam":
            got["m"] = s["m"]
        return got
    if k == "conv":
        g, W = s["geom"], s["W"]
        L1.csr_conv_fwd(g, W, s["X"], s["Y"])
        L1.csc_build(W, s["csc"])
        L1.csr_conv_bwd_data(g, c["n_out"], s["csc"], s["dY"], s["dX"], nnz=W.nnz)
        L1.conv_im2col(g, s["X"], s["Xcol"])
        L1.dense_wgrad(s["dY"].view(c["n_out"], -1), s["Xcol"], s["dW"])
        # no threshold (the small filter bank keeps every weight): W' comes back whole, whatever the order of dW's sums
        L1.prox_l1_recompress(W, s["dW"], ETA, 0.0, out=s["out"])
        return {"Y": s["Y"], "dX": s["dX"], "dW": s["dW"], "row_ptr": s["out"].row_ptr, "col_idx": s["out"].col_idx,
                "vals": s["out"].vals}
    g1, p1, g2, p2 = s["g"]
    W = s["W"]
    L1.csr_conv_fwd(g1, W["conv1"], s["X"], s["y1"])
    L1.maxpool_fwd(p1, s["y1"], s["q1"])
    L1.csr_conv_fwd(g2, W["conv2"], s["q1"], s["y2"])
    L1.maxpool_fwd(p2, s["y2"], s["q2"])
    L1.csr_spmm_fwd(W["fc1"], s["q2"], s["h1"])
    L1.relu_fwd(s["h1"], s["r1"])
    L1.csr_spmm_fwd(W["fc2"], s["r1"], s["z"])
    return {"logits": s["z"], "fc1": s["h1"], "pool2": s["q2"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c = case
    k = c["kind"]
    if k == "lenet":
        B = c["B"]
        macs = LENET["conv1"][2] * 576 + LENET["conv2"][2] * 64 + LENET["fc1"][2] + LENET["fc2"][2]
        maps = 784 + 2 * (20 * 576 + 20 * 144 + 50 * 64 + 800 + 500 + 500) + 10
        return {"bytes": 4.0 * maps * B + 8.0 * sum(v[2] for v in LENET.values()), "flops": 2.0 * macs * B}
    if k == "conv":
        geom = L1.ConvGeom(c["C"], c["H"], c["W"], c["KH"], c["KW"], 1, 1, c["P"], c["P"])
        OH, OW = geom.out_hw
        N, K, F = c["n_out"], geom.filter_cols, OH * OW * c["B"]
        nnz = c["density"] * N * K
        # maps in and out of both products, the lowered operand written and read, the gradient and W'
        moved = 4.0 * (2 * geom.in_rows * c["B"] + 2 * N * F + 2 * K * F + 2 * N * K) + 16.0 * nnz + 8.0 * N * K
        return {"bytes": moved, "flops": 4.0 * nnz * F + 2.0 * N * K * F}
    N, K = c["N"], c["K"]
    nnz = c["density"] * N * K
    if k == "update":
        state = {"plain": 0.0, "rmsprop": 8.0, "adam": 16.0}[c["solver"]]
        return {"bytes": (4.0 + state + 8.0) * N * K + 8.0 * nnz, "flops": 4.0 * N * K}
    B = c["B"]
    acts = 4.0 * 2 * (N + K) * B
    if k == "debias":
        # W and its CSC read by the products, gradient written and read, both copies of the values written
        return {"bytes": acts + 36.0 * nnz, "flops": 6.0 * nnz * B}
    kept = max(nnz, N * K * _kept(c))
    return {"bytes": acts + 4.0 * 2 * N * K + 8.0 * kept + 24.0 * nnz, "flops": 4.0 * nnz * B + 2.0 * N * K * B}


def _kept(c):
    """The share of unstored weights that the l1 step brings back: gradients beyond the threshold."""
    sigma = math.sqrt(c["B"] / 3.0) * c["dy_scale"]
    return math.erfc(c["lam"] / sigma / math.sqrt(2.0))


# ---------------------------------------------------------------------------
# how exact the outputs are
# ---------------------------------------------------------------------------

def tolerance(case):
    k = case["kind"]
    if k == "update":
        # no sum is involved: the step is computed in double and rounded once.  The adaptive steps hold a square
        # root and divisions, whose last bit may differ
        return "exact" if case["solver"] == "plain" else {"rel": 1e-7, "max": 1e-6, "differ": 0.0}
    if k == "l1" and case["precision"] == "bf16x3":
        # operands split into two bf16 parts: 2^-16 of the products is dropped
        return {"rel": 2e-5, "max": 4e-4, "differ": 1e-2}
    # fp32 sums in any order (6e-7 seen); a weight at the threshold changes its row's length
    return {"rel": 4e-6, "max": 1e-4, "differ": 1e-2 if k == "l1" else 0.0}


def _prox64(w, step, lam_eta):
    z = w - step
    z = torch.sign(z) * (z.abs() - lam_eta).clamp(min=0)
    return z


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def exact(case, seed):
    """The outputs of run() on these inputs, in 64 bits; None for those that are whole numbers."""
    c = case
    s = _inputs(c, seed)
    X = s["X"].double() if "X" in s else None
    k = c["kind"]
    if k in ("l1", "debias"):
        w, dY = s["dense"].double(), s["dY"].double()
        grad = dY @ X.t()
        got = {"Y": w @ X, "dX": w.t() @ dY}
        if k == "l1":
            got["Z"] = _prox64(w, _f32(ETA) * grad, _f32(ETA) * _f32(c["lam"]))
            got["row_lengths"] = None
            return got
        mask = s["dense"] != 0
        new = torch.where(mask, w - _f32(ETA) * grad, torch.zeros_like(w))
        got["gv"], got["vals"] = grad[mask], new[mask]
        got["vals_t"] = new.t()[mask.t()]
        return got
    if k == "update":
        return _exact_update(c, s)
    if k == "conv":
        g, n, B = s["geom"], c["n_out"], c["B"]
        OH, OW = g.out_hw
        col = _lowered(X, c["C"], c["H"], c["W"], c["KH"], c["P"])
        w, dY = s["dense"].double(), s["dY"].double().view(n, -1)
        # gradient to the maps: the lowered gradient summed back where each of its rows came from
        back = (w.t() @ dY).view(c["C"] * c["KH"] * c["KW"], OH * OW, B).permute(2, 0, 1).contiguous()
        dX = torch.nn.functional.fold(back, (c["H"], c["W"]), (c["KH"], c["KW"]), padding=c["P"])
        dW = dY @ col.t()
        return {"Y": (w @ col).view(-1, B), "dX": dX.reshape(B, -1).t().contiguous(), "dW": dW, "row_ptr": None,
                "col_idx": None, "vals": (w - _f32(ETA) * dW).reshape(-1)}
    B, d = c["B"], {name: v.double() for name, v in s["dense"].items()}

    def layer(w, x, ch, side):
        out = side - 4
        y = (w @ _lowered(x, ch, side, side, 5, 0)).view(w.shape[0], out, out, B)
        return torch.nn.functional.max_pool2d(y.permute(3, 0, 1, 2).contiguous(), 2).permute(1, 2, 3, 0).reshape(-1, B)

    q1 = layer(d["conv1"], X, 1, 28)
    q2 = layer(d["conv2"], q1, 20, 12)
    h1 = d["fc1"] @ q2
    return {"logits": d["fc2"] @ h1.clamp(min=0), "fc1": h1, "pool2": q2}


def _lowered(X, C, H, W, k, pad):
    """[C*k*k][OH*OW*B] from maps [C*H*W][B]."""
    B = X.shape[1]
    x = X.t().reshape(B, C, H, W)
    u = torch.nn.functional.unfold(x, (k, k), padding=pad)  # [B][C*k*k][OH*OW]
    return u.permute(1, 2, 0).reshape(C * k * k, -1)


def _exact_update(c, s):
    w, G = s["dense"].double(), s["G"].double()
    got = {}
    if c["solver"] == "plain":
        z = _prox64(w, _f32(ETA) * G, _f32(ETA) * _f32(c["lam"]))
    else:
        b1, b2, eps, eta = _f32(0.9), _f32(0.999), _f32(1e-8), _f32(ADAPTIVE_ETA)
        v = (b2 * s["v"].double() + (1 - b2) * G * G).float().double()
        got["v"] = v
        if c["solver"] == "adam":
            m = (b1 * s["m"].double() + (1 - b1) * G).float().double()
            got["m"] = m
            u = (m / (1 - b1 ** ADAPTIVE_T)) / ((v / (1 - b2 ** ADAPTIVE_T)).sqrt() + eps)
        else:
            u = G / (v.sqrt() + eps)
        z = _prox64(w, eta * u, eta * _f32(c["lam"]))
    keep = z.float() != 0
    vals = torch.zeros(c["N"] * c["K"], dtype=torch.float64, device="cuda")
    kept = z[keep]
    vals[:kept.numel()] = kept
    got.update(row_ptr=None, col_idx=None, vals=vals)
    return got
