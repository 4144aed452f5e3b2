"""Workloads of the likelihood library, for timing and for comparing results.

Each case is one call (or the short fixed sequence of calls) that a fitting
program makes through the package's public classes: one evaluation of the NLL
and its gradient, the Hessian at the end of a fit, a batch of production
vectors, a multi-start fit, a step of many fits, the kinematic likelihood, and
the training and screening of the surrogate network.  Inputs are the stand-in
of ``synth`` (Breit-Wigner amplitudes times Y_J^0, the |V| log-uniform law) made
on the GPU from the seed alone.  ``exact`` repeats each computation in plain
64-bit torch.
"""
import math

import numpy as np
import torch

from paper_1108_5882_amd import Context, KinContext, MultiFit
from paper_1108_5882_amd._lib import Mlp

M_LO, M_HI = 0.99, 3.0      # K+K- mass range in GeV
CHUNK = 1 << 18             # rows per step of the 64-bit reference
NET_HIDDEN, NET_BATCH = 256, 1024


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a toy fit on the K = 4 table: one evaluation is all latency
        dict(name="eval_k4_f64", op="eval", prec="f64", k=4, nd=10_000, nm=100_000, weighted=False,
             extended=False, gram=False, tune=False),
        # the headline fit: one minimiser step streams 768 MB
        dict(name="eval_k16_f32", op="eval", prec="f32", k=16, nd=1_000_000, nm=5_000_000, weighted=False,
             extended=False, gram=False, tune=True),
        # an ordinary fit with weighted MC, sizes that divide nothing, never tuned
        dict(name="eval_k23_weighted", op="eval", prec="f32", k=23, nd=77_777, nm=388_901, weighted=True,
             extended=True, gram=False, tune=False),
        # a fit starts: a new MC sample (already on the GPU), its matrix, the first evaluation
        dict(name="gram_start_k24", op="gram_start", prec="f32", k=24, nd=200_000, nm=1_000_000, weighted=True,
             extended=False),
        # second derivatives again and again at new points (Newton steps, profile scans)
        dict(name="hessian_k16", op="hessian", prec="f32", k=16, nd=1_000_000, nm=1_000_000, weighted=False,
             extended=False),
        # a fit ends on its samples: error matrix of a wide model, MC matrix included
        dict(name="errors_k37", op="errors", prec="f32", k=37, nd=100_003, nm=500_009, weighted=False,
             extended=False),
        # 256 vectors over the largest sample in one pass
        dict(name="batch_k32_v256", op="batch", k=32, nv=256, nd=2_000_000, nm=10_000_000, split=3, gram=False),
        # multi-start fit of a small sample: every iteration is a chain of short kernels
        dict(name="multistart_k8", op="multistart", k=8, nv=32, nd=4_000, nm=16_000, iters=20, polar=False,
             gram=False),
        # 24 uneven fits, four minimiser iterations together
        dict(name="many_fits_24", op="many", fits=24, lo=2_000, hi=50_000, steps=4),
        # floating masses and widths on the headline sample
        dict(name="kin_k16", op="kin", k=16, nd=1_000_000, nm=5_000_000, weighted=False, extended=False),
        # surrogate: training steps of 1024 rows on 10^5 pairs
        dict(name="train_k16", op="train", k=16, n=100_000, batch=NET_BATCH, steps=64),
        # surrogate: 10^5 candidate starts screened for the best 256
        dict(name="screen_k16", op="screen", k=16, n=100_000, top=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["eval", "eval", "eval", "gram_start", "hessian", "errors", "batch", "batch", "multistart",
                     "many", "kin", "kin", "train", "screen"])
    prec = "f64" if rng.random() < 0.3 else "f32"
    k = rng.randint(2, 48)
    nd = _log_int(rng, 2_000, 600_000)
    nm = int(nd * rng.uniform(2.0, 8.0))
    if op == "eval":
        return dict(op=op, prec=prec, k=k, nd=nd // 2, nm=nm // 2, weighted=rng.random() < 0.5,
                    extended=rng.random() < 0.3, gram=rng.random() < 0.25, tune=False)
    if op == "gram_start":
        return dict(op=op, prec=prec, k=k, nd=nd // 2, nm=nm // 2, weighted=rng.random() < 0.5,
                    extended=rng.random() < 0.3)
    if op in ("hessian", "errors"):
        return dict(op=op, prec=prec, k=k, nd=nd, nm=nd if op == "hessian" else nm // 2,
                    weighted=rng.random() < 0.5, extended=rng.random() < 0.3)
    if op == "batch":
        return dict(op=op, k=k, nv=_log_int(rng, 4, 300), nd=nd // 2, nm=nm // 2, split=rng.choice([2, 3]),
                    gram=rng.random() < 0.3)
    if op == "multistart":
        return dict(op=op, k=rng.randint(3, 24), nv=_log_int(rng, 8, 256), nd=_log_int(rng, 2_000, 100_000),
                    nm=_log_int(rng, 10_000, 300_000), iters=rng.randint(8, 24), polar=rng.random() < 0.3,
                    gram=rng.random() < 0.5)
    if op == "many":
        return dict(op=op, fits=rng.randint(4, 24), lo=1_000, hi=rng.randint(8_000, 40_000),
                    steps=rng.randint(2, 6))
    if op == "kin":
        return dict(op=op, k=rng.randint(2, 24), nd=nd, nm=nm, weighted=rng.random() < 0.5,
                    extended=rng.random() < 0.3)
    if op == "train":
        return dict(op=op, k=rng.randint(3, 32), n=rng.randint(5_000, 100_000), batch=_log_int(rng, 200, 2_048),
                    steps=rng.randint(8, 48))
    return dict(op=op, k=rng.randint(3, 32), n=_log_int(rng, 2_000, 150_000), top=_log_int(rng, 16, 512))


# ---------------------------------------------------------------- inputs (GPU)
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + 7_919 * stream + 11)
    return g


def _uniform(g, lo, hi, n):
    return lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _vectors(g, nv, k):
    """Production vectors: |V| log-uniform in [0.1, 10], phase uniform."""
    mag = 10.0 ** _uniform(g, -1.0, 1.0, (nv, k))
    ph = _uniform(g, 0.0, 2.0 * math.pi, (nv, k))
    return torch.polar(mag, ph)


def _waves(g, k):
    """Masses U[1.2, 2.8], widths U[0.03, 0.3], spins cycling through 0, 2, 4."""
    return (_uniform(g, 1.2, 2.8, k).cpu().numpy(), _uniform(g, 0.03, 0.3, k).cpu().numpy(),
            np.array([(0, 2, 4)[a % 3] for a in range(k)], dtype=np.int32))


def _y_j0(J, x):
    p0, p1 = torch.ones_like(x), x
    if J == 0:
        p1 = p0
    for n in range(1, J):
        p0, p1 = p1, ((2 * n + 1) * x * p1 - n * p0) / (n + 1)
    return math.sqrt((2 * J + 1) / (4.0 * math.pi)) * p1


def _amplitudes(m, x, waves, dtype, ld=None):
    """A[n, ld] of the events (zero columns past the waves)."""
    mass, width, spin = waves
    out = torch.zeros((m.shape[0], ld or len(mass)), dtype=dtype, device="cuda")
    real = torch.view_as_real(out)
    ys = {int(J): _y_j0(int(J), x) for J in set(spin.tolist())}
    for a in range(len(mass)):
        d, c = float(mass[a]) ** 2 - m * m, float(mass[a] * width[a])
        f = ys[int(spin[a])] / (d * d + c * c)
        real[:, a, 0] = d * f
        real[:, a, 1] = c * f
    return out


def _kinematics(seed, nd, nm, waves, v_true):
    """MC events flat in (m, cos theta); data events that follow the model at v_true."""
    g = _gen(seed, 1)
    m_mc, x_mc = _uniform(g, M_LO, M_HI, nm), _uniform(g, -1.0, 1.0, nm)
    pool_m, pool_x = _uniform(g, M_LO, M_HI, 65536), _uniform(g, -1.0, 1.0, 65536)
    z = _amplitudes(pool_m, pool_x, waves, torch.complex128) @ v_true
    cdf = torch.cumsum(z.real ** 2 + z.imag ** 2, 0)
    at = torch.searchsorted(cdf, cdf[-1] * torch.rand(nd, generator=g, device="cuda", dtype=torch.float64))
    at = at.clamp(max=65535)
    m_d = (pool_m[at] + _uniform(g, -2e-3, 2e-3, nd)).clamp(M_LO, M_HI)
    x_d = (pool_x[at] + _uniform(g, -2e-3, 2e-3, nd)).clamp(-1.0, 1.0)
    return (m_d, x_d), (m_mc, x_mc)


def _sample(case, seed, dtype, ld=None):
    """waves, data rows, MC rows, MC weights or None, N_gen, evaluation vector."""
    g = _gen(seed, 0)
    waves = _waves(g, case["k"])
    vs = _vectors(g, 2, case["k"])
    data, mc = _kinematics(seed, case["nd"], case["nm"], waves, vs[0])
    w = None
    if case.get("weighted"):
        real = torch.float32 if dtype == torch.complex64 else torch.float64
        w = _uniform(g, 0.5, 1.5, case["nm"]).to(real)
    return (waves, _amplitudes(*data, waves, dtype, ld), _amplitudes(*mc, waves, dtype, ld), w,
            1.25 * case["nm"], vs[1])


def _dtype(case):
    return torch.complex128 if case.get("prec") == "f64" else torch.complex64


def _context(case, seed):
    """A context whose samples are the caller's own arrays in the library's layout."""
    prec = case.get("prec", "f32")
    ctx = Context(0, prec)
    ld = ctx.layout_ld(case["k"])
    _, Ad, Am, w, n_gen, v = _sample(case, seed, _dtype(case), ld)
    torch.cuda.synchronize()     # the context's stream reads what the torch stream wrote
    ctx.set_amplitudes("data", Ad, borrow=True, k=case["k"])
    ctx.set_amplitudes("mc", Am, w=w, n_gen=n_gen, borrow=True, k=case["k"])
    ctx.set_mc_mode("gram" if case.get("gram") else "stream", case.get("extended", False))
    return ctx, v.cpu().numpy()


def _fit_sizes(case):
    """(N_data, K, N_MC = 5 N_data) per fit: N_data log-uniform, K uniform in 4..48."""
    g = np.random.default_rng([11, case["fits"], case["lo"], case["hi"]])
    nd = np.round(np.exp(g.uniform(math.log(case["lo"]), math.log(case["hi"]), case["fits"]))).astype(int)
    return [(int(n), int(k), 5 * int(n)) for n, k in zip(nd, g.integers(4, 49, case["fits"]))]


def _fit_inputs(case, seed):
    for f, (nd, k, nm) in enumerate(_fit_sizes(case)):
        _, Ad, Am, _, _, v = _sample(dict(k=k, nd=nd, nm=nm), 1000 * seed + f, torch.complex64)
        yield Ad, Am, v


def _net_inputs(case, seed):
    """Vectors [n, k], a network's start parameters, and the vectors' NLL on a small sample."""
    k, n = case["k"], case["n"]
    g = _gen(seed, 3)
    V = _vectors(g, n, k)
    _, Ad, Am, _, _, _ = _sample(dict(k=k, nd=256, nm=1024), seed, torch.complex128)
    V_r = torch.view_as_real(V).reshape(n, 2 * k).contiguous()
    data, mc = _parts(Ad, V), _parts(Am, V)
    nll = 1000.0 * (-torch.log(data).sum(0) + 256.0 * torch.log(mc.mean(0)))
    n_in, h = 2 * k, NET_HIDDEN
    parts = []
    for fan_in, count in ((n_in, h * n_in), (n_in, h), (h, h * h), (h, h), (h, h), (h, 1)):
        parts.append(_uniform(g, -1.0 / math.sqrt(fan_in), 1.0 / math.sqrt(fan_in), count))
    return V_r, torch.cat(parts).float().contiguous(), nll.contiguous()


def _parts(A, V):
    """|A V^T|^2 [rows, vectors]."""
    z = A @ V.T.contiguous()
    return z.real ** 2 + z.imag ** 2


# -------------------------------------------------------------- prepare and run
def prepare(case, seed):
    op = case["op"]
    s = dict(case=case)
    if op == "eval":
        s["ctx"], s["V"] = _context(case, seed)
        if case["tune"]:
            s["ctx"].autotune(reps=5)
        if case["gram"]:
            s["ctx"].nll(s["V"])       # builds the MC matrix
    elif op in ("gram_start", "errors"):
        _, s["Ad"], s["Am"], s["w"], s["n_gen"], v = _sample(case, seed, _dtype(case))
        s["V"] = v.cpu().numpy()
        s["ctx"] = Context(0, case["prec"])
        torch.cuda.synchronize()
        s["ctx"].set_amplitudes("data", s["Ad"])
    elif op == "hessian":
        s["ctx"], s["V"] = _context(case, seed)
        s["ctx"].hessian(s["V"])       # builds the MC matrix
    elif op in ("batch", "multistart"):
        s["ctx"], _ = _context(case, seed)
        s["V"] = _vectors(_gen(seed, 2), case["nv"], case["k"]).cpu().numpy()
        if op == "batch":
            s["ctx"].nll_batch(s["V"], split=case["split"])      # operand planes and workspace
        else:
            s["ctx"].nll_batch(s["V"], split=3)
    elif op == "many":
        samples, s["V0"] = [], []
        for Ad, Am, v in _fit_inputs(case, seed):
            samples.append((Ad.cpu().numpy(), Am.cpu().numpy(), None, None))
            s["V0"].append(v.cpu().numpy())
        s["fits"] = MultiFit(samples, s["V0"])
    elif op == "kin":
        g = _gen(seed, 0)
        waves = _waves(g, case["k"])
        vs = _vectors(g, 2, case["k"])
        (md, xd), (mm, xm) = _kinematics(seed, case["nd"], case["nm"], waves, vs[0])
        w = _uniform(g, 0.5, 1.5, case["nm"]).float() if case["weighted"] else None
        s["res"] = np.stack([waves[0], waves[1]], axis=1).ravel()
        s["V"] = vs[1].cpu().numpy()
        s["mx"] = torch.stack([md, xd], 1).float().contiguous(), torch.stack([mm, xm], 1).float().contiguous()
        torch.cuda.synchronize()
        s["kin"] = KinContext(waves[2])
        s["kin"].set_events("data", s["mx"][0], borrow=True)
        s["kin"].set_events("mc", s["mx"][1], w=w, n_gen=1.25 * case["nm"], borrow=True)
        s["kin"].set_mode(case["extended"])
        s["w"] = w
    else:
        s["V"], s["P"], nll = _net_inputs(case, seed)
        s["net"] = Mlp(2 * case["k"], NET_HIDDEN, max_batch=8192)
        s["net"].set_params(s["P"])
        if op == "train":
            s["X"] = s["net"].features(s["V"])
            s["t"] = s["net"].targets(nll)
            s["perm"] = _permutation(case, seed)
    return s


def _permutation(case, seed):
    g = _gen(seed, 4)
    per = case["n"] // case["batch"] * case["batch"]
    need = case["steps"] * case["batch"]
    epochs = [torch.randperm(case["n"], generator=g, device="cuda")[:per] for _ in range(-(-need // per))]
    return torch.cat(epochs)[:need].to(torch.int32).contiguous()


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "eval":
        nll, grad = s["ctx"].nll_grad(s["V"])
        return dict(nll=nll, grad=grad)
    if op == "gram_start":
        s["ctx"].set_amplitudes("mc", s["Am"], w=s["w"], n_gen=s["n_gen"])
        s["ctx"].set_mc_mode("gram", case["extended"])
        nll, grad = s["ctx"].nll_grad(s["V"])
        return dict(nll=nll, grad=grad)
    if op == "errors":
        s["ctx"].set_amplitudes("data", s["Ad"])
        s["ctx"].set_amplitudes("mc", s["Am"], w=s["w"], n_gen=s["n_gen"])
        s["ctx"].set_mc_mode("stream", case["extended"])
        return dict(hessian=s["ctx"].hessian(s["V"]))
    if op == "hessian":
        return dict(hessian=s["ctx"].hessian(s["V"]))
    if op == "batch":
        nll, grad = s["ctx"].nll_batch(s["V"], split=case["split"])
        return dict(nll=nll, grad=grad)
    if op == "multistart":
        V, nll, status, _ = s["ctx"].batch_fit(s["V"], case["iters"], polar=case["polar"])
        return dict(V=V, nll=nll, status=status)
    if op == "many":
        s["fits"].reset(s["V0"])
        s["fits"].step(case["steps"])
        V, nll, status, iters = s["fits"].get()
        return dict(V=np.concatenate(V), nll=nll, status=status, iters=iters)
    if op == "kin":
        nll, grad_v, grad_res = s["kin"].nll_grad(s["V"], s["res"])
        return dict(nll=nll, grad_v=grad_v, grad_res=grad_res)
    if op == "train":
        s["net"].set_params(s["P"])
        losses, _ = s["net"].train(s["X"], s["t"], s["perm"], case["batch"])
        return dict(losses=losses, params=s["net"].get_params())
    y = s["net"].predict(s["net"].features(s["V"]))
    return dict(y=y, best=s["net"].select(y, case["top"]))


# ------------------------------------------------------------ least work of a pass
def work(case):
    op = case["op"]
    if op in ("train", "screen"):
        n_in, h = 2 * case["k"], NET_HIDDEN
        params = h * (n_in + h + 3) + 1
        layer = 2.0 * h * (n_in + h + 1)
        if op == "train":
            rows = case["steps"] * case["batch"]
            # forward, dH1 and both weight gradients; parameters and moments in and out once
            return dict(bytes=4.0 * (rows * (n_in + 2) + 6 * params),
                        flops=rows * (2.0 * layer + 2.0 * h * h))
        return dict(bytes=case["n"] * (16.0 * case["k"] + 4.0) + 4.0 * (params + case["top"]),
                    flops=case["n"] * layer)
    if op == "many":
        rows = [(nd + nm, k) for nd, k, nm in _fit_sizes(case)]
        return dict(bytes=case["steps"] * sum(8.0 * n * k for n, k in rows),
                    flops=case["steps"] * sum(16.0 * n * k for n, k in rows))
    k, nd, nm = case["k"], case["nd"], case["nm"]
    if op == "kin":
        return dict(bytes=8.0 * (nd + nm) + (4.0 * nm if case["weighted"] else 0.0),
                    flops=(nd + nm) * (66.0 * k + 30.0))
    row = 16.0 * k if case.get("prec") == "f64" else 8.0 * k
    wb = row / (2.0 * k) * nm if case.get("weighted") else 0.0
    gram_flops = 4.0 * k * k * nm
    if op == "eval":
        rows = nd if case["gram"] else nd + nm
        return dict(bytes=rows * row + (0.0 if case["gram"] else wb), flops=16.0 * k * rows)
    if op == "gram_start":
        return dict(bytes=(nd + nm) * row + wb, flops=16.0 * k * nd + gram_flops)
    hess_flops = (4.0 * k * (k + 1) + 14.0 * k) * nd
    if op == "hessian":
        return dict(bytes=nd * row, flops=hess_flops)
    if op == "errors":
        return dict(bytes=(nd + nm) * row + wb, flops=hess_flops + gram_flops)
    rows = nd if case["gram"] else nd + nm
    passes = case["iters"] if op == "multistart" else 1
    return dict(bytes=passes * rows * 8.0 * k, flops=passes * 16.0 * k * rows * case["nv"])


# --------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    op = case["op"]
    with torch.no_grad():
        if op in ("eval", "gram_start"):
            _, Ad, Am, w, n_gen, v = _sample(case, seed, _dtype(case))
            nll, grad = _nll_grad(Ad, Am, w, n_gen, v[None], case["extended"])
            return dict(nll=float(nll[0]), grad=grad[0].cpu().numpy())
        if op in ("hessian", "errors"):
            _, Ad, Am, w, n_gen, v = _sample(case, seed, _dtype(case))
            return dict(hessian=_hessian(Ad, Am, w, n_gen, v, case["extended"]).cpu().numpy())
        if op == "batch":
            _, Ad, Am, _, n_gen, _ = _sample(case, seed, torch.complex64)
            V = _vectors(_gen(seed, 2), case["nv"], case["k"])
            nll, grad = _nll_grad(Ad, Am, None, n_gen, V, False)
            return dict(nll=nll.cpu().numpy(), grad=grad.cpu().numpy())
        if op == "kin":
            return _kin(case, seed)
        if op == "train":
            return _train(case, seed)
        if op == "screen":
            V, P, _ = _net_inputs(case, seed)
            P = _unpack(P.double(), 2 * case["k"])
            return dict(y=_forward(P, _features(V))[-1].cpu().numpy(), best=None)
    return None      # trajectories of a minimiser have no closed form


def _chunks(A, w=None):
    for r in range(0, A.shape[0], CHUNK):
        yield A[r:r + CHUNK].to(torch.complex128), None if w is None else w[r:r + CHUNK].double()


def _nll_grad(Ad, Am, w, n_gen, V, extended):
    """NLL [nv] and real gradient [nv, 2k] of the vectors V [nv, k]."""
    Vt = V.T.contiguous()
    nv, k = V.shape
    log_sum = torch.zeros(nv, dtype=torch.float64, device="cuda")
    S = torch.zeros_like(log_sum)
    G = torch.zeros((k, nv), dtype=torch.complex128, device="cuda")
    H = torch.zeros_like(G)
    for A, _ in _chunks(Ad):
        z = A @ Vt
        I = z.real ** 2 + z.imag ** 2
        log_sum += torch.log(I).sum(0)
        G += A.conj().T.resolve_conj().contiguous() @ (z / I)
    for A, wc in _chunks(Am, w):
        z = A @ Vt
        u = z if wc is None else z * wc[:, None]
        S += (u * z.conj()).real.sum(0)
        H += A.conj().T.resolve_conj().contiguous() @ u
    nd = float(Ad.shape[0])
    nll = -log_sum + (S / n_gen if extended else nd * torch.log(S / n_gen))
    g = -G + H * (1.0 / n_gen if extended else nd / S)
    return nll, 2.0 * torch.view_as_real(g.T.contiguous()).reshape(nv, 2 * k)


def _hessian(Ad, Am, w, n_gen, v, extended):
    k, nd = v.shape[0], float(Ad.shape[0])
    T = torch.zeros((k, k), dtype=torch.complex128, device="cuda")
    M = torch.zeros_like(T)
    for A, _ in _chunks(Ad):
        B = A / (A @ v)[:, None]
        T += B.T.contiguous() @ B
    for A, wc in _chunks(Am, w):
        M += A.conj().T.resolve_conj().contiguous() @ (A if wc is None else A * wc[:, None])
    M = M / n_gen

    def blocks(rr, ri, ir, ii):
        out = torch.empty((k, 2, k, 2), dtype=torch.float64, device="cuda")
        out[:, 0, :, 0], out[:, 0, :, 1], out[:, 1, :, 0], out[:, 1, :, 1] = rr, ri, ir, ii
        return out.reshape(2 * k, 2 * k)

    d2_log = blocks(-2 * T.real, 2 * T.imag, 2 * T.imag, 2 * T.real)
    d2_s = blocks(2 * M.real, -2 * M.imag, 2 * M.imag, 2 * M.real)
    if extended:
        return -d2_log + d2_s
    mv = M @ v
    S = (v.conj() * mv).sum().real
    ds = 2.0 * torch.view_as_real(mv).reshape(-1)
    return -d2_log + nd * (d2_s / S - torch.outer(ds, ds) / (S * S))


def _kin(case, seed):
    g = _gen(seed, 0)
    mass, width, spin = waves = _waves(g, case["k"])
    vs = _vectors(g, 2, case["k"])
    data, mc = _kinematics(seed, case["nd"], case["nm"], waves, vs[0])
    w = _uniform(g, 0.5, 1.5, case["nm"]).float().double() if case["weighted"] else None
    v, k = vs[1], case["k"]
    m_a, g_a = (torch.from_numpy(a).cuda() for a in (mass, width))
    n_gen = 1.25 * case["nm"]

    def sums(events, weights, is_data):
        t = torch.zeros((), dtype=torch.float64, device="cuda")
        G = torch.zeros(k, dtype=torch.complex128, device="cuda")
        R = torch.zeros((k, 2), dtype=torch.float64, device="cuda")
        for r in range(0, events[0].shape[0], CHUNK):
            m, x = (e[r:r + CHUNK].float().double() for e in events)
            y = torch.stack([_y_j0(int(J), x) for J in spin], 1)
            bw = 1.0 / torch.complex((m_a * m_a)[None] - (m * m)[:, None], -(m_a * g_a)[None].expand(m.shape[0], k))
            A = bw * y
            z = A @ v
            I = z.real ** 2 + z.imag ** 2
            c = 1.0 / I if is_data else (weights[r:r + CHUNK] if weights is not None else torch.ones_like(I))
            t += (torch.log(I) if is_data else c * I).sum()
            u = z * c
            G += A.conj().T.resolve_conj().contiguous() @ u
            e = (u.conj()[:, None] * (y * bw * bw)).sum(0) * v
            R[:, 0] += 2.0 * (e * -torch.complex(2.0 * m_a, -g_a)).real
            R[:, 1] += 2.0 * (e * torch.complex(torch.zeros_like(m_a), m_a)).real
        return t, G, R

    log_sum, G, Rd = sums(data, None, True)
    S, H, Rm = sums(mc, w, False)
    nd = float(case["nd"])
    nll = -log_sum + (S / n_gen if case["extended"] else nd * torch.log(S / n_gen))
    c = 1.0 / n_gen if case["extended"] else nd / S
    return dict(nll=float(nll), grad_v=(2.0 * torch.view_as_real(-G + c * H).reshape(-1)).cpu().numpy(),
                grad_res=(-Rd + c * Rm).reshape(-1).cpu().numpy())


def _features(V):
    """Canonical features of the rows (Re, Im interleaved), rounded to the network's input type."""
    v = torch.view_as_complex(V.reshape(V.shape[0], -1, 2).contiguous())
    v = v * (v[:, :1].conj() / v[:, :1].abs()) / v.abs().square().sum(1, keepdim=True).sqrt()
    out = torch.view_as_real(v).reshape(V.shape[0], -1).clone()
    out[:, 1] = 0.0
    return out.float().double()


def _unpack(P, n_in):
    h, out, at = NET_HIDDEN, [], 0
    for shape in ((h, n_in), (h,), (h, h), (h,), (h,), (1,)):
        n = math.prod(shape)
        out.append(P[at:at + n].reshape(shape).clone())
        at += n
    return out


def _gelu(z):
    return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _gelu_d(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _forward(P, X):
    z1 = X @ P[0].T.contiguous() + P[1]
    h1 = _gelu(z1)
    z2 = h1 @ P[2].T.contiguous() + P[3]
    h2 = _gelu(z2)
    return z1, h1, z2, h2, h2 @ P[4] + P[5]


def _train(case, seed):
    V, P, nll = _net_inputs(case, seed)
    perm = _permutation(case, seed).long()
    X = _features(V)
    t = torch.log1p(nll - nll.min()).float().double()
    P = _unpack(P.double(), 2 * case["k"])
    m1, m2 = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    losses = []
    B = case["batch"]
    for s in range(case["steps"]):
        rows = perm[s * B:(s + 1) * B]
        xb = X[rows]
        z1, h1, z2, h2, y = _forward(P, xb)
        d = y - t[rows]
        losses.append((d * d).mean())
        dy = 2.0 * d / B
        dz2 = dy[:, None] * P[4] * _gelu_d(z2)
        dz1 = (dz2 @ P[2]) * _gelu_d(z1)
        grads = [dz1.T.contiguous() @ xb, dz1.sum(0), dz2.T.contiguous() @ h1, dz2.sum(0), dy @ h2, dy.sum()[None]]
        for p, g, a, b in zip(P, grads, m1, m2):
            a.mul_(0.9).add_(0.1 * g)
            b.mul_(0.999).add_(0.001 * g * g)
            p -= 1e-3 * (a / (1.0 - 0.9 ** (s + 1))) / ((b / (1.0 - 0.999 ** (s + 1))).sqrt() + 1e-8)
    return dict(losses=torch.stack(losses).cpu().numpy(), params=torch.cat([p.reshape(-1) for p in P]).cpu().numpy())
