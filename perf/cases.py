"""Timed cases of the sampler and of its network: what each stands for, its inputs, one pass,
the bytes and operations a pass cannot do without, and what it returns in 64-bit arithmetic.

A case is a dict of plain values.  Kinds:

  trajectory  one HMC trajectory of the density for every chain of a sampler;
  sweep       one full block sweep (density, P(k), the joint move, Nbar, bias, refresh);
  forward     the network's forward pass over one grid;
  train       one training step of the network.

`chains` lists the grids of a sampler's chains as "N x count" groups, e.g. "64x8" or
"64x8,128x6,192x2".  The survey of a group follows the shapes the benchmark uses: 8^3 to
32^3 boxes of 500 Mpc/h, 7.8125 Mpc/h voxels from 64^3 up to 192^3, 1500 Mpc/h at 256^3.
"""
import math

import numpy as np
import torch

from paper_1306_1821_amd import learned
from paper_1306_1821_amd.binding import CNN, Sampler

GRIDS = (8, 16, 32, 64, 128, 192, 256)
# leapfrog step sizes near the benchmark's and the tuned ones of the studies
EPS = {8: 0.05, 16: 0.05, 32: 0.05, 64: 0.04, 128: 0.035, 192: 0.03, 256: 0.02}
# chains of one size that a program advances together (the benchmark's batches)
MOST_CHAINS = {8: 8, 16: 8, 32: 8, 64: 8, 128: 6, 192: 2, 256: 1}


def listed():
    def sampler(name, kind, chains, c, nb, steps, **kw):
        return dict(dict(name=name, kind=kind, chains=chains, c=c, nb=nb, steps=steps, rj=False,
                         mass="plain", graph=False, tau=False, growth=False, queued=False), **kw)
    return [
        # the smallest call: one trajectory of an 8^3 box, two subsamples (a first look, unit tests)
        sampler("trajectory_8", "trajectory", "8x1", 2, 4, 20),
        # a small box sampled whole, replayed from graphs as the studies run their chains
        sampler("sweep_16", "sweep", "16x1", 2, 8, 20, rj=True, graph=True),
        # the plain method at CPU scale: four 32^3 chains for R-hat, one subsample, no joint move
        sampler("sweep_32", "sweep", "32x4", 1, 16, 20),
        # step-size tuning of eight 64^3 chains: bare trajectories, each waited for
        sampler("trajectory_64", "trajectory", "64x8", 2, 20, 30),
        # the 128^3 survey of the studies: four chains, joint move, graphs
        sampler("sweep_128", "sweep", "128x4", 4, 40, 30, rj=True, graph=True),
        # the paper's scenario: one 128^3 chain with fifteen magnitude bins
        sampler("sweep_128_bins", "sweep", "128x1", 15, 40, 30, rj=True),
        # chains under the network's mass
        sampler("learned_128", "trajectory", "128x4", 4, 40, 30, mass="learned", graph=True),
        # a size that is no power of two, trajectories queued without a host wait
        sampler("trajectory_192", "trajectory", "192x2", 3, 60, 30, queued=True),
        # sixteen chains of three sizes advancing together (one launch per size)
        sampler("sweep_mixed", "sweep", "64x8,128x6,192x2", 3, 20, 30, rj=True, graph=True),
        # the headline survey: 256^3, six subsamples, 60 shells, joint move
        sampler("sweep_256", "sweep", "256x1", 6, 60, 30, rj=True),
        # training on 128^3 draws, and the network applied to the 256^3 survey
        dict(name="train_128", kind="train", n=128),
        dict(name="forward_256", kind="forward", n=256),
    ]


def draw(rng):
    kind = rng.choice(["trajectory", "trajectory", "sweep", "sweep", "forward", "train"])
    if kind in ("forward", "train"):
        most = 256 if kind == "forward" else 128  # any multiple of 4
        return dict(kind=kind, n=4 * round(math.exp(rng.uniform(math.log(4), math.log(most // 4)))))
    if kind == "sweep" and rng.random() < 0.2:
        chains = ",".join("%dx%d" % (n, rng.randint(1, most)) for n, most in ((64, 8), (128, 5), (192, 1)))
        nb_most, c_most = 32, 4
    else:
        n = rng.choice(GRIDS)
        chains = "%dx%d" % (n, rng.randint(1, MOST_CHAINS[n]))
        nb_most, c_most = min(n // 2, 80), 6 if n == 256 else 8 if n == 192 else 15
    mass = rng.choice(["plain", "plain", "plain", "learned", "diagonal"]) if kind == "trajectory" else "plain"
    return dict(kind=kind, chains=chains, c=rng.randint(1, c_most), nb=rng.randint(3, nb_most),
                steps=rng.randint(3, 30), rj=kind == "sweep" and rng.random() < 0.7, mass=mass,
                graph=rng.random() < 0.5, tau=rng.random() < 0.2, growth=rng.random() < 0.2,
                queued=kind == "trajectory" and rng.random() < 0.3)


# ------------------------------------------------------------------ inputs
def groups(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["chains"].split(",")]


def box_of(n):
    return 500.0 if n <= 32 else 1500.0 if n == 256 else 7.8125 * n


def shape_of(k):
    """P(k) up to its amplitude, k in h/Mpc."""
    return k / (1.0 + (k / 0.02) ** 3)


def freqs(n, dev):
    f = torch.arange(n, device=dev, dtype=torch.int64)
    f = torch.where(f <= n // 2, f, f - n)
    return f[:, None, None] ** 2 + f[None, :, None] ** 2 + torch.arange(n // 2 + 1, device=dev)[None, None, :] ** 2


def weights(n, dev):
    w = torch.full((n // 2 + 1,), 2.0, dtype=torch.float64, device=dev)
    w[0] = w[n // 2] = 1.0
    return w


def field(n, box, gen, dev):
    """A Gaussian truth field of standard deviation 0.5 and the amplitude of its P(k)."""
    k = 2.0 * math.pi / box * freqs(n, dev).double().sqrt()
    p = shape_of(k)
    amp = 0.25 * box ** 3 / float((p * weights(n, dev)).sum())
    w = torch.randn((n, n, n), generator=gen, device=dev)
    dk = torch.fft.rfftn(w, norm="ortho") * (amp * p * n ** 3 / box ** 3).sqrt().float()
    dk[0, 0, 0] = 0
    return torch.fft.irfftn(dk, s=(n, n, n), norm="ortho"), amp


def geometry(n, box, gen, dev):
    """Angular mask (a cap with rings and holes cut out of it) and distance from the observer."""
    c = (torch.arange(n, device=dev) + 0.5) * (box / n) - 0.5 * box
    x, y, z = c[:, None, None], c[None, :, None], c[None, None, :]
    r = (x * x + y * y + z * z).sqrt()
    polar = torch.rad2deg(torch.arccos((z / r).clamp(-1, 1)))
    mask = polar <= (60.0 if n <= 32 else 50.47)
    if n > 32:
        for ring in (12.6, 25.2, 37.9):
            mask &= (polar - ring).abs() >= 1.0
        u = torch.rand((2, 200), generator=gen, device=dev).cpu().tolist()
        for a, b in zip(*u):
            ct = math.cos(math.radians(50.47)) * (1 - a) + a
            st, ph = math.sqrt(1 - ct * ct), 2 * math.pi * b
            mask &= (x * (st * math.cos(ph)) + y * (st * math.sin(ph)) + z * ct) / r <= math.cos(math.radians(0.5))
    return mask.float(), r


def selection(r, rs):
    rp = rs * (4.0 / 3.0) ** (2.0 / 3.0)
    return (r / rp) ** 2 * torch.exp((rp / rs) ** 1.5 - (r / rs) ** 1.5)


def survey(case, n, gen, dev):
    """One size group's survey: host arrays as a program loads them, and its truth field."""
    box, c = box_of(n), case["c"]
    delta, amp = field(n, box, gen, dev)
    mask, r = geometry(n, box, gen, dev)
    rs = 150.0 if n <= 32 else 0.3 * box
    bias = [1.0 + 0.9 * l / max(1, c - 1) for l in range(c)]
    nbar = [5.0 * 0.1 ** (l / max(1, c - 1)) for l in range(c)]
    if c > 8:  # magnitude bins: a selection of its own for each
        sel = [selection(r, rs * (0.5 + l / c)) for l in range(c)]
    else:
        sel = [selection(r, rs)] * c
    R, counts = np.empty((c, n, n, n), np.float32), np.empty((c, n, n, n), np.float32)
    for l in range(c):
        Rl = mask * sel[l]
        noise = torch.randn((n, n, n), generator=gen, device=dev)
        counts[l] = (nbar[l] * Rl * (1 + bias[l] * delta) + (nbar[l] * Rl).sqrt() * noise).cpu().numpy()
        R[l] = Rl.cpu().numpy()
    kc = math.sqrt(3.0) * (n // 2) * 2.0 * math.pi / box
    pk = [amp * shape_of((m + 0.5) * kc / case["nb"]) for m in range(case["nb"])]
    growth = (1.0 - 0.2 * r / r.max()).cpu().numpy() if case["growth"] else None
    lv = -1.386 - torch.log1p(4.0 * mask * sel[0]) + 0.2 * delta.roll(1, 0)
    return dict(n=n, box=box, nb=case["nb"], R=R, counts=counts, bias=bias, nbar=nbar, pk=pk,
                growth=growth), delta, lv


def surveys(case, seed, dev):
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    out = []
    for n, count in groups(case):
        spec, delta, lv = survey(case, n, gen, dev)
        for _ in range(count):
            out.append((dict(spec, nsteps=case["steps"], eps=EPS[n], rj=case["rj"], tau_mode=case["tau"],
                             seed=2013 + seed, chain_id=len(out)), delta, lv))
    return out


def net_inputs(n, seed, dev):
    """Network inputs (normalised data, mask, selection) and a target field."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    box = 7.8125 * n
    delta, _ = field(n, box, gen, dev)
    mask, r = geometry(n, box, gen, dev)
    sel = selection(r, 0.3 * box)
    noise = torch.randn((n, n, n), generator=gen, device=dev)
    return torch.stack([mask * (sel * delta + 0.3 * sel.sqrt() * noise), mask, sel]), delta


LR = 2e-3


def prepare(case, seed):
    dev = torch.device("cuda:0")
    if case["kind"] in ("forward", "train"):
        x, target = net_inputs(case["n"], seed, dev)
        return dict(case=case, net=CNN(learned.init_params(seed)), x=x, target=target)
    chains = surveys(case, seed, dev)
    s = Sampler([spec for spec, _, _ in chains])
    for i, (_, delta, lv) in enumerate(chains):
        s.set_state(i, delta)
        if case["mass"] != "plain":
            s.set_mass(i, lv, kind=case["mass"])
    if len(groups(case)) > 1:
        for pass_class in range(3):
            s.set_launch(pass_class, -1)  # what the autotuner picks for batches of several sizes
    if case["graph"]:
        s.use_graph(True)
    k = len(chains)
    return dict(case=case, s=s, i=0, dH=torch.zeros(k, dtype=torch.float64, device=dev),
                accepted=torch.zeros(k, dtype=torch.int32, device=dev))


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    if case["kind"] == "forward":
        mu, lv = state["net"].forward(state["x"])
        return dict(mu=mu, lv=lv)
    if case["kind"] == "train":
        loss = state["net"].train_step(state["x"], state["target"], LR)
        return dict(loss=loss, params=state["net"].params())
    s, i = state["s"], state["i"]
    state["i"] += 1
    # dH itself, a difference of two energies of the order of the number of voxels, is all
    # rounding in its last digits; the states it judges are returned whole
    if case["kind"] == "trajectory":
        names = ("delta_k", "mom_k", "grad_k", "delta_r")
        if case["queued"]:
            s.trajectory_async(i, state["dH"], state["accepted"])
            out = dict(accepted=state["accepted"])
        else:
            out = dict(accepted=s.trajectory(i)[1].astype(np.int32))
    else:
        names = ("delta_k", "grad_k", "delta_r")
        st = s.sweep(i)
        # the traces a program keeps, at the precision of the state they are drawn from
        out = {key: np.concatenate([x[key] for x in st]).astype(np.float32) for key in ("pk", "bias", "nbar")}
        out["accepted"] = np.array([[x["accepted"], x["rj_accepted"]] for x in st], np.int32)
    out["state"] = [[s.tensors(c)[name] for name in names] for c in range(len(s.chains))]
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["kind"] in ("forward", "train"):
        v = case["n"] ** 3
        macs = 27 * (3 * 16 + 2 * 16 * 16 + 16 * 2)
        if case["kind"] == "forward":  # three inputs read, two outputs written
            return dict(bytes=20.0 * v, flops=2.0 * macs * v)
        # the activations (bf16) and pre-activations (f32) of three layers of 16 channels are
        # written and read again by the backward pass
        return dict(bytes=(16.0 + 2 * 3 * 16 * 6) * v, flops=2.0 * v * (3 * macs - 27 * 3 * 16))
    bytes_, flops = 0.0, 0.0
    for n, count in groups(case):
        v, h = n ** 3, n * n * (n // 2 + 1)
        fft = 2.5 * v * math.log2(v)
        steps = case["steps"] * (0.5 if case["tau"] else 1.0)
        # a step is two real transforms and the update of delta_hat, p_hat; from 64^3 on the
        # grid is larger than a compute unit's memory and a step needs two passes over it:
        # delta_hat, p_hat and the intermediate grid twice, alpha and beta once
        b, f = 24.0 * h + 8.0 * v + (40.0 * h + 4.0 * v), 6 * fft
        step = 40.0 * v if n >= 64 else 0.0
        b += steps * step
        f += steps * (2 * fft + 20.0 * v)
        if case["mass"] != "plain":  # three more real transforms, three more fields
            b += steps * (36.0 * v if n >= 64 else 0.0)
            f += steps * 3 * fft
        if case["kind"] == "sweep":
            b += 8.0 * case["c"] * v + 16.0 * v + 24.0 * h  # R, counts, alpha, beta, the new gradient
            f += 2 * fft + 20.0 * case["c"] * v
            if case["rj"]:  # per step the scaled field forward and back, its shell products
                b += steps * (32.0 * v if n >= 64 else 0.0)
                f += steps * (2 * fft + 12.0 * v)
        bytes_ += count * b
        flops += count * f
    return dict(bytes=bytes_, flops=flops)


# ------------------------------------------------------------------ 64-bit values
def philox(block, draw_index, chain, stream, seed):
    """Philox4x32-10 words of the given blocks (Salmon et al., SC'11), int64 tensors."""
    def mul(a, m):
        lo, hi = a * (m & 0xFFFF), a * (m >> 16)
        mid = hi + (lo >> 16)
        return mid >> 16, ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)
    c = [block, torch.full_like(block, draw_index), torch.full_like(block, (chain << 8) | stream), torch.zeros_like(block)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def unit(words):
    return (words.double() + 0.5) * 2.0 ** -32


def normals(count, draw_index, chain, stream, seed, dev):
    w = philox(torch.arange((count + 3) // 4, device=dev), draw_index, chain, stream, seed)
    out = []
    for a, b in ((0, 1), (2, 3)):
        r, t = (-2.0 * unit(w[a]).log()).sqrt(), 2.0 * math.pi * unit(w[b])
        out += [r * t.cos(), r * t.sin()]
    return torch.stack(out, 1).reshape(-1)[:count]


def one_uniform(draw_index, chain, stream, seed, dev):
    return float(unit(philox(torch.zeros(1, dtype=torch.int64, device=dev), draw_index, chain, stream, seed)[0])[0])


def exact_trajectory(spec, delta, lv, mass, index, steps):
    n, dev = spec["n"], delta.device
    fwd = lambda x: torch.fft.rfftn(x, norm="ortho")  # noqa: E731
    inv = lambda x: torch.fft.irfftn(x, s=(n, n, n), norm="ortho")  # noqa: E731
    q, qmax, nb = freqs(n, dev), 3 * (n // 2) ** 2, spec["nb"]
    shell = torch.zeros_like(q)
    for m in range(1, nb):
        shell += m * m * qmax < nb * nb * q
    keep = (q > 0).double()
    w = weights(n, dev) * keep
    lam = torch.tensor(spec["pk"], dtype=torch.float64, device=dev)[shell] * n ** 3 / spec["box"] ** 3
    alpha = torch.zeros((n, n, n), dtype=torch.float64, device=dev)
    beta = torch.zeros_like(alpha)
    for R, counts, b, nbar in zip(spec["R"], spec["counts"], spec["bias"], spec["nbar"]):
        R, counts = (torch.from_numpy(a).to(dev).double() for a in (R, counts))
        alpha += b * b * nbar * R
        beta += torch.where(R > 0, b * (counts - nbar * R), 0.0)
    if spec["growth"] is not None:
        g = torch.from_numpy(spec["growth"]).to(dev).double()
        alpha, beta = alpha * g * g, beta * g
    inv_m = keep / (1.0 / lam + alpha.mean())
    sqrt_d = None
    if mass != "plain":
        v = lv.double().exp()
        sqrt_d = (v / v.mean()).sqrt()
        if mass == "diagonal":
            inv_m = keep * v.mean()

    def force(dk):
        """the momentum's force, the data gradient in k space, the field"""
        x = inv(dk)
        data = alpha * x - beta
        gk = fwd(data) * keep
        if sqrt_d is None:
            return dk / lam + gk, gk, x
        g = inv(dk / lam) + data
        return fwd(sqrt_d * (g - g.mean())) * keep, gk, x

    def drift(pk):
        return pk * inv_m if sqrt_d is None else fwd(sqrt_d * inv(pk * inv_m)) * keep

    def energy(dk, pk, x):
        k = float((w * inv_m * (pk.real ** 2 + pk.imag ** 2)).sum())
        p = float((w / lam * (dk.real ** 2 + dk.imag ** 2)).sum())
        return 0.5 * k + 0.5 * p + float(((0.5 * alpha * x - beta) * x).sum())

    seed, chain = spec["seed"], spec["chain_id"]
    dk0 = fwd(delta.double()) * keep
    root_m = torch.where(inv_m > 0, 1.0 / inv_m.clamp(min=1e-300), 0.0).sqrt()
    pk = fwd(normals(n ** 3, index, chain, 3, seed, dev).reshape(n, n, n)) * root_m
    dk, eps = dk0, spec["eps"]
    f, gk0, x0 = force(dk)
    h0 = energy(dk, pk, x0)
    pk = pk - 0.5 * eps * f
    for step in range(steps):
        dk = dk + eps * drift(pk)
        f, gk, x = force(dk)
        pk = pk - (eps if step < steps - 1 else 0.5 * eps) * f
    ok = math.log(one_uniform(index, chain, 4, seed, dev)) < -(energy(dk, pk, x) - h0)
    return ok, [dk, pk, gk, x] if ok else [dk0, pk, gk0, x0]


def layers(flat):
    out, at = [], 0
    for ci, co in ((3, 16), (16, 16), (16, 16), (16, 2)):
        out.append((flat[at:at + 27 * ci * co].reshape(27, ci, co), flat[at + 27 * ci * co:at + 27 * ci * co + co]))
        at += 27 * ci * co + co
    return out


def shifted(a, t):
    """The [n, n, n, c] view of the padded [n + 2, n + 2, n + 2, c] array that tap t reads."""
    n = a.shape[0] - 2
    x, y, z = t // 9, t // 3 % 3, t % 3
    return a[x:x + n, y:y + n, z:z + n]


def pad(a):
    return torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))


def exact_net(case, seed, dev):
    x, target = net_inputs(case["n"], seed, dev)
    flat = torch.from_numpy(learned.init_params(seed)).to(dev).double()
    net = layers(flat)
    train = case["kind"] == "train"
    acts, pre, a = [], [], x.double().permute(1, 2, 3, 0)
    for l, (W, b) in enumerate(net):
        p = pad(a)
        z = b.expand(*a.shape[:3], -1).clone()
        for t in range(27):
            z += shifted(p, t) @ W[t]
        if train:
            acts.append(a)
            pre.append(z)
        a = z * torch.special.ndtr(z) if l < 3 else z
    mu, s = a[..., 0], a[..., 1]
    if not train:
        return dict(mu=mu.contiguous(), lv=s.contiguous())
    v, d, e = target.numel(), target.double() - mu, torch.exp(-s)
    loss = float((0.5 * (d * d * e + s)).mean())
    dz = torch.stack([-d * e / v, 0.5 * (1.0 - d * d * e) / v], -1)
    grads = [None] * 4
    for l in range(3, -1, -1):
        p, flat_dz = pad(acts[l]), dz.reshape(v, -1)
        dW = torch.stack([shifted(p, t).reshape(v, -1).T @ flat_dz for t in range(27)])
        grads[l] = torch.cat([dW.reshape(-1), flat_dz.sum(0)])
        if l > 0:
            p, da = pad(dz), torch.zeros_like(acts[l])
            for t in range(27):
                da += shifted(p, 26 - t) @ net[l][0][t].T
            z = pre[l - 1]
            dz = da * (torch.special.ndtr(z) + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi))
    g = torch.cat(grads)
    return dict(loss=loss, params=flat - LR * g / (g.abs() + 1e-8))  # Adam's first step


def exact(case, seed):
    dev = torch.device("cuda:0")
    if case["kind"] in ("forward", "train"):
        return exact_net(case, seed, dev)
    if case["kind"] == "sweep":
        # a sweep chains two Metropolis tests and the rejection samplers of P, Nbar and b:
        # its end state is a random draw that follows the trajectory's, not a value of its own
        return None
    chains = surveys(case, seed, dev)
    steps = case["steps"]
    if case["tau"]:
        first = chains[0][0]
        steps = min(steps, 1 + int(one_uniform(0, first["chain_id"], 10, first["seed"], dev) * steps))
    got = [exact_trajectory(spec, delta, lv, case["mass"], 0, steps) for spec, delta, lv in chains]
    return dict(accepted=None, state=[st for _, st in got])
