"""The training rounds that this framework is run for, as measurable cases.

A case is one Session: m replicas, a model (or caller-made gradients), a data type and a synchronisation rule.  One
pass is two rounds in the paper's order -- 2 tau local steps, each round closed by the pull-back and the anchor refresh
-- so that a pass holds forward, backward, local step, pull-back and anchor average, the overlap of a refresh with the
steps that follow it, and a pull-back toward an anchor that the path itself produced.  What comes back is the state
the rounds leave: every replica, every momentum buffer, the anchor, and the gradients of the last step where the path
stores them.

The data follow the laws of `ols_inputs/generate.py` (class means plus noise; caller-made gradients N(0, 1e-2)), drawn
on the device.  `exact` runs the same rounds with plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2002_09539_amd import binding as B
from paper_2002_09539_amd.session import Session

MU = 0.9      # local momentum of every model case; least squares runs without, as its configuration does


# ------------------------------------------------------------------------------------------------------------------
# cases
# ------------------------------------------------------------------------------------------------------------------
def _mlp(name, m, dims, batch, tau, dtype, nb, alpha=0.6, **more):
    # bf16: a late phase of a learning-rate schedule.  At the first phase's 0.05 the last bit of the starting point
    # moves the momenta of the deep bf16 networks by 2e-2 within two rounds, and outputs could not be compared.
    return dict(name=name, kind="mlp", m=m, dims="-".join(map(str, dims)), batch=batch, tau=tau, dtype=dtype, nb=nb,
                alpha=alpha, gamma=0.05 if dtype == "f32" else 0.005, **more)


def _conv(name, m, channels, height, width, classes, batch, tau, dtype, batch_norm, nb=2):
    return dict(name=name, kind="conv", m=m, dims="%d-%d-%d-%d" % (channels, height, width, classes), batch=batch,
                tau=tau, dtype=dtype, batch_norm=batch_norm, nb=nb, alpha=0.6, gamma=0.05)


def listed():
    return [
        # Configuration 1, the smallest call: four workers, 131 kFLOP per worker and step; launches and latency.
        dict(name="lsq_m4", kind="lsq", m=4, d=1024, batch=32, tau=2, nb=50, alpha=0.6, gamma=0.01),
        # Configuration 2, the ordinary fp32 MLP: 16 workers with the paper's batch of 128.
        _mlp("mlp_f32_m16", 16, (3072, 512, 10), 128, 2, "f32", 24),
        # Configuration 5: many workers on a small batch, long rounds; state traffic outweighs the products.
        _mlp("mlp_f32_m64", 64, (3072, 1024, 10), 64, 8, "f32", 12, alpha=0.5),
        # A small, ragged fp32 MLP with two hidden layers: no dimension is a whole number of tiles; also the delta GEMM.
        _mlp("mlp_f32_ragged", 5, (788, 300, 124, 7), 36, 3, "f32", 4),
        # Configuration 3, the wide bf16 MLP: the largest parameter vectors (14.7 M per worker).
        _mlp("mlp_bf16_m16", 16, (3072, 2048, 2048, 2048, 10), 256, 4, "bf16", 6, alpha=0.5),
        # A small, ragged bf16 MLP.
        _mlp("mlp_bf16_ragged", 6, (1032, 520, 264, 10), 72, 2, "bf16", 4),
        # Configuration 4, caller-made gradients on a ResNet-18-sized vector: local step, step + pull-back, and the
        # refresh on its side stream (the library's default rule).
        dict(name="stream_m16", kind="stream", m=16, d=11_200_000, tau=2, rule="paper", alpha=0.6, gamma=0.1),
        # The same path with the synchronisation as one pass, on an odd parameter count and few workers.
        dict(name="stream_one_pass_odd", kind="stream", m=7, d=3_333_337, tau=2, rule="one_pass", alpha=0.6, gamma=0.1),
        # Configuration 7: the network's first residual stage with batch normalisation in fp32; the largest work.
        _conv("conv_bn_f32_m16", 16, 64, 32, 32, 10, 128, 2, "f32", True),
        # Configuration 8: the plain block with bf16 operands.
        _conv("conv_bf16_m16", 16, 64, 32, 32, 10, 128, 2, "bf16", False),
        # Configuration 9: the normalised block with bf16 operands, the residual network's own stage.
        _conv("conv_bn_bf16_m16", 16, 64, 32, 32, 10, 128, 2, "bf16", True),
        # A small normalised block with twice the channels on images whose size is no multiple of a tile.
        _conv("conv_bn_bf16_odd", 3, 128, 13, 15, 7, 20, 2, "bf16", True),
    ]


def _log_int(rng, low, high, multiple=1):
    v = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
    return max(multiple, v // multiple * multiple)


def draw(rng):
    """One more case: a path, then sizes spread over the range in which the listed ones lie."""
    kind = rng.choice(["lsq", "mlp_f32", "mlp_f32", "mlp_bf16", "mlp_bf16", "stream", "stream", "conv_f32", "conv_bf16", "conv_bf16"])
    tau = rng.choice([1, 2, 2, 3, 4, 8])
    alpha = rng.choice([0.5, 0.6])
    if kind == "lsq":
        return dict(kind="lsq", m=rng.randint(2, 16), d=_log_int(rng, 200, 20000, 4), batch=rng.randint(8, 128), tau=tau,
                    nb=8, alpha=alpha, gamma=0.002)
    if kind in ("mlp_f32", "mlp_bf16"):
        multiple = 4 if kind == "mlp_f32" else 8
        # (three narrow bf16 layers on a small batch are left out: the last bit of the start moves them by 3e-2)
        m, batch = _log_int(rng, 2, 64), _log_int(rng, 16 if kind == "mlp_f32" else 64, 256, multiple)
        hidden = [_log_int(rng, 64, 2048, multiple) for _ in range(rng.randint(1, 3 if kind == "mlp_f32" else 2))]
        dims = [_log_int(rng, 256, 3072, multiple)] + hidden + [rng.randint(2, 20)]
        while m > 2 and m * sum(a * b for a, b in zip(dims, dims[1:])) * (4 * MU + batch / 64) > 8e8:
            m //= 2
        c = _mlp("", m, dims, batch, tau, kind[4:], 3, alpha=alpha, nesterov=rng.random() < 0.8,
                 beta_z=rng.choice([0.0, 0.0, 0.7]))
        del c["name"]
        return c
    if kind == "stream":
        m = _log_int(rng, 2, 32)
        return dict(kind="stream", m=m, d=min(_log_int(rng, 20_000, 20_000_000), 180_000_000 // m), tau=tau,
                    rule=rng.choice(["paper", "paper", "one_pass", "stale", "mixing"]), alpha=alpha, gamma=0.1)
    bf16 = kind == "conv_bf16"
    batch_norm = rng.random() < 0.6
    channels = rng.choice([64, 64, 128] if bf16 or batch_norm else [16, 32, 48, 64, 64, 128])
    height, width = _log_int(rng, 6, 36), _log_int(rng, 6, 40)
    m, batch = rng.randint(1, 16), _log_int(rng, 8, 128)
    while batch > 2 and m * batch * height * width * channels * channels > (5e9 if bf16 else 2.5e9):
        batch //= 2
    c = _conv("", m, channels, height, width, rng.randint(2, 12), batch, min(tau, 3), "bf16" if bf16 else "f32", batch_norm)
    del c["name"]
    return c


def _dims(case):
    return [int(v) for v in case["dims"].split("-")]


def _params(case):
    if case["kind"] == "mlp":
        dims = _dims(case)
        return sum(a * b + b for a, b in zip(dims, dims[1:]))
    if case["kind"] == "conv":
        c, _, _, classes = _dims(case)
        return 2 * (9 * c * c + (2 if case["batch_norm"] else 1) * c) + c * classes + classes
    return case["d"]


def _mu(case):
    return 0.0 if case["kind"] == "lsq" else MU


# ------------------------------------------------------------------------------------------------------------------
# what a program has in hand before the call
# ------------------------------------------------------------------------------------------------------------------
def _inputs(case, seed):
    """Device tensors made from the seed alone: starting point, data (or gradients), targets (or labels)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(20200209 + 7919 * seed)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")  # noqa: E731
    m, d = case["m"], _params(case)
    if case["kind"] == "stream":
        ld = B.ols_row_stride(d)
        pool = torch.zeros(2, m, ld, device="cuda")
        for t in pool:
            for row in t:
                row[:d] = 0.1 * normal(d)
        return 0.1 * normal(d), pool, None
    nb, batch = case["nb"], case["batch"]
    if case["kind"] == "lsq":
        w = normal(d) / math.sqrt(d)
        A = normal(m, nb, batch, d)
        y = (A.double() @ w.double() + 0.1 * normal(m, nb, batch).double()).float()
        return torch.zeros(d, device="cuda"), A, y
    dims = _dims(case)
    if case["kind"] == "mlp":
        shape, classes = (dims[0],), dims[-1]
        x0 = torch.cat([t.reshape(-1) for a, b in zip(dims, dims[1:])
                        for t in (normal(a, b) / math.sqrt(a), 0.02 * normal(b))])
    else:
        c, h, w, classes = dims
        shape, parts = (h, w, c), []
        for _ in range(2):
            parts.append(normal(9 * c * c) / math.sqrt(9 * c))
            if case["batch_norm"]:
                parts.append(1.0 + 0.05 * normal(c))
            parts.append(0.02 * normal(c))
        x0 = torch.cat(parts + [normal(c * classes) / math.sqrt(c), torch.zeros(classes, device="cuda")])
    means = 0.5 * normal(classes, *shape)
    labels = torch.randint(0, classes, (m, nb, batch), generator=gen, device="cuda")
    X = torch.empty(m, nb, batch, *shape, device="cuda")
    for i in range(m):
        for j in range(nb):
            X[i, j] = normal(batch, *shape) + means[labels[i, j]]
    return x0, X, labels.int()


def _mixing_matrix(m):
    """Periodic averaging of the replicas blended with each replica's own model; the anchor becomes their mean."""
    w = np.zeros((m + 1, m + 1))
    w[:m, :m] = 0.5 * np.eye(m) + 0.5 / m
    w[:m, m] = 1.0 / m
    return w


class _State:
    def __init__(self, case, seed):
        self.case = case
        self.x0, self.data, self.target = _inputs(case, seed)
        m, d = case["m"], _params(case)
        stream = case["kind"] == "stream"
        s = self.session = Session(m, d, case["tau"], case["alpha"], case["gamma"], _mu(case), own_gradient=not stream)
        if stream:
            s.bind(self.data[0])
        if not case.get("nesterov", True):
            s.set_option(B.OLS_OPT_NESTEROV, 0)
        if case.get("beta_z", 0.0):
            s.set_anchor_momentum(case["beta_z"])
        if case["kind"] == "lsq":
            s.attach_lsq(case["batch"])
        elif case["kind"] == "mlp":
            s.attach_mlp(_dims(case), case["batch"], case["dtype"])
        elif case["kind"] == "conv":
            s.attach_convblock(*_dims(case), case["batch"], batch_norm=case["batch_norm"], gemm_dtype=case["dtype"])
        s.init_params(self.x0)
        rule = case.get("rule", "paper")
        if rule == "one_pass":
            s.set_option(B.OLS_OPT_FUSE_MEAN, 1)
        elif rule == "stale":
            s.set_stale_average()
        elif rule == "mixing":
            s.set_mixing(_mixing_matrix(m))
        # The two replica buffers change roles with every round after the first in which a refresh runs beside the
        # local steps; refreshes of at most 1 MiB, one-pass and mixing synchronisations run in line and never swap.
        # The stale-average rule at tau = 1 and the deferred update at tau = 1 rewrite the models in place.
        in_line = rule in ("one_pass", "mixing") or (4 * m + 4) * s.ld <= 1 << 20
        self.swaps = not in_line and (case["kind"] in ("lsq", "mlp") or case["tau"] > 1 or rule == "stale")
        if case["kind"] == "lsq":    # larger least-squares problems update through the stored gradients
            self.swaps = not in_line and (case["tau"] > 1 or (case["batch"] <= 64 and d <= 4096))
        # (A pass is two rounds, so it ends on the same buffer every time.)
        self.models = s.x_alt if self.swaps else s.x

    def __del__(self):
        if getattr(self, "session", None) is not None:
            self.session.close()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    """Two rounds.  Models step over the resident data inside the library; caller-made gradients take the call per step."""
    s, case = state.session, state.case
    steps = 2 * case["tau"]
    if case["kind"] == "stream":
        s.run(steps, lambda k: s.set_gradient(state.data[k % 2]))
    else:
        s.run_resident(steps, state.data, state.target)
    out = {"models": state.models, "anchor": s.z}
    if s.buf is not None:
        out["momentum"] = s.buf
    if case["kind"] == "conv":
        out["gradient"] = s.g
    return out


# ------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------------------------
def work(case):
    m, d, tau = case["m"], _params(case), case["tau"]
    state = 4 * m * d * (4 if _mu(case) else 2)          # parameters and momenta, read and written
    refresh = 4 * (m + 1) * d                            # replicas read, anchor written
    pull = 4 * d
    if case["kind"] == "stream":
        rule = case["rule"]
        sync = {"paper": refresh + pull, "one_pass": 2 * pull, "mixing": 8 * (m + 1) * d, "stale": 16 * m * d + pull + refresh}[rule]
        step_flops = 4 * m * d
        return dict(bytes=2 * (tau * (state + 4 * m * d) + sync), flops=2 * tau * step_flops)
    batch = case["batch"]
    if case["kind"] == "lsq":
        per_step = 4 * m * batch * (d + 1) + state
        flops = 4 * m * batch * d
    elif case["kind"] == "mlp":
        dims = _dims(case)
        pairs = list(zip(dims, dims[1:]))
        per_step = 4 * m * batch * (dims[0] + 1) + state + (2 * m * d * 2 if case["dtype"] == "bf16" else 0)
        flops = 2 * m * batch * (3 * sum(a * b for a, b in pairs) - pairs[0][0] * pairs[0][1])
    else:
        c, h, w, classes = _dims(case)
        act = m * batch * h * w * c                      # elements of one activation tensor
        size = 2 if case["dtype"] == "bf16" else 4
        # the batch read once; a1, the two deltas and the normalisations' inputs written and read again
        per_step = 4 * act + 2 * size * act * 3 + (2 * 4 * act * 2 if case["batch_norm"] else 0) + state + 8 * m * d
        flops = 5 * 2 * 9 * c * act
    return dict(bytes=2 * (tau * per_step + refresh + pull), flops=2 * tau * flops)


def tolerance(case):
    # About four times what a start moved by its last bit changes over one and two passes (momenta and gradients: fp32
    # models up to 9e-4, single entries 0.4 of the rms where one ReLU input changes sides; bf16 up to 1.5e-2 and 0.5).
    kind, dtype = case["kind"], case.get("dtype", "f32")
    if kind == "stream":
        return {"rel": 1e-6, "max": 1e-5}      # a few fp32 roundings per element
    if kind == "lsq":
        return {"rel": 1e-5, "max": 1e-4}
    if dtype == "f32":
        return {"rel": 4e-3, "max": 0.9}
    return {"rel": 3e-2, "max": 0.95}


# ------------------------------------------------------------------------------------------------------------------
# the same rounds in 64 bits
# ------------------------------------------------------------------------------------------------------------------
def _mlp_grad(dims, x, X, labels):
    """Gradients [m][d] of the mean cross-entropy at x [m][d]; X [m][B][in], labels [m][B]."""
    acts, pre, ws, off = [X], [], [], 0
    m = x.shape[0]
    for a, b in zip(dims, dims[1:]):
        w = x[:, off:off + a * b].reshape(m, a, b)
        bias = x[:, off + a * b:off + a * b + b]
        off += a * b + b
        z = torch.baddbmm(bias[:, None, :], acts[-1], w)
        ws.append(w)
        pre.append(z)
        acts.append(torch.relu(z))
    dz = torch.softmax(pre[-1], -1)
    dz.scatter_add_(2, labels.long()[..., None], torch.full_like(dz[..., :1], -1.0))
    dz /= X.shape[1]
    parts = []
    for l in range(len(ws) - 1, -1, -1):
        grads = [torch.bmm(acts[l].transpose(1, 2).contiguous(), dz).reshape(m, -1), dz.sum(1)]
        parts = grads + parts
        if l:
            dz = torch.bmm(dz, ws[l].transpose(1, 2).contiguous()) * (pre[l - 1] > 0)
    return torch.cat(parts, 1)


def _pad(t):
    return torch.nn.functional.pad(t, (0, 0, 1, 1, 1, 1))


def _conv3(t, w):
    """t [B][H][W][C], w [3][3][C][C] (input channel, output channel): cross-correlation with zero padding."""
    p, (h, wd) = _pad(t), t.shape[1:3]
    out = torch.zeros_like(t)
    for i in range(3):
        for j in range(3):
            out += p[:, i:i + h, j:j + wd] @ w[i, j]
    return out


def _conv3_dw(t, dz):
    p, (n, h, wd, c) = _pad(t), t.shape
    out = []
    for i in range(3):
        for j in range(3):
            a = p[:, i:i + h, j:j + wd].reshape(n, h * wd, c).transpose(1, 2).contiguous()
            out.append(torch.bmm(a, dz.reshape(n, h * wd, c)).sum(0))
    return torch.stack(out).reshape(3, 3, c, c)


def _conv3_dx(dz, w):
    return _conv3(dz, w.flip(0, 1).transpose(2, 3).contiguous())


def _norm(z, scale, shift):
    inv = 1.0 / torch.sqrt(z.var((0, 1, 2), unbiased=False) + float(np.float32(1e-5)))
    xhat = (z - z.mean((0, 1, 2))) * inv
    return xhat * scale + shift, xhat, inv


def _norm_back(dy, xhat, inv, scale):
    dshift, dscale = dy.sum((0, 1, 2)), (dy * xhat).sum((0, 1, 2))
    n = dy.numel() // dy.shape[-1]
    return scale * inv * (dy - dshift / n - xhat * (dscale / n)), dscale, dshift


def _conv_grad(case, x, X, labels):
    """Gradient [d] of one worker; X [B][H][W][C], labels [B]."""
    c, h, w, classes = _dims(case)
    sizes = ([9 * c * c, c, c] if case["batch_norm"] else [9 * c * c, c]) * 2 + [c * classes, classes]
    p = list(torch.split(x, sizes))
    per = len(p) // 2 - 1
    wa, wb = p[0].reshape(3, 3, c, c), p[per].reshape(3, 3, c, c)
    wh, bh = p[-2].reshape(c, classes), p[-1]
    if case["batch_norm"]:
        n1, xhat1, inv1 = _norm(_conv3(X, wa), p[1], p[2])
        a1 = torch.relu(n1)
        n2, xhat2, inv2 = _norm(_conv3(a1, wb), p[4], p[5])
    else:
        a1 = torch.relu(_conv3(X, wa) + p[1])
        n2 = _conv3(a1, wb) + p[3]
    a2 = torch.relu(n2 + X)
    pooled = a2.mean((1, 2))
    dl = torch.softmax(pooled @ wh + bh, -1)
    dl[torch.arange(len(dl), device=dl.device), labels.long()] -= 1.0
    dl /= len(dl)
    dwh, dbh = pooled.T.contiguous() @ dl, dl.sum(0)
    dz2 = (dl @ wh.T.contiguous() / (h * w))[:, None, None, :] * (a2 > 0)
    if case["batch_norm"]:
        dz2, dg2, db2 = _norm_back(dz2, xhat2, inv2, p[4])
        dz1, dg1, db1 = _norm_back(_conv3_dx(dz2, wb) * (a1 > 0), xhat1, inv1, p[1])
        parts = [_conv3_dw(X, dz1), dg1, db1, _conv3_dw(a1, dz2), dg2, db2, dwh, dbh]
    else:
        dz1 = _conv3_dx(dz2, wb) * (a1 > 0)
        parts = [_conv3_dw(X, dz1), dz1.sum((0, 1, 2)), _conv3_dw(a1, dz2), dz2.sum((0, 1, 2)), dwh, dbh]
    return torch.cat([t.reshape(-1) for t in parts])


def exact(case, seed):
    x0, data, target = _inputs(case, seed)
    m, d, tau = case["m"], _params(case), case["tau"]
    f32 = lambda v: float(np.float32(v))  # noqa: E731  (the boundary takes its rates as 32-bit floats)
    alpha, gamma, mu, beta_z = f32(case["alpha"]), f32(case["gamma"]), f32(_mu(case)), f32(case.get("beta_z", 0.0))
    rule = case.get("rule", "paper")
    z = x0.double()
    x = z.repeat(m, 1)
    buf, v, snap = torch.zeros_like(x), torch.zeros_like(z), x.clone() if rule == "stale" else None
    for k in range(2 * tau):
        if case["kind"] == "stream":
            g = data[k % 2][:, :d].double()
        else:
            X, y = data[:, k % case["nb"]].double(), target[:, k % case["nb"]]
            if case["kind"] == "lsq":
                g = torch.bmm((torch.bmm(X, x[..., None])[..., 0] - y.double())[:, None, :], X)[:, 0] / case["batch"]
            elif case["kind"] == "mlp":
                g = _mlp_grad(_dims(case), x, X, y)
            else:
                g = torch.stack([_conv_grad(case, x[i], X[i], y[i]) for i in range(m)])
        buf.mul_(mu).add_(g)
        step = torch.add(g, buf, alpha=mu) if case.get("nesterov", True) else buf
        x = torch.add(x, step if mu else g, alpha=-gamma)
        if (k + 1) % tau:
            continue
        if rule == "mixing":
            w = torch.from_numpy(_mixing_matrix(m).astype(np.float32)).to(x).double()
            both = w.T.contiguous() @ torch.cat([x, z[None]])
            x, z = both[:m].contiguous(), both[m].contiguous()
            continue
        if rule == "stale":
            x = z + (x - snap)
            snap = x.clone()
        else:
            x = x - alpha * (x - z)
        v = beta_z * v + (x.mean(0) - z)
        z = z + v
    whole = lambda t: torch.nn.functional.pad(t, (0, B.ols_row_stride(d) - d))  # noqa: E731
    out = {"models": whole(x), "anchor": whole(z)}
    if mu:
        out["momentum"] = whole(buf)
    if case["kind"] == "conv":
        out["gradient"] = whole(g)
    return out
