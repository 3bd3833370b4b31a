"""Performance cases of the scene-flow matching framework.

Every case is a piece of work that a program hands to the framework through its
public Python entry points: the matching stage of a pair or a batch of pairs
(`PairMatcher.run`), the steps after it (region filter, sparsification, SGM
disparity fill), the paper's SIFT-PCA features and the refinement with them,
the differentiable window cost with its backward pass, the learned-feature
network's training pass and the learned matcher.  Sizes are those of the
repository's named workloads (160x96 grey pairs, 1242x375 and 1024x436 RGB
pairs, batches of 16) plus ragged ones in between.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and handles on the GPU
    run(state)          one pass; returns its outputs
    work(case)          bytes and operations a pass cannot do without
    exact(case, seed)   float64 outputs by plain torch, where they exist

Images are rendered on the GPU with the statistics of the repository's scenes:
Gaussian-smoothed noise, Voronoi segments with planar disparity and their own
motion, z-buffered forward splatting, optional occluder and salt noise.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1710_10096_amd as sff
from paper_1710_10096_amd.featnet import FeatNet, LearnedMatcher, TripletPool, images_bf16

DEV = "cuda"
TRIPLES, MARGIN = 4096, 0.5  # the training loop's defaults


# --------------------------------------------------------------------- cases

def _pair(name, H, W, C, levels, iters, fmax, dmax, batch=1, s_c=0, leaves=1):
    return dict(name=name, kind="pair", H=H, W=W, C=C, levels=levels, iters=iters, fmax=fmax, dmax=dmax,
                batch=batch, s_c=s_c, leaves=leaves)


def listed():
    return [
        # The smallest call of the stage: a grey thumbnail pair, one level; latency and launches.
        _pair("pair_160x96", 96, 160, 1, 1, 4, 32, 32),
        # The ordinary call: one KITTI-size RGB pair (the benchmark's workload).
        _pair("pair_1242x375", 375, 1242, 3, 3, 6, 256, 192),
        # Offline processing of a sequence: 16 KITTI-size pairs in one call.
        _pair("pair_1242x375_b16", 375, 1242, 3, 3, 6, 256, 192, batch=16),
        # Sintel-size pair down to interpolation seeds, with four temporal leaves at the start.
        _pair("pair_1024x436_seeds", 436, 1024, 3, 3, 6, 400, 128, s_c=150, leaves=4),
        # After the match of a KITTI-size pair: region filter, sparsification, SGM disparity and fill.
        dict(name="post_1242x375", kind="post", H=375, W=1242, C=3, levels=3, iters=6, fmax=256, dmax=192, batch=1),
        # The paper's own features (dense SIFT, PCA) of a KITTI-size pair.
        dict(name="sift_features_1242x375", kind="sift_features", H=375, W=1242, C=3, batch=1),
        # Refinement of a KITTI-size pair's fields with the paper's own cost, the workload's 6 iterations.
        dict(name="sift_match_1242x375", kind="sift_match", H=375, W=1242, C=3, fmax=256, dmax=192, iters=6, batch=1),
        # Differentiable window cost of a KITTI-size pair's matches, 32 channels: forward and backward.
        dict(name="cost_1242x375_c32", kind="cost", H=375, W=1242, fmax=256, dmax=192, channels=32, batch=1),
        # The same on two small crops with fewer channels and odd sizes, as in a training loop on crops.
        dict(name="cost_161x97_c16_b2", kind="cost", H=97, W=161, fmax=32, dmax=48, channels=16, batch=2),
        # One training pass of the learned features on a KITTI-size pair: feature maps, loss and all gradients.
        dict(name="train_1242x375", kind="train", H=375, W=1242, fmax=256, dmax=192),
        # The learned matcher on a Sintel-size pair: three network passes and the record matcher.
        dict(name="learned_1024x436", kind="learned", H=436, W=1024, levels=3, iters=6, fmax=400, dmax=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pair", "pair", "pair", "post", "sift_features", "sift_match", "cost", "cost", "train", "learned"])
    H, W = _log_int(rng, 90, 440), _log_int(rng, 150, 1250)
    fmax = rng.choice([32, 64, 256, 400])
    dmax = min(rng.choice([32, 64, 128, 192]), W - 1)
    if kind == "pair":
        # batches of at most 16 KITTI-size pairs' pixels
        batch = _log_int(rng, 1, min(16, max(1, 16 * 375 * 1242 // (H * W))))
        return dict(kind=kind, H=H, W=W, C=rng.choice([1, 2, 3, 3, 3, 4]), levels=rng.randint(1, 3) if H * W < 40000 else 3,
                    iters=rng.randint(2, 6), fmax=fmax, dmax=dmax, batch=batch, s_c=rng.choice([0, 0, 20, 150]),
                    leaves=rng.choice([1, 1, 1, 2, 4]) if batch <= 4 else 1)
    if kind == "post":
        return dict(kind=kind, H=H, W=W, C=rng.choice([1, 3, 3]), levels=3, iters=rng.randint(2, 6), fmax=fmax, dmax=dmax,
                    batch=rng.randint(1, 3))
    if kind == "sift_features":
        return dict(kind=kind, H=H, W=W, C=rng.choice([1, 3, 3]), batch=rng.randint(1, 2))
    if kind == "sift_match":
        return dict(kind=kind, H=H, W=W, C=rng.choice([1, 3, 3]), fmax=fmax, dmax=dmax, iters=rng.randint(1, 6), batch=1)
    if kind == "cost":
        return dict(kind=kind, H=H, W=W, fmax=fmax, dmax=dmax, channels=rng.choice([8, 16, 32, 32, 64]), batch=rng.randint(1, 2))
    if kind == "train":
        return dict(kind=kind, H=H, W=W, fmax=fmax, dmax=dmax)
    return dict(kind=kind, H=H, W=W, levels=rng.randint(1, 2) if H * W < 40000 else 3, iters=rng.randint(2, 6), fmax=fmax, dmax=dmax)


# -------------------------------------------------------------------- scenes

def _texture(g, H, W, C):
    """Uniform noise, Gaussian-smoothed (sigma 1.5, replicated border), stretched to 0..255 per channel."""
    a = torch.rand((C, H, W), generator=g, device=DEV, dtype=torch.float32)
    r = 6
    k = [math.exp(-0.5 * (i / 1.5) ** 2) for i in range(-r, r + 1)]
    s = sum(k)
    for dim, n in ((1, H), (2, W)):
        pos = torch.arange(n, device=DEV)
        a = sum(a.index_select(dim, (pos + i).clamp(0, n - 1)) * (k[i + r] / s) for i in range(-r, r + 1))
    lo, hi = a.amin((1, 2), keepdim=True), a.amax((1, 2), keepdim=True)
    return ((a - lo) * (255.0 / (hi - lo))).round().clamp(0, 255).to(torch.uint8).permute(1, 2, 0).contiguous()


def _splat(src, ty, tx, depth, fill):
    """Forward splat; the larger depth wins, ties to the smaller source index."""
    H, W, C = src.shape
    n = H * W
    ok = ((ty >= 0) & (ty < H) & (tx >= 0) & (tx < W)).flatten()
    idx = torch.arange(n, device=DEV)
    t = (ty * W + tx).flatten()[ok]
    key = (depth.flatten() * n + (n - 1 - idx))[ok]
    best = torch.full((n,), -1, dtype=torch.int64, device=DEV).scatter_reduce_(0, t, key, "amax")
    hit = best >= 0
    out = fill.reshape(n, C).clone()
    out[hit] = src.reshape(n, C)[n - 1 - best[hit] % n]
    return out.reshape(H, W, C)


def _scene(seed, H, W, C, fmax, dmax, salt=0.05):
    """uint8 [4][H][W][C]: l0, l1, r0, r1."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    r = np.random.default_rng(int(seed))
    nseg = int(r.integers(8, 21))
    yy, xx = torch.meshgrid(torch.arange(H, device=DEV), torch.arange(W, device=DEV), indexing="ij")
    sy, sx = r.uniform(0, H, nseg), r.uniform(0, W, nseg)
    dist = torch.stack([(yy - a) ** 2 + (xx - b) ** 2 for a, b in zip(sy, sx)])
    lab = dist.argmin(0)
    dhi = min(dmax, W // 3)
    u, v, d0, d1 = (torch.zeros((H, W), dtype=torch.int64, device=DEV) for _ in range(4))
    F, Fv = min(fmax, W // 3), min(fmax, H // 3)
    for s in range(nseg + 1):
        us, vs, dd = int(r.integers(-F, F + 1)), int(r.integers(-Fv, Fv + 1)), int(r.integers(-4, 5))
        if s < nseg:
            m = lab == s
            bx, by = r.uniform(-0.02, 0.02, 2) * dhi / 64.0
            plane = (r.uniform(0, dhi) + bx * (xx - sx[s]) + by * (yy - sy[s])).round().clamp(0, dhi).long()
        else:  # an occluder in front
            cy, cx = r.uniform(0.25, 0.75) * H, r.uniform(0.2, 0.8) * W
            m = ((yy - cy) / (0.17 * H)) ** 2 + ((xx - cx) / (0.09 * W)) ** 2 <= 1
            plane = torch.full_like(d0, dhi)
        u[m], v[m], d0[m], d1[m] = us, vs, plane[m], (plane[m] + dd).clamp(0, dhi)
    l0 = _texture(g, H, W, C)
    imgs = [l0, _splat(l0, yy + v, xx + u, d1, _texture(g, H, W, C)), _splat(l0, yy, xx - d0, d0, _texture(g, H, W, C)),
            _splat(l0, yy + v, xx + u - d1, d1, _texture(g, H, W, C))]
    for im in imgs:
        im[torch.rand((H, W), generator=g, device=DEV) < salt] = 255
    return torch.stack(imgs)


# ------------------------------------------------------------------- prepare

def _params(c, **kw):
    p = dict(H=c["H"], W=c["W"], C=c.get("C", 3), levels=c.get("levels", 3), iters=c.get("iters", 6), rs_r0=32,
             rs_samples=6, fmax=c.get("fmax", 256), dmax=c.get("dmax", 192), tau=1)
    p.update(kw)
    return p


def _inputs(c, seed):
    p, B = _params(c), c.get("batch", 1)
    imgs = torch.stack([_scene(1000 * seed + b, p["H"], p["W"], p["C"], p["fmax"], p["dmax"]) for b in range(B)])
    seeds = torch.tensor([100 * seed + b for b in range(B)], dtype=torch.int64, device=DEV)
    return p, B, imgs, seeds


def prepare(case, seed):
    p, B, imgs, seeds = _inputs(case, seed)
    k = case["kind"]
    H, W = p["H"], p["W"]
    st = dict(kind=k, p=p, imgs=imgs, seeds=seeds)
    if k == "pair":
        st["m"] = sff.PairMatcher(p, B, DEV, s_c=case["s_c"] or None, leaves=case["leaves"])
    elif k == "post":
        st["m"] = sff.PairMatcher(p, B, DEV, s_c=150)
        st["m"].run(imgs, seeds)
    elif k == "sift_features":
        st["ws"] = torch.empty(sff.sff_sift_workspace_bytes(p, 4 * B), dtype=torch.uint8, device=DEV)
        st["out"] = None
    elif k == "sift_match":
        phi = torch.zeros((B, 4, H, W, 4), dtype=torch.float32, device=DEV)
        phi[..., :3] = torch.stack([_sift_pca64(im)["phi"] for im in imgs]).float()
        st["phi"] = phi
        st["start"] = sff.PairMatcher(p, B, DEV).run(imgs, seeds)["hyp"]
        st["hyp"] = torch.empty_like(st["start"])
        st["cost"] = torch.empty((2, B, H, W), dtype=torch.float32, device=DEV)
    elif k == "cost":
        feat, hyp, w = _cost_inputs(case, seed, p, B, imgs, seeds)
        st.update(feat=feat.requires_grad_(True), hyp=hyp, w=w)
    elif k == "train":
        x, trip, net = _train_inputs(seed, p, imgs, seeds)
        st.update(x=x, trip=trip, net=net, grad=torch.zeros((4 * H * W, 32), dtype=torch.float32, device=DEV))
    else:
        st["m"] = LearnedMatcher(FeatNet(seed=seed, device=DEV), p, 1)
    return st


def _cost_inputs(case, seed, p, B, imgs, seeds):
    """Normal feature maps, the WHT matcher's forward field, the weights of the loss."""
    hyp = sff.PairMatcher(p, B, DEV).run(imgs, seeds)["hyp"][0].clone()
    g = torch.Generator(device=DEV).manual_seed(seed + 5)
    feat = torch.randn((B, 4, p["H"], p["W"], case["channels"]), generator=g, device=DEV)
    return feat, hyp, torch.rand((B, p["H"], p["W"]), generator=g, device=DEV)


def _train_inputs(seed, p, imgs, seeds):
    out = sff.PairMatcher(p, 1, DEV).run(imgs, seeds)
    valid = out["valid"][0].cpu().numpy() > 0
    valid[p["H"] // 2, p["W"] // 2] |= not valid.any()
    pool = TripletPool(out["hyp"][0, 0].cpu().numpy(), valid)
    trip = np.clip(pool.sample(np.random.default_rng(seed), TRIPLES), 0, 4 * p["H"] * p["W"] - 1)
    return images_bf16(imgs[0]), torch.from_numpy(trip).to(DEV), FeatNet(seed=seed, device=DEV)


# ----------------------------------------------------------------------- run

def run(st):
    k, p = st["kind"], st["p"]
    if k in ("pair", "learned"):
        return st["m"].run(st["imgs"], st["seeds"])
    if k == "post":
        m = st["m"]
        m.filter_and_sparsify()
        out = m.disparity_fill(st["imgs"])
        return dict(keep=m.keep, seeds=m.seeds, **out)
    if k == "sift_features":
        st["out"] = sff.sff_sift_pca(p, st["imgs"], out=st["out"], workspace=st["ws"])
        return st["out"]
    if k == "sift_match":
        st["hyp"].copy_(st["start"])  # the refinement works in place on the matcher's fields
        cost = sff.sff_match_sift(p, st["phi"], st["seeds"], st["hyp"], cost=st["cost"])
        return dict(hyp=st["hyp"], cost=cost)
    if k == "cost":
        cost = sff.MatchCost.apply(st["feat"], st["hyp"], sff.DIR_FORWARD)
        (grad,) = torch.autograd.grad(cost, st["feat"], st["w"])
        return dict(cost=cost.detach(), grad=grad)
    net = st["net"]
    wb = net.weights_bf16()
    out, acts = net.forward(st["x"], 1, keep=True, wb=wb)
    loss = sff.sff_triplet_loss(out, st["trip"], MARGIN, st["grad"], weight=1.0 / TRIPLES)
    dout = sff.sff_take_grad_bf16(st["grad"]).view(4, p["H"], p["W"], 32)
    grads = net.backward(acts, dout, 1, wb=wb)
    return dict(features=out, loss=loss, grads=grads)


# ---------------------------------------------------------------------- work

def work(case):
    """Inputs read once, outputs written once; operations of the method itself
    (descriptor distances, window sums, products), not of an implementation."""
    k, p, B = case["kind"], _params(case), case.get("batch", 1)
    H, W, C = p["H"], p["W"], p["C"]
    N = H * W
    grids = [((H + (1 << l) - 1) >> l) * ((W + (1 << l) - 1) >> l) for l in range(p["levels"])]
    feats = 32 if k == "learned" else 16 * C  # values of a descriptor

    def match_flops(ngrid, iters, per):
        return 2 * ngrid * iters * (4 + p["rs_samples"]) * per

    if k in ("pair", "learned"):
        ev = sum(match_flops(n, p["iters"], 3 * feats * 3) for n in grids)
        box = min(2 * p["fmax"] + 1, W) * min(2 * p["fmax"] + 1, H) / float(4 ** (p["levels"] - 1))
        init = 2 * grids[-1] * box * 2 * feats
        net = 0 if k == "pair" else 4 * N * p["levels"] * 2 * 9 * (3 * 32 + 3 * 32 * 32)
        out = N * (2 * (8 + 4) + 1 + 4) + (N + 4 * N / 9 if case.get("s_c") else 0)
        return dict(bytes=B * (4 * N * C + out), flops=B * (ev + init + net))
    if k == "post":  # fields, mask, error and two views in; mask, seeds, disparity and fill out; 8 path steps per disparity
        return dict(bytes=B * N * (8 + 1 + 4 + 2 * C + 1 + 4 / 9 + 2 + 1), flops=B * N * (p["dmax"] + 1) * 8 * 6)
    if k == "sift_features":  # images in, phi out; the covariance's upper half and the projection
        return dict(bytes=B * N * 4 * (C + 16), flops=B * 4 * N * (128 * 129 + 2 * 3 * 128))
    if k == "sift_match":
        return dict(bytes=B * N * (4 * 16 + 2 * (8 + 8 + 4)), flops=B * match_flops(N, p["iters"], 3 * 49 * 9))
    if k == "cost":  # maps read for the cost and for its gradient, vectors, weights; cost and gradient maps out
        cf = case["channels"]
        return dict(bytes=B * N * (3 * 16 * cf + 8 + 8), flops=B * N * 3 * 64 * cf * (3 + 6))
    flops = 2 * 9 * (3 * 32 + 3 * 32 * 32)
    # network: input, kept activations written and read, gradients through them; forward, weight and input gradients
    return dict(bytes=4 * N * (2 * 2 * 3 + 3 * 2 * 64 + 64), flops=4 * N * (2 * flops + 2 * 9 * 3 * 32 * 32))


# --------------------------------------------------------------------- exact

def exact(case, seed):
    k = case["kind"]
    if k not in ("cost", "sift_features", "train"):
        return None  # whole numbers, or 32-bit costs of the fields found
    p, B, imgs, seeds = _inputs(case, seed)
    if k == "cost":
        feat, hyp, w = _cost_inputs(case, seed, p, B, imgs, seeds)
        res = [_window_cost64(feat[b], hyp[b], w[b]) for b in range(B)]
        return dict(cost=torch.stack([r[0] for r in res]), grad=torch.stack([r[1] for r in res]))
    if k == "sift_features":
        res = [_sift_pca64(im) for im in imgs]
        out = {n: torch.stack([r[n] for r in res]) for n in ("mean", "cov", "eigval", "axes")}
        phi = torch.zeros((B, 4, p["H"], p["W"], 4), dtype=torch.float64, device=DEV)
        phi[..., :3] = torch.stack([r["phi"] for r in res])
        return dict(out, phi=phi)
    x, trip, net = _train_inputs(seed, p, imgs, seeds)
    return _train64(x, trip, net)


def _window_cost64(feat, hyp, w):
    """Squared feature distances over the 8x8 window at clamped targets, and the gradient of sum(w * cost)."""
    _, H, W, cf = feat.shape
    F = feat.double().reshape(4, H * W, cf)
    G = torch.zeros_like(F)
    yy, xx = torch.meshgrid(torch.arange(H, device=DEV), torch.arange(W, device=DEV), indexing="ij")
    u, v, d0, d1 = hyp.long().unbind(-1)
    cost = torch.zeros((H, W), dtype=torch.float64, device=DEV)
    at = lambda y, x: (y.clamp(0, H - 1) * W + x.clamp(0, W - 1)).flatten()
    for dy in range(-3, 5):
        for dx in range(-3, 5):
            q = at(yy + dy, xx + dx)
            for m, (ty, tx) in ((1, (yy + v, xx + u)), (2, (yy, xx - d0)), (3, (yy + v, xx + u - d1))):
                t = at(ty.clamp(0, H - 1) + dy, tx.clamp(0, W - 1) + dx)
                d = F[0][q] - F[m][t]
                cost += (d * d).sum(-1).view(H, W)
                d *= 2 * w.double().view(-1, 1)
                G[0].index_add_(0, q, d)
                G[m].index_add_(0, t, d, alpha=-1)
    return cost, G.view(4, H, W, cf)


def _sift_pca64(imgs):
    """Dense SIFT (4x4 cells of 3 pixels, 8 orientations), PCA over the four images: imgs uint8 [4][H][W][C]."""
    n, H, W, _ = imgs.shape
    g = imgs.double().mean(-1)
    ys, xs = torch.arange(H, device=DEV), torch.arange(W, device=DEV)
    gx = g[:, :, (xs + 1).clamp(max=W - 1)] - g[:, :, (xs - 1).clamp(min=0)]
    gy = g[:, (ys + 1).clamp(max=H - 1)] - g[:, (ys - 1).clamp(min=0)]
    pos = torch.remainder(torch.atan2(gy, gx) / (math.pi / 4), 8.0)
    lo = pos.floor()
    frac, m, b0 = pos - lo, torch.hypot(gx, gy), lo.long() % 8
    O = torch.zeros((n, H, W, 8), dtype=torch.float64, device=DEV)
    O.scatter_add_(3, b0.unsqueeze(-1), (m * (1 - frac)).unsqueeze(-1))
    O.scatter_add_(3, ((b0 + 1) % 8).unsqueeze(-1), (m * frac).unsqueeze(-1))
    ey, ex = torch.arange(-6, H + 5, device=DEV).clamp(0, H - 1), torch.arange(-6, W + 5, device=DEV).clamp(0, W - 1)
    O = O[:, ey][:, :, ex]
    cells = sum(O[:, a:a + H + 9, c:c + W + 9] for a in range(3) for c in range(3))
    f = torch.cat([cells[:, 3 * i:3 * i + H, 3 * j:3 * j + W] for i in range(4) for j in range(4)], -1).reshape(-1, 128)
    unit = lambda a: torch.where((s := a.norm(dim=-1, keepdim=True)) > 0, a / s, torch.zeros_like(a))
    f = unit(unit(f).clamp(max=0.2))
    mean = f.mean(0)
    f = f - mean
    cov = f.t().contiguous() @ f / f.shape[0]
    lam, vec = np.linalg.eigh(cov.cpu().numpy())
    axes = vec[:, ::-1][:, :3].T.copy()
    for a in axes:
        a *= np.sign(a[np.argmax(np.abs(a))])
    ax = torch.from_numpy(axes).to(DEV)
    return dict(mean=mean, cov=cov, eigval=torch.from_numpy(lam[::-1][:3].copy()).to(DEV), axes=ax,
                phi=(f @ ax.t().contiguous()).view(n, H, W, 3))


def _train64(x, trip, net):
    """The network, the triplet loss and every gradient in float64 (no intermediate rounding)."""
    n, H, W, _ = x.shape
    ps = [(t.to(torch.bfloat16) if i % 2 == 0 else t).double().requires_grad_(True) for i, t in enumerate(net.params)]
    h = x.double()
    for l in range(4):
        w, b = ps[2 * l], ps[2 * l + 1]
        hp = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1))
        h = b + sum(hp[:, ky:ky + H, kx:kx + W].reshape(n * H * W, -1) @ w[:, ky, kx].t().contiguous()
                    for ky in range(3) for kx in range(3)).view(n, H, W, 32)
        h = h.relu() if l < 3 else h
    f = h.reshape(-1, 32)[trip.long().t().contiguous()]
    a, q, r = (f / f.norm(dim=-1, keepdim=True).clamp(min=1e-12)).unbind(0)
    loss = (MARGIN + ((a - q) ** 2).sum(-1) - ((a - r) ** 2).sum(-1)).clamp(min=0)
    grads = torch.autograd.grad(loss.mean(), ps)
    return dict(features=h.detach(), loss=loss.detach(), grads=list(grads))
