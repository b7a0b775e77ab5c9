"""The work that is timed: frame steps, batches, differentiation and the
centralised solver through the package's public entry points.

A case is a frame (or a batch of frames, or an unrolled clip) handed to an
object that a tracking program holds: keyframe set, earlier frames tracked,
the camera moving by a fraction of a pixel per frame, as at video rate. The
images are rendered from the seed: a slanted textured surface about one metre
away, seen by the keyframe camera and by moving target cameras, with a little
sensor noise. Sizes are those of the repository's own sequences (32x24,
128x96, 256x256, 320x240, 640x480, up to 1920x1080) and odd ones between.

exact() evaluates the same model in 64 bits with torch (no FP32 planes between
iterations): the synchronous iteration on the grid and on the quadtree, its
derivative by torch.autograd, and the centralised normal equations.
"""

import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

import paper_2606_03989_amd as pv

# ---------------------------------------------------------------------------
# the cases


def listed():
    # sigma_P: the weakest prior whose first iterations after a keyframe stay calm, narrower for longer focal lengths
    return [
        # the smallest call: a 32x24 pair on host arrays, 50 iterations (latency and launches)
        dict(name="frame_32x24", kind="track", H=24, W=32, iters=50, warm=2, sigma_P=0.01, huber_k=10.0, host=True),
        # a pixel-processor-array frame, the paper's resolution class, camera frames on the host
        dict(name="frame_256x256", kind="track", H=256, W=256, iters=20, warm=2, sigma_P=0.01, huber_k=400.0,
             host=True),
        # the headline frame: 640x480, 20 iterations, device tensors in and out
        dict(name="frame_640x480", kind="track", H=480, W=640, iters=20, warm=2, sigma_P=0.004, huber_k=10.0),
        # the largest frame that the depth-transfer scratch is sized for
        dict(name="frame_1920x1080", kind="track", H=1080, W=1920, iters=20, warm=2, sigma_P=0.002, huber_k=400.0),
        # a ragged crop with a sensor's sigma map and temporal priors (pose and per-pixel log-depth means)
        dict(name="frame_maps_333x245", kind="track", H=245, W=333, iters=20, warm=2, sigma_P=0.01, huber_k=10.0,
             maps=True),
        # a damped frame: the per-factor schedule is the one that supports damping
        dict(name="frame_damped_320x240", kind="track", H=240, W=320, iters=20, warm=2, sigma_P=0.01, huber_k=10.0,
             damping=0.2),
        # the hierarchical topology of the paper's main experiments
        dict(name="quadtree_640x480", kind="track", H=480, W=640, iters=20, warm=2, sigma_P=0.004, huber_k=10.0,
             tree=True),
        # four small sequences of mixed resolution advanced together
        dict(name="batch_4_mixed", kind="batch", n=4, base=0, iters=15, warm=2, sigma_P=0.004, huber_k=400.0),
        # the serving batch: 64 sequences of mixed resolution
        dict(name="batch_64_mixed", kind="batch", n=64, base=0, iters=15, warm=1, sigma_P=0.004, huber_k=400.0),
        # a training step on a small crop: forward, loss, backward to sigma map, sigma_N and Huber threshold
        dict(name="train_48x48", kind="unroll", H=48, W=48, frames=2, iters=10, ckpt=4, sigma_P=0.004, huber_k=1.0),
        # the training clip at the differentiation sequence's resolution
        dict(name="train_320x240", kind="unroll", H=240, W=320, frames=4, iters=30, ckpt=10, sigma_P=0.003,
             huber_k=1.0),
        # the centralised baseline at its comparison settings: IRLS with conjugate gradients to 1e-8
        dict(name="central_640x480", kind="central", H=480, W=640, iters=3, sigma_P=0.01, huber_k=400.0,
             cg_tol=1e-8),
    ]


def draw(rng):
    """One more case: the same kinds, sizes spread over 24 .. 1080 rows (odd ones among them)."""
    kind = rng.choice(["track", "track", "track", "tree", "damped", "batch", "unroll", "central"])
    top = {"track": 1080, "tree": 700, "damped": 480, "unroll": 240, "central": 480, "batch": 300}[kind]
    H = int(round(24 * (top / 24) ** rng.random()))
    W = max(16, min(1920, int(round(H * rng.uniform(0.8, 1.7))), 1920 * 1080 // H))
    hk, sp = rng.choice([10.0, 400.0]), round(0.01 * min(1.0, 256.0 / W), 4)
    c = dict(kind="track", H=H, W=W, iters=rng.randint(12, 20 if H > 500 else 30), warm=2, sigma_P=sp, huber_k=hk)
    if kind == "track":
        return dict(c, host=rng.random() < 0.4, maps=rng.random() < 0.3)
    if kind == "tree":
        return dict(c, tree=True, host=rng.random() < 0.3)
    if kind == "damped":
        return dict(c, damping=rng.choice([0.1, 0.3]), iters=rng.randint(12, 20))
    if kind == "batch":
        return dict(kind="batch", n=rng.randint(2, 40), base=rng.randint(0, 96), iters=rng.randint(8, 15), warm=2,
                    sigma_P=0.004, huber_k=rng.choice([10.0, 400.0]))
    if kind == "unroll":
        it = rng.randint(6, 20)
        return dict(kind="unroll", H=H, W=W, frames=rng.randint(1, 3), iters=it, ckpt=rng.randint(2, it),
                    sigma_P=0.003, huber_k=1.0)
    return dict(kind="central", H=H, W=W, iters=rng.randint(1, 3), sigma_P=0.01, huber_k=400.0, cg_tol=1e-8)


def batch_shapes(case):
    """Resolutions of a batch: the serving classes, or (base > 0) odd sizes around them."""
    cls = [(96, 128), (256, 256), (240, 320), (480, 640)]
    if not case["base"]:
        return [cls[i % 4] for i in range(case["n"])]
    b = case["base"]
    return [(cls[i % 4][0] - (7 * i + b) % 61, cls[i % 4][1] - (11 * i + b) % 83) for i in range(case["n"])]


# ---------------------------------------------------------------------------
# inputs


def intrinsics(H, W):
    """Pinhole at 30/32 of the width, principal point in the image centre; FP32 values as the library takes them."""
    f = float(np.float32(30.0 * W / 32.0))
    return f, f, W / 2.0, H / 2.0


def rotation(w):
    th = math.sqrt(float(w @ w))
    K = np.array([[0.0, -w[2], w[1]], [w[2], 0.0, -w[0]], [-w[1], w[0], 0.0]])
    return np.eye(3) + math.sin(th) / th * K + (1.0 - math.cos(th)) / th ** 2 * (K @ K)


def clip(H, W, seed, n_frames, device):
    """(keyframe image, normals, [frames]): a slanted textured surface and a camera that backs away from it, drifting
    and turning a little, by a fraction of a pixel per frame. FP32 tensors on `device`."""
    rng = np.random.default_rng(1_000_003 * (H * 4099 + W) + seed)
    fx, fy, cx, cy = intrinsics(H, W)
    n = np.array([rng.uniform(-0.25, 0.25), rng.uniform(-0.25, 0.25), -1.0])
    n /= np.linalg.norm(n)
    d = n[2] * rng.uniform(0.97, 1.06)
    e1 = np.cross(n, [0.0, 1.0, 0.0])
    e1 /= np.linalg.norm(e1)
    e2 = np.cross(n, e1)
    waves = 28
    ang, ph = rng.uniform(0, 2 * math.pi, (2, waves))
    freq = 2 * math.pi * fx / np.exp(rng.uniform(math.log(9.0), math.log(48.0), waves))
    amp = rng.uniform(0.5, 1.0, waves)
    amp *= 0.2 / math.sqrt(float((amp ** 2).sum()))
    v, u = torch.meshgrid(torch.arange(H, device=device, dtype=torch.float64),
                          torch.arange(W, device=device, dtype=torch.float64), indexing="ij")
    ray = ((u - cx) / fx, (v - cy) / fy, torch.ones_like(u))
    gen = torch.Generator(device=device).manual_seed(7919 * seed + H + 31 * W)

    def view(R, c):
        # camera at position c with orientation R (camera to world)
        w = [R[i, 0] * ray[0] + R[i, 1] * ray[1] + R[i, 2] for i in range(3)]
        s = (d - float(n @ c)) / (n[0] * w[0] + n[1] * w[1] + n[2] * w[2])
        x = [float(c[i]) + s * w[i] for i in range(3)]
        a = e1[0] * x[0] + e1[1] * x[1] + e1[2] * x[2]
        b = e2[0] * x[0] + e2[1] * x[1] + e2[2] * x[2]
        img = torch.full_like(a, 0.5)
        for k in range(waves):
            img += amp[k] * torch.sin(freq[k] * (math.cos(ang[k]) * a + math.sin(ang[k]) * b) + ph[k])
        img += 0.002 * torch.randn(img.shape, dtype=torch.float64, device=device, generator=gen)
        return img.clamp_(0.0, 1.0).float()

    I0 = view(np.eye(3), np.zeros(3))
    normals = torch.tensor(n, dtype=torch.float32, device=device).expand(H, W, 3).contiguous()
    # every border moves inwards by about half a pixel per frame: no pixel of the keyframe stays on the edge of a
    # frame, where its warp would be in or out by rounding
    step_t = rng.uniform(-0.1, 0.1, 3) / fx
    step_t[2] = -rng.uniform(0.45, 0.65) / (0.5 * min(H, W))
    step_r = np.append(rng.uniform(-0.07, 0.07, 2), rng.uniform(-0.02, 0.02)) / fx
    frames = []
    for k in range(1, n_frames + 1):
        frames.append(view(rotation(k * step_r), k * step_t))
    return I0, normals, frames


def sigma_map(H, W, seed, device):
    gen = torch.Generator(device=device).manual_seed(104729 * seed + H * W)
    return 5e-3 * (1.0 + 0.2 * (2.0 * torch.rand((H, W), device=device, generator=gen) - 1.0))


def cotangents(case, seed):
    """Cotangents of a training loss: of the poses (F, 6) and of the inverse-depth maps."""
    rng = np.random.default_rng(15_485_863 + seed)
    gen = torch.Generator().manual_seed(seed)
    return (torch.tensor(rng.normal(size=(case["frames"], 6))),
            (1.0 + torch.randn((case["frames"], case["H"], case["W"]), generator=gen)) / (case["H"] * case["W"]))


def params(case):
    return dict(sigma_P=case["sigma_P"], huber_k=case["huber_k"], damping=case.get("damping", 0.0),
                kf_max_frames=1_000_000)


def tracker(case, seed):
    H, W = case["H"], case["W"]
    I0, normals, frames = clip(H, W, seed, case["warm"] + 1, "cuda")
    sigma = sigma_map(H, W, seed, "cuda") if case.get("maps") else None
    t = pv.Tracker(H, W, intrinsics(H, W), **params(case))
    if case.get("tree"):
        t.set_topology(pv.TOPO_QUADTREE)
    if case.get("host"):
        I0, normals, frames = I0.cpu().numpy(), normals.cpu().numpy(), [f.cpu().numpy() for f in frames]
    t.set_keyframe(I0, normals)
    if sigma is not None:
        t.set_sigma_map(sigma)
    for f in frames[:-1]:
        t.track(f, case["iters"], maps=False)
        if case.get("maps"):
            t.set_prior_from_state()
    return t, frames[-1]


def prepare(case, seed):
    torch.cuda.set_device(0)
    if case["kind"] == "track":
        t, frame = tracker(case, seed)
        return dict(case=case, t=t, frame=frame)
    if case["kind"] == "batch":
        shapes = batch_shapes(case)
        clips = [clip(h, w, 1000 * seed + i, case["warm"] + 1, "cuda") for i, (h, w) in enumerate(shapes)]
        b = pv.Batch(shapes, [intrinsics(h, w) for h, w in shapes], **params(case))
        b.set_keyframes(list(range(len(shapes))), [c[0] for c in clips], [c[1] for c in clips])
        for k in range(case["warm"]):
            b.track([c[2][k] for c in clips], case["iters"])
        return dict(case=case, b=b, frames=[c[2][-1] for c in clips], keep=clips)
    if case["kind"] == "unroll":
        H, W = case["H"], case["W"]
        I0, normals, frames = clip(H, W, seed, case["frames"], "cuda")
        u = pv.Unrolled(H, W, intrinsics(H, W), case["iters"], case["frames"], case["ckpt"], sigma_P=case["sigma_P"],
                        huber_k=case["huber_k"])
        u.set_keyframe(I0, normals)
        xi_w, rho_w = cotangents(case, seed)
        return dict(case=case, u=u, frames=torch.stack(frames), xi_w=xi_w.float().cuda(), rho_w=rho_w.cuda(),
                    sigma=sigma_map(H, W, seed, "cuda").requires_grad_(),
                    sigma_N=torch.tensor(1e-3, device="cuda", requires_grad=True),
                    huber_k=torch.tensor(case["huber_k"], device="cuda", requires_grad=True))
    H, W = case["H"], case["W"]
    I0, normals, frames = clip(H, W, seed, 2, "cuda")
    c = pv.Central(H, W, intrinsics(H, W), cg_tol=case["cg_tol"], sigma_P=case["sigma_P"], huber_k=case["huber_k"])
    c.set_keyframe(I0, normals)
    return dict(case=case, c=c, frame=frames[-1])


def pose(x):
    """A pose at the type of the per-pixel state that it is the mean of. Of a frame's two forms, the world pose
    Exp(xi)^-1 and the tangent xi, the first: it is what a program uses."""
    return np.asarray(x, np.float32)


def run(state):
    case = state["case"]
    if case["kind"] == "track":
        r = state["t"].track(state["frame"], case["iters"], out_device=not case.get("host", False))
        return dict(T_world=pose(r["T_world"]), valid=np.float32(r["valid_fraction"]),
                    inv_depth=r["inv_depth"], inv_depth_var=r["inv_depth_var"], flags=r["flags"])
    if case["kind"] == "batch":
        rs = state["b"].track(state["frames"], case["iters"], maps=True)
        return dict(T_world=pose([r["T_world"] for r in rs]),
                    valid=np.array([r["valid_fraction"] for r in rs], np.float32),
                    flags=np.array([r["flags"] for r in rs]),
                    inv_depth=np.concatenate([r["inv_depth"].reshape(-1) for r in rs]),
                    inv_depth_var=np.concatenate([r["inv_depth_var"].reshape(-1) for r in rs]))
    if case["kind"] == "unroll":
        p = [state["sigma"], state["sigma_N"], state["huber_k"]]
        xi, rho = pv.unrolled_track(state["u"], state["frames"], *p)
        loss = (state["xi_w"] * xi.float()).sum() + (state["rho_w"] * rho).sum()
        g = torch.autograd.grad(loss, p)
        return dict(xi=xi.float(), inv_depth=rho, g_sigma=g[0], g_sigma_N=g[1], g_huber_k=g[2])
    c = state["c"]
    c.set_point(np.zeros(6), np.zeros((case["H"], case["W"])))
    r = c.track(state["frame"], case["iters"], out_device=True)
    return dict(xi=pose(r["xi"]), inv_depth=r["inv_depth"], valid=np.float32(r["valid_fraction"]), flags=r["flags"])


# ---------------------------------------------------------------------------
# what one pass cannot do without


def work(case):
    """Bytes: the state planes read and written once per iteration (FP32), frames and maps once, the reverse sweep's
    state and cotangent planes. FP64 operations: the per-pixel algebra of one iteration, two operations per fused
    multiply-add: two linearisations, four inverses of 6x6 matrices, a 7x7 solve, a 6x6 elimination, five Exp or Log."""
    grid_b, grid_f, tree_b, tree_f = 8 * 123 + 24, 4600.0, 8 * 42 + 24 + 0.34 * 8 * 141, 4500.0
    if case["kind"] == "batch":
        px = float(sum(h * w for h, w in batch_shapes(case)))
        return dict(bytes=px * (case["iters"] * grid_b + 20), flops=px * case["iters"] * grid_f)
    px = float(case["H"] * case["W"])
    if case["kind"] == "track":
        b, f = (tree_b, tree_f) if case.get("tree") else (grid_b, grid_f)
        return dict(bytes=px * (case["iters"] * b + 20), flops=px * case["iters"] * f)
    if case["kind"] == "unroll":
        it = case["frames"] * case["iters"]
        return dict(bytes=px * it * (grid_b + 3 * 8 * 123), flops=px * it * 4 * grid_f)
    # about 140 CG iterations of 12 reads and 5 writes of an FP64 plane
    return dict(bytes=px * case["iters"] * 140 * 17 * 8, flops=px * case["iters"] * 140 * 60)


# ---------------------------------------------------------------------------
# the model in 64 bits

LEFT, RIGHT, UP, DOWN = range(4)
EPS = 1e-3   # tolerance of the valid-warp window, pixels


def lam(sigma, level=0):
    return 1.0 / (float(np.float32(sigma)) * 2.0 ** -level) ** 2


def mv(A, x):
    return (A * x.unsqueeze(0)).sum(1)


def mm(A, B):
    return (A.unsqueeze(2) * B.unsqueeze(0)).sum(1)


def tr(A):
    return A.transpose(0, 1)


def hat(w):
    z = torch.zeros_like(w[0])
    return torch.stack([torch.stack([z, -w[2], w[1]]), torch.stack([w[2], z, -w[0]]), torch.stack([-w[1], w[0], z])])


def eye(n, like):
    return torch.eye(n, dtype=like.dtype, device=like.device).reshape(n, n, *([1] * like.dim())).expand(n, n, *like.shape)


def series(x, coeffs):
    r = torch.full_like(x, coeffs[-1])
    for c in coeffs[-2::-1]:
        r = r * x + c
    return r


SIN = [(-1.0) ** k / math.factorial(2 * k + 1) for k in range(8)]
COS = [(-1.0) ** k / math.factorial(2 * k + 2) for k in range(8)]
CUB = [(-1.0) ** k / math.factorial(2 * k + 3) for k in range(8)]
ASIN = [math.factorial(2 * k) / (4.0 ** k * math.factorial(k) ** 2 * (2 * k + 1)) for k in range(14)]
# (1 - x cot x) / (4 x^2) with x = theta / 2, from theta^2 / 12 + theta^4 / 720 + ...
VINV = [1 / 12, 1 / 720, 1 / 30240, 1 / 1209600, 1 / 47900160, 691 / 1307674368000]


def se3_exp(xi):
    w = xi[:3]
    th2 = (w * w).sum(0)
    W = hat(w)
    W2 = mm(W, W)
    I = eye(3, th2)
    R = I + series(th2, SIN) * W + series(th2, COS) * W2
    V = I + series(th2, COS) * W + series(th2, CUB) * W2
    return R, mv(V, xi[3:])


def se3_log(R, t):
    v = torch.stack([R[2, 1] - R[1, 2], R[0, 2] - R[2, 0], R[1, 0] - R[0, 1]])
    s2 = 0.25 * (v * v).sum(0)
    w = 0.5 * series(s2, ASIN) * v
    W = hat(w)
    Wt = mv(W, t)
    th2 = (w * w).sum(0)
    return torch.cat([w, t - 0.5 * Wt + series(th2, VINV) * mv(W, Wt)])


def inverse(A):
    """Inverse of SPD matrices A (n, n, ...) by Gauss-Jordan elimination."""
    n = A.shape[0]
    for k in range(n):
        d = 1.0 / A[k, k]
        row, col = A[k] * d, A[:, k]
        B = A - col.unsqueeze(1) * row.unsqueeze(0)
        keep = torch.arange(n, device=A.device) == k
        r = keep.reshape(n, 1, *([1] * (A.dim() - 2)))
        c = keep.reshape(1, n, *([1] * (A.dim() - 2)))
        B = torch.where(r, row.unsqueeze(0).expand_as(B), B)
        B = torch.where(c, (-col * d).unsqueeze(1).expand_as(B), B)
        A = torch.where(r & c, d.expand_as(B), B)
    return A


def shift(x, d):
    """x of the neighbour in direction d at every pixel (the border repeats; callers mask it)."""
    H, W = x.shape[-2:]
    if d == LEFT:
        return torch.cat([x[..., :, :1], x[..., :, :-1]], -1)
    if d == RIGHT:
        return torch.cat([x[..., :, 1:], x[..., :, -1:]], -1)
    if d == UP:
        return torch.cat([x[..., :1, :], x[..., :-1, :]], -2)
    return torch.cat([x[..., 1:, :], x[..., -1:, :]], -2)


class Model:
    """One keyframe: geometry, factor strengths, normal targets, priors."""

    def __init__(self, H, W, I0, normals, case, sigma=None, sigma_N=None, huber_k=None):
        self.H, self.W, dev = H, W, I0.device
        self.fx, self.fy, self.cx, self.cy = intrinsics(H, W)
        f64 = torch.float64
        v, u = torch.meshgrid(torch.arange(H, device=dev, dtype=f64), torch.arange(W, device=dev, dtype=f64),
                              indexing="ij")
        self.u, self.v = u, v
        self.q = torch.stack([(u - self.cx) / self.fx, (v - self.cy) / self.fy, torch.ones_like(u)])
        self.Is = I0.double()
        n = normals.double().permute(2, 0, 1)
        nq = (n * self.q).sum(0)
        ok = nq.abs() >= 1e-3 * (self.q * self.q).sum(0).sqrt()
        # targets towards the right and lower neighbour, and which edges are active
        self.c = {}
        for d, comp, f in ((RIGHT, 0, self.fx), (DOWN, 1, self.fy)):
            t = torch.where(ok, n[comp] / (f * torch.where(ok, nq, torch.ones_like(nq))), torch.zeros_like(nq))
            self.c[d] = (t.float().double(), ok)
        self.has = [u > 0, u < W - 1, v > 0, v < H - 1]
        self.lamP, self.lamR = lam(case["sigma_P"]), lam(4e-4)
        self.lamN = lam(1e-3) if sigma_N is None else 1.0 / sigma_N ** 2
        self.huber_k = float(case["huber_k"]) if huber_k is None else huber_k
        self.isig = 1.0 / float(np.float32(5e-3)) if sigma is None else 1.0 / sigma
        self.prior = None                                  # (R, t) of Exp(prior)^-1
        self.prior_ell = torch.zeros_like(u)
        self.beta = float(np.float32(case.get("damping", 0.0)))

    def frame(self, It):
        It = It.double()
        gx, gy = torch.empty_like(It), torch.empty_like(It)
        gx[:, 1:-1] = 0.5 * (It[:, 2:] - It[:, :-2])
        gx[:, 0], gx[:, -1] = It[:, 1] - It[:, 0], It[:, -1] - It[:, -2]
        gy[1:-1] = 0.5 * (It[2:] - It[:-2])
        gy[0], gy[-1] = It[1] - It[0], It[-1] - It[-2]
        self.img = torch.stack([It, gx, gy])

    def set_prior(self, xi, ell):
        R, t = se3_exp(xi.reshape(6, 1, 1))
        self.prior = (tr(R), -mv(tr(R), t))
        self.prior_ell = ell

    def photometric(self, R, t, ell):
        """Jacobian rows (7), weight, residual, valid-warp flag; everything 0 for an invalid warp."""
        rho = torch.exp(-ell)
        a = mv(R, self.q) + rho * t
        front = a[2] > 0
        iz = 1.0 / torch.where(front, a[2], torch.ones_like(a[2]))
        wx, wy = self.fx * a[0] * iz + self.cx, self.fy * a[1] * iz + self.cy
        ok = front & (wx >= -EPS) & (wx <= self.W - 1 + EPS) & (wy >= -EPS) & (wy <= self.H - 1 + EPS)
        x = torch.where(ok, wx, torch.zeros_like(wx)).clamp(0.0, self.W - 1.0)
        y = torch.where(ok, wy, torch.zeros_like(wy)).clamp(0.0, self.H - 1.0)
        x0 = x.detach().floor().clamp(0, self.W - 2)
        y0 = y.detach().floor().clamp(0, self.H - 2)
        fx, fy = x - x0, y - y0
        o = (y0 * self.W + x0).long()
        flat = self.img.reshape(3, -1)
        s = [flat[:, o + k] for k in (0, 1, self.W, self.W + 1)]
        It, gx, gy = (1 - fy) * ((1 - fx) * s[0] + fx * s[1]) + fy * ((1 - fx) * s[2] + fx * s[3])
        r = self.Is - It
        c = torch.stack([-gx * self.fx * iz, -gy * self.fy * iz, (gx * self.fx * a[0] + gy * self.fy * a[1]) * iz * iz])
        b = mv(tr(R), c)
        J = torch.cat([torch.linalg.cross(self.q, b, dim=0), rho * b, (-rho * (c * t).sum(0)).unsqueeze(0)])
        M = r.abs() * self.isig
        kM = self.huber_k / torch.where(M > self.huber_k, M, torch.ones_like(M))
        w = torch.where(M > self.huber_k, kM * (2.0 - kM), torch.ones_like(M)) * self.isig ** 2
        z = ok.to(r.dtype)
        return J * z, w * z, r * z, ok

    def pose_prior(self, tau, R, t, lamP):
        """(information, -gradient) of a pose prior of precision lamP at tau, (R, t) = Exp(tau)."""
        r = tau
        if self.prior is not None:
            Rp, tp = (p.expand(*p.shape[:-2], *tau.shape[-2:]) for p in self.prior)
            r = se3_log(mm(Rp, R), mv(Rp, t) + tp)
        w, q = hat(r[:3]), hat(r[3:])
        S = eye(3, r[0]) + 0.5 * w + mm(w, w) / 12.0
        Q = 0.5 * q + (mm(q, w) + mm(w, q)) / 12.0
        J = torch.cat([torch.cat([S, torch.zeros_like(S)], 1), torch.cat([Q, S], 1)], 0)
        return lamP * mm(tr(J), J), -lamP * mv(tr(J), r)

    def unary(self, tau, ell):
        R, t = se3_exp(tau)
        J, w, r, ok = self.photometric(R, t, ell)
        L = w * J.unsqueeze(1) * J.unsqueeze(0)
        eta = -w * r * J
        Lp, ep = self.pose_prior(tau, R, t, self.lamP)
        pad = torch.nn.functional.pad
        z = [0, 0] * tau[0].dim()
        L = L + pad(Lp, z + [0, 1, 0, 1])
        last = (torch.arange(7, device=tau.device) == 6).reshape(7, 1, 1).to(tau.dtype)
        L = L + self.lamP * last.unsqueeze(1) * last.unsqueeze(0)
        eta = eta + pad(ep, z + [0, 1]) - self.lamP * last * (ell - self.prior_ell)
        return L, eta, R, t, ok

    def normal_edge(self, d):
        """(target, active) of the edge towards direction d."""
        if d in (RIGHT, DOWN):
            return self.c[d][0], self.c[d][1] & self.has[d]
        c, ok = self.c[d ^ 1]
        return shift(c, d), shift(ok, d) & self.has[d]

    def normal_messages(self, ell, D, dv, mn):
        """New messages (eta, lambda) of the four normal-integration factors, and where they are defined."""
        out = []
        for d in range(4):
            c, ok = self.normal_edge(d)
            s = d ^ 1
            ls = shift(D - mn[s][1], d)
            vs = shift(dv - mn[s][0], d)
            lp = self.lamN * ls / (self.lamN + ls)
            h = self.lamN * vs / (self.lamN + ls)
            r = ell - shift(ell, d) + (c if d in (LEFT, UP) else -c)
            z = ok.to(ell.dtype)
            out.append(torch.stack([z * (h - lp * r), z * lp]))
        return torch.stack(out)

    def depth_marginal(self, L, eta):
        Ai = inverse(L[:6, :6])
        y = mv(Ai, L[:6, 6])
        return L[6, 6] - (L[:6, 6] * y).sum(0), eta[6] - (y * eta[:6]).sum(0)

    def update(self, L, eta, tau, ell, R, t):
        C = inverse(L)
        m = mv(C, eta)
        Rm, tm = se3_exp(m[:6])
        return m, se3_log(mm(R, Rm), mv(R, tm) + t), ell + m[6], C[6, 6]


def identity_message(P, p, back_L, back_e, lamR, r):
    """Message of an identity factor: sender's pose marginal less the factor's message to it, receiver's residual r."""
    V = P - back_L
    Ai = inverse(V + lamR * eye(6, r[0]))
    Ln = lamR * eye(6, r[0]) - lamR ** 2 * Ai
    return Ln, lamR * mv(Ai, p - back_e) - mv(Ln, r)


def between(Rj, tj, Ri, ti):
    return se3_log(mm(tr(Rj), Ri), mv(tr(Rj), ti - tj))


def embed(L6):
    return torch.nn.functional.pad(L6, [0, 0] * (L6.dim() - 2) + [0, 1, 0, 1])


class Grid:
    """The state of the grid topology: (tau, ell, identity messages, normal messages)."""

    def __init__(self, model):
        m, z = model, torch.zeros_like(model.u)
        self.m = m
        self.state = (z.expand(6, *z.shape), z, z.expand(4, 6, 6, *z.shape), z.expand(4, 6, *z.shape),
                      z.expand(4, 2, *z.shape))

    def iterate(self, tau, ell, mL, me, mn):
        m = self.m
        L0, e0, R, t, ok = m.unary(tau, ell)
        L = L0 + embed(mL.sum(0))
        e = e0 + torch.cat([me.sum(0), mn[:, 0].sum(0, keepdim=True)])
        L = L + torch.nn.functional.pad(mn[:, 1].sum(0)[None, None], [0, 0, 0, 0, 6, 0, 6, 0])
        i66 = 1.0 / L[6, 6]
        P = L[:6, :6] - i66 * L[:6, 6].unsqueeze(1) * L[:6, 6].unsqueeze(0)
        p = e[:6] - L[:6, 6] * i66 * e[6]
        D, dv = m.depth_marginal(L, e)
        nL, ne = [], []
        for d in range(4):
            s = d ^ 1
            r = between(shift(R, d), shift(t, d), R, t)
            Ln, en = identity_message(shift(P, d), shift(p, d), shift(mL[s], d), shift(me[s], d), m.lamR, r)
            z = m.has[d].to(ell.dtype)
            nL.append(z * Ln)
            ne.append(z * en)
        nL, ne, nn = torch.stack(nL), torch.stack(ne), m.normal_messages(ell, D, dv, mn)
        if m.beta:
            nL, ne, nn = ((1 - m.beta) * a + m.beta * b for a, b in ((nL, mL), (ne, me), (nn, mn)))
        L = L0 + embed(nL.sum(0)) + torch.nn.functional.pad(nn[:, 1].sum(0)[None, None], [0, 0, 0, 0, 6, 0, 6, 0])
        e = e0 + torch.cat([ne.sum(0), nn[:, 0].sum(0, keepdim=True)])
        st, tau, ell, var = m.update(L, e, tau, ell, R, t)
        ne = ne - (nL * st[:6].unsqueeze(0).unsqueeze(0)).sum(2)
        nn = torch.stack([nn[:, 0] - nn[:, 1] * st[6], nn[:, 1]], 1)
        return tau, ell, nL, ne, nn, var, ok

    def track(self, It, iters):
        self.m.frame(It)
        for _ in range(iters):
            *s, self.var, self.ok = self.iterate(*self.state)
            self.state = tuple(s)
        return self.outputs()

    def outputs(self):
        tau, ell = self.state[:2]
        rho = torch.exp(-ell)
        return tau.reshape(6, -1).mean(1), rho, rho * rho * self.var, self.ok.double().mean()


class Quadtree(Grid):
    """Pixels tied to a quadtree of pose nodes: levels 1 .. L of (6, Hl, Wl) poses. Every edge joins a node to its
    parent and keeps two messages: to the child (down) and to the parent (up)."""

    def __init__(self, model):
        self.m = m = model
        z = torch.zeros_like(m.u)
        self.shapes = [(m.H, m.W)]
        while self.shapes[-1] != (1, 1):
            h, w = self.shapes[-1]
            self.shapes.append(((h + 1) // 2, (w + 1) // 2))
        zero = lambda *s: torch.zeros(s, dtype=torch.float64, device=z.device)  # noqa: E731
        self.tau = [zero(6, h, w) for h, w in self.shapes]
        self.ell, self.mn = z, zero(4, 2, m.H, m.W)
        edges = self.shapes[:-1]
        self.down = [(zero(6, 6, h, w), zero(6, h, w)) for h, w in edges]
        self.up = [(zero(6, 6, h, w), zero(6, h, w)) for h, w in edges]
        self.lamP = [lam(m_sigma(m), l) for l in range(len(self.shapes))]
        self.lamR = [lam(4e-4, l) for l in range(len(edges))]

    def spread(self, x, l):
        """A parent field (level l + 1) at its children (level l)."""
        h, w = self.shapes[l]
        return x.repeat_interleave(2, -2)[..., :h, :].repeat_interleave(2, -1)[..., :w]

    def gather(self, x, l):
        """Sum over the children (level l) at their parents (level l + 1)."""
        h, w = self.shapes[l]
        x = torch.nn.functional.pad(x, [0, w % 2, 0, h % 2])
        x = x[..., 0::2, :] + x[..., 1::2, :]
        return x[..., 0::2] + x[..., 1::2]

    def track(self, It, iters):
        m = self.m
        m.frame(It)
        n = len(self.shapes)
        pad = torch.nn.functional.pad
        for _ in range(iters):
            poses = [se3_exp(x) for x in self.tau]
            L0, e0, R, t, self.ok = m.unary(self.tau[0], self.ell)
            unary = [(L0, e0)] + [m.pose_prior(self.tau[l], *poses[l], self.lamP[l]) for l in range(1, n)]

            def belief(down, up, mn):
                L = unary[0][0] + embed(down[0][0]) + pad(mn[:, 1].sum(0)[None, None], [0, 0, 0, 0, 6, 0, 6, 0])
                e = unary[0][1] + torch.cat([down[0][1], mn[:, 0].sum(0, keepdim=True)])
                out = [(L, e)]
                for l in range(1, n):
                    a, b = unary[l][0] + self.gather(up[l - 1][0], l - 1), unary[l][1] + self.gather(up[l - 1][1], l - 1)
                    if l < n - 1:
                        a, b = a + down[l][0], b + down[l][1]
                    out.append((a, b))
                return out

            bel = belief(self.down, self.up, self.mn)
            L, e = bel[0]
            D, dv = m.depth_marginal(L, e)
            i66 = 1.0 / L[6, 6]
            marg = [(L[:6, :6] - i66 * L[:6, 6].unsqueeze(1) * L[:6, 6].unsqueeze(0), e[:6] - L[:6, 6] * i66 * e[6])]
            marg += bel[1:]
            down, up = [], []
            for l in range(n - 1):
                Rp, tp = (self.spread(x, l) for x in poses[l + 1])
                Rc, tc = poses[l]
                P, p = (self.spread(x, l) for x in marg[l + 1])
                down.append(identity_message(P, p, *self.up[l], self.lamR[l], between(Rp, tp, Rc, tc)))
                up.append(identity_message(*marg[l], *self.down[l], self.lamR[l], between(Rc, tc, Rp, tp)))
            mn = m.normal_messages(self.ell, D, dv, self.mn)
            bel = belief(down, up, mn)
            st, tau0, self.ell, self.var = m.update(*bel[0], self.tau[0], self.ell, R, t)
            steps, tau = [st[:6]], [tau0]
            for l in range(1, n):
                x = mv(inverse(bel[l][0]), bel[l][1])
                Rm, tm = se3_exp(x)
                Rl, tl = poses[l]
                steps.append(x)
                tau.append(se3_log(mm(Rl, Rm), mv(Rl, tm) + tl))
            self.tau = tau
            self.down = [(Ln, en - mv(Ln, steps[l])) for l, (Ln, en) in enumerate(down)]
            self.up = [(Ln, en - mv(Ln, self.spread(steps[l + 1], l))) for l, (Ln, en) in enumerate(up)]
            self.mn = torch.stack([mn[:, 0] - mn[:, 1] * st[6], mn[:, 1]], 1)
        self.state = (self.tau[0], self.ell)
        return self.outputs()


def m_sigma(model):
    return 1.0 / math.sqrt(model.lamP)


def invert_pose(xi):
    R, t = se3_exp(xi.reshape(6, 1))
    T = torch.eye(4, dtype=torch.float64, device=xi.device)
    T[:3, :3] = R[..., 0].T
    T[:3, 3] = -(R[..., 0].T @ t[:, 0])
    return T


def exact_track(case, seed, shape=None, clip_=None, device="cuda"):
    H, W = shape or (case["H"], case["W"])
    I0, normals, frames = clip_ or clip(H, W, seed, case["warm"] + 1, device)
    sigma = sigma_map(H, W, seed, device).double() if case.get("maps") else None
    m = Model(H, W, I0, normals, case, sigma)
    s = Quadtree(m) if case.get("tree") else Grid(m)
    for f in frames:
        xi, rho, var, ok = s.track(f, case["iters"])
        if case.get("maps") and f is not frames[-1]:
            m.set_prior(xi, s.state[1])
    return xi, invert_pose(xi), ok, rho, var


def exact_unroll(case, seed, device="cuda"):
    H, W, F = case["H"], case["W"], case["frames"]
    I0, normals, frames = clip(H, W, seed, F, device)
    sigma = sigma_map(H, W, seed, device).double().requires_grad_()
    sN = torch.tensor(float(np.float32(1e-3)), dtype=torch.float64, device=device, requires_grad=True)
    k = torch.tensor(float(case["huber_k"]), dtype=torch.float64, device=device, requires_grad=True)
    xi_w, rho_w = cotangents(case, seed)
    m = Model(H, W, I0, normals, case, sigma, sN, k)
    g = Grid(m)
    xis, rhos, loss = [], [], 0.0
    for f in range(F):
        m.frame(frames[f])
        img = m.img

        def step(img, sigma, sN, k, *state):
            m.img, m.isig, m.lamN, m.huber_k = img, 1.0 / sigma, 1.0 / sN ** 2, k
            return g.iterate(*state)[:5]

        for _ in range(case["iters"]):
            g.state = checkpoint(step, img, sigma, sN, k, *g.state, use_reentrant=False)
        tau, ell = g.state[:2]
        xis.append(tau.reshape(6, -1).mean(1))
        rhos.append(torch.exp(-ell))
        loss = loss + (xi_w[f].to(device) * xis[-1]).sum() + (rho_w[f].to(device).double() * rhos[-1]).sum()
    gr = torch.autograd.grad(loss, [sigma, sN, k])
    return dict(xi=torch.stack(xis).detach(), inv_depth=torch.stack(rhos).detach(), g_sigma=gr[0], g_sigma_N=gr[1],
                g_huber_k=gr[2])


def exact_central(case, seed, device="cuda"):
    """IRLS Gauss-Newton on one pose and per-pixel log-depths; the normal equations by conjugate gradients on the
    depth block's Schur complement of the pose, to 1e-13."""
    H, W = case["H"], case["W"]
    I0, normals, frames = clip(H, W, seed, 2, device)
    m = Model(H, W, I0, normals, case)
    m.frame(frames[-1])
    xi, ell = torch.zeros(6, dtype=torch.float64, device=device), torch.zeros_like(m.u)
    edges = [m.normal_edge(d) for d in range(4)]
    act = [e[1].to(ell.dtype) for e in edges]
    for _ in range(case["iters"]):
        R, t = se3_exp(xi.reshape(6, 1, 1).expand(6, H, W))
        J, w, r, ok = m.photometric(R, t, ell)
        Lp, ep = m.pose_prior(xi.reshape(6, 1, 1), *se3_exp(xi.reshape(6, 1, 1)), m.lamP)
        A = (w * J[:6].unsqueeze(1) * J[:6].unsqueeze(0)).sum((2, 3)) + Lp[..., 0, 0]
        gp = -(w * r * J[:6]).sum((1, 2)) + ep[..., 0, 0]
        B = w * J[:6] * J[6]
        D = w * J[6] ** 2 + m.lamP
        gd = -w * r * J[6] - m.lamP * (ell - m.prior_ell)
        for d in range(4):
            c = edges[d][0]
            D = D + m.lamN * act[d]
            gd = gd - m.lamN * act[d] * (ell - shift(ell, d) + (c if d in (LEFT, UP) else -c))

        def apply(x):
            y = D * x
            for d in range(4):
                y = y - m.lamN * act[d] * shift(x, d)
            return y

        def solve(b):
            x = torch.zeros_like(b)
            res = b.clone()
            z = res / D
            p, rz = z.clone(), (res * z).sum((-2, -1), keepdim=True)
            r0 = rz.sqrt()
            for k in range(3000):
                q = apply(p)
                a = rz / (p * q).sum((-2, -1), keepdim=True).clamp_min(1e-300)
                x, res = x + a * p, res - a * q
                z = res / D
                new = (res * z).sum((-2, -1), keepdim=True)
                if k % 16 == 0 and bool((new.sqrt() <= 1e-13 * r0).all()):
                    break
                p, rz = z + new / rz.clamp_min(1e-300) * p, new
            return x

        S = solve(torch.cat([B, gd.unsqueeze(0)]))
        dx = torch.linalg.solve(A - (B.unsqueeze(1) * S[:6].unsqueeze(0)).sum((2, 3)), gp - (B * S[6]).sum((1, 2)))
        ell = ell + S[6] - (S[:6] * dx.reshape(6, 1, 1)).sum(0)
        Rm, tm = se3_exp(dx.reshape(6, 1))
        R1, t1 = se3_exp(xi.reshape(6, 1))
        xi = se3_log(mm(R1, Rm), mv(R1, tm) + t1)[:, 0]
    return xi, torch.exp(-ell), ok.double().mean()


def exact(case, seed):
    if case["kind"] == "unroll":
        return exact_unroll(case, seed)
    with torch.no_grad():
        if case["kind"] == "central":
            xi, rho, ok = exact_central(case, seed)
            return dict(xi=xi, inv_depth=rho, valid=ok, flags=None)
        if case["kind"] == "track":
            xi, T, ok, rho, var = exact_track(case, seed)
            return dict(T_world=T, valid=ok, inv_depth=rho, inv_depth_var=var, flags=None)
        rs = [exact_track(case, None, s, clip(*s, 1000 * seed + i, case["warm"] + 1, "cuda"))
              for i, s in enumerate(batch_shapes(case))]
        return dict(T_world=torch.stack([r[1] for r in rs]),
                    valid=torch.stack([r[2] for r in rs]), flags=None,
                    inv_depth=torch.cat([r[3].reshape(-1) for r in rs]),
                    inv_depth_var=torch.cat([r[4].reshape(-1) for r in rs]))
