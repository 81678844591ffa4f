"""The work a program has this library do, as timed cases.

Each case is one call sequence through the public binding (``paper_2207_14507_amd.prnu``)
on synthetic inputs of the statistics the library meets: a fingerprint K ~ N(0, 0.02^2),
residual frames W = T(I K) + N(0, 0.05^2) of a smooth scene I under a walk of small
similarity transforms T, and for the estimators images in [0, 255] carrying the
multiplicative pattern and noise.

Kinds:

  score       PCE, NCC and shift of every candidate of one frame (``prnu_score_grid``)
  enrol       a new fingerprint opened, one frame checked against it, closed again
  search      the frames of one video: the full grid on every frame, the warm-started
              chain, or the coarse-to-fine schedule (``prnu_search_frames``)
  transforms  general 8-parameter transforms scored on one frame
  serve       several videos submitted to the serving engine and polled
  residuals   noise residuals of images (``prnu_extract_residuals``)
  estimate    the reference fingerprint of images and residuals

The scores of the search (PCE, NCC) come out of single-precision transforms and are kept
as float32, as a program that stores them would; grid nodes, shifts and indices are kept
as they are.
"""
import atexit
import math
import random

import numpy as np
import torch

from paper_2207_14507_amd import prnu as P

# The exhaustive grid and the warm-start options of the repository's workloads.
FULL = (41, 0.85, 1.15, 21, -2.0, 2.0)
LOCAL = (9, 9, 0.005, 0.1)
COLS = (64, 96, 120, 160, 256, 720, 1080, 1280, 1920, 2160)  # supported heights
ROWS = COLS + (3840,)                                        # supported widths

_ctx = None


def _context():
    """The one library context a program keeps per device."""
    global _ctx
    if _ctx is None:
        _ctx = P.prnu_create(0)
        atexit.register(_destroy)
    return _ctx


def _destroy():
    global _ctx
    c, _ctx = _ctx, None
    if c is not None:
        P.prnu_destroy(c)


class _Fingerprint:
    """A device-resident fingerprint, closed with its last reference."""

    def __init__(self, K):
        self.handle = P.prnu_open_fingerprint(_context(), K)

    def __del__(self):
        if _ctx is not None:
            P.prnu_close_fingerprint(_ctx, self.handle)


# ---------------------------------------------------------------------------
# Cases.

def _grid_case(kind, M, N, **kw):
    c = dict(kind=kind, M=M, N=N, Mf=M, Nf=N, F=1, radius=64, dtype="f32", host=False,
             n_scale=FULL[0], n_rot=FULL[3], mode="plain")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one 256 x 256 frame from host memory, 11 x 11 grid
        dict(_grid_case("score", 256, 256, radius=16, n_scale=11, n_rot=11, host=True), name="score_256_host"),
        # a camera enrolled and one frame checked as it is, 3 x 3 candidates around it
        dict(_grid_case("enrol", 720, 1280, n_scale=3, n_rot=3), name="enrol_720p"),
        # a matching 720p video followed by the warm start (81 candidates a frame)
        dict(_grid_case("search", 720, 1280, F=8, mode="warm"), name="warm_720p"),
        # the headline workload's step, fewer frames: the full 41 x 21 grid on every frame
        dict(_grid_case("search", 1080, 1920, F=4), name="full_1080p"),
        # 4K residuals stored in bf16, the largest frames
        dict(_grid_case("search", 2160, 3840, F=2, dtype="bf16"), name="full_4k_bf16"),
        # the paper's coarse-to-fine schedule with its own values
        dict(_grid_case("search", 1080, 1920, F=2, mode="refine"), name="refine_1080p"),
        # frames cropped by the stabilisation, against the full-size fingerprint
        dict(_grid_case("search", 1080, 1920, Mf=720, Nf=1280), name="cropped_720p_in_1080p"),
        # general transforms proposed by a co-registration step
        dict(_grid_case("transforms", 1080, 1920, n_scale=256, n_rot=1), name="transforms_1080p"),
        # two matching and two foreign videos of two sizes at once
        dict(kind="serve", M=720, N=1280, M2=1080, N2=1920, videos=4, F=4, radius=64, name="serve_mixed"),
        # residuals of a video's frames on the device
        dict(kind="residuals", L=16, M=1080, N=1920, host=False, name="residuals_1080p"),
        # residuals of a few small cropped images, sides that are no multiple of anything
        dict(kind="residuals", L=3, M=333, N=501, host=False, name="residuals_333x501"),
        # the reference fingerprint of flat-field images and their residuals
        dict(kind="estimate", L=32, M=1080, N=1920, host=False, name="estimate_1080p"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed cases' ranges."""
    kind = rng.choice(["score", "enrol", "search", "search", "search", "search", "transforms", "serve", "residuals",
                       "residuals", "estimate"])
    host = rng.random() < 0.2
    if kind in ("residuals", "estimate"):
        M, N = _log_int(rng, 64, 2160), _log_int(rng, 64, 3840)
        L = _log_int(rng, 1, max(1, min(32, (32 * 1080 * 1920) // (M * N))))
        return dict(kind=kind, L=L, M=M, N=N, host=host and L * M * N < 8 << 20)
    big = 1722 * 2160 * 3840  # candidates x pixels of the largest listed case
    M = rng.choice(COLS if rng.random() < 0.25 else COLS[4:])
    N = rng.choice(ROWS if rng.random() < 0.25 else ROWS[4:])
    radius = rng.randint(4, min(64, (min(M, N) - 11) // 2))
    if kind == "serve":
        M2, N2 = rng.choice(COLS[4:]), rng.choice(ROWS[4:9])
        radius = min(radius, 64)
        videos = rng.randint(2, 4)
        F = rng.randint(1, 4)
        while videos * F * 942 * max(M * N, M2 * N2) > big and F > 1:
            F -= 1
        while videos * F * 942 * max(M * N, M2 * N2) > big and videos > 1:
            videos -= 1
        return dict(kind=kind, M=M, N=N, M2=M2, N2=N2, videos=videos, F=F, radius=radius)
    c = _grid_case(kind, M, N, radius=radius, host=host, dtype="bf16" if rng.random() < 0.25 else "f32")
    c["n_scale"], c["n_rot"] = 2 * _log_int(rng, 1, 20) + 1, 2 * _log_int(rng, 1, 10) + 1
    if kind == "enrol":
        c["n_scale"] = c["n_rot"] = rng.choice((1, 3, 5))
        c["dtype"] = "f32"
        return c
    if rng.random() < 0.2:  # a frame smaller than the fingerprint, any size
        c["Mf"] = rng.randint(max(2 * radius + 11, M // 2), M)
        c["Nf"] = rng.randint(max(2 * radius + 11, N // 2), N)
    if kind == "transforms":
        c["n_scale"], c["n_rot"] = _log_int(rng, 4, min(861, big // (M * N))), 1
    if kind == "search":
        c["mode"] = rng.choice(("plain", "plain", "warm", "refine"))
        c["F"] = rng.randint(1, 8)
        if c["mode"] == "warm":
            c["n_scale"], c["n_rot"] = FULL[0], FULL[3]
        per = {"plain": c["n_scale"] * c["n_rot"], "warm": 942, "refine": 1353}[c["mode"]]
        c["F"] = max(1, min(c["F"], big // (M * N * per), 4000 // per))
    return c


# ---------------------------------------------------------------------------
# Inputs, from the seed alone.

def _walk(r, n, radius):
    """Similarity transforms (scale, degrees, dx, dy) of a handheld video: a random walk
    from (1, 0, 0, 0) in the repository's steps."""
    s, t, dx, dy = 1.0, 0.0, 0, 0
    out = []
    for _ in range(n):
        s = min(1.15, max(0.85, s + r.gauss(0.0, 0.003)))
        t = min(2.0, max(-2.0, t + r.gauss(0.0, 0.1)))
        dx = min(radius, max(-radius, dx + round(r.gauss(0.0, 2.0))))
        dy = min(radius, max(-radius, dy + round(r.gauss(0.0, 2.0))))
        out.append((s, t, dx, dy))
    return out


def _scene(g, M, N):
    """Smooth intensity in [0.2, 0.9], correlated over about N / 16 pixels."""
    z = torch.randn((1, 1, max(4, round(16 * M / N)), 16), generator=g, device="cuda")
    z = torch.nn.functional.interpolate(z, size=(M, N), mode="bicubic", align_corners=True)[0, 0]
    return torch.clamp(0.55 + 0.25 * (z - z.mean()) / z.std().clamp_min(1e-6), 0.2, 0.9)


def _stabilised(g, K, move, Mf, Nf):
    """A residual frame of the camera with pattern K under the transform `move`, its
    first Mf x Nf pixels."""
    M, N = K.shape
    s, t, dx, dy = move
    c, n = math.cos(math.radians(t)), math.sin(math.radians(t))
    uy = (torch.arange(M, device="cuda", dtype=torch.float32) - (M - 1) / 2)[:, None]
    ux = (torch.arange(N, device="cuda", dtype=torch.float32) - (N - 1) / 2)[None, :]
    xs = (s * (c * ux + n * uy) + dx) * (2.0 / (N - 1))
    ys = (s * (-n * ux + c * uy) + dy) * (2.0 / (M - 1))
    img = (_scene(g, M, N) * K)[None, None]
    w = torch.nn.functional.grid_sample(img, torch.stack((xs, ys), -1)[None], mode="bilinear", padding_mode="zeros",
                                        align_corners=True)[0, 0]
    w = w + torch.randn((M, N), generator=g, device="cuda") * 0.05
    return w[:Mf, :Nf]


def _video(seed, M, N, Mf, Nf, F, radius, foreign=False):
    """A fingerprint and F residual frames of a video of that camera (or of another)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    K = torch.randn((M, N), generator=g, device="cuda") * 0.02
    own = torch.randn((M, N), generator=g, device="cuda") * 0.02 if foreign else K
    moves = _walk(random.Random(seed), F, min(radius, 16))
    return K, torch.stack([_stabilised(g, own, m, Mf, Nf) for m in moves]).contiguous()


def _store(frames, dtype):
    """(frames as stored, scales or None): bf16 storage divides each frame by the power
    of two at or above its largest magnitude."""
    if dtype == "f32":
        return frames, None
    top = frames.abs().amax(dim=(1, 2)).double()
    scale = torch.exp2(torch.ceil(torch.log2(top))).float()
    return (frames / scale[:, None, None]).to(torch.bfloat16), scale


def _images(seed, L, M, N):
    """L images in [0, 255] of one camera: smooth scenes, the pattern, noise of s.d. 2."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    K = torch.randn((M, N), generator=g, device="cuda") * 0.02
    return torch.stack([_scene(g, M, N) * 255.0 * (1.0 + K) + torch.randn((M, N), generator=g, device="cuda") * 2.0
                        for _ in range(L)])


def _estimate_inputs(seed, L, M, N):
    g = torch.Generator(device="cuda").manual_seed(seed)
    K = torch.randn((M, N), generator=g, device="cuda") * 0.02
    I = torch.stack([_scene(g, M, N) for _ in range(L)])
    return I, I * K + torch.randn((L, M, N), generator=g, device="cuda") * 0.05


def _transforms(seed, n):
    """n general transforms near the identity (centred coordinates)."""
    r = np.random.default_rng(seed)
    T = np.tile(np.eye(3), (n, 1, 1))
    T[:, :2, :2] += r.uniform(-0.03, 0.03, (n, 2, 2))
    T[:, 2, :2] = r.uniform(-3e-5, 3e-5, (n, 2))
    T[0] = np.eye(3)
    return T


def _videos(case, seed):
    """The serving case's videos: sizes in turn, every second pair of another camera."""
    out = []
    for v in range(case["videos"]):
        M, N = (case["M"], case["N"]) if v % 2 == 0 else (case["M2"], case["N2"])
        R = min(case["radius"], (min(M, N) - 11) // 2)
        out.append((M, N, R, *_video(seed * 64 + v, M, N, M, N, case["F"], R, foreign=v % 4 >= 2)))
    return out


def _grid(case):
    if case["kind"] == "enrol":  # the frame as it is and its neighbours
        h = 0.005 * (case["n_scale"] // 2)
        return (case["n_scale"], 1.0 - h, 1.0 + h, case["n_rot"], -20.0 * h, 20.0 * h)
    return (case["n_scale"], FULL[1], FULL[2], case["n_rot"], FULL[4], FULL[5])


def _options(case):
    return P.make_opts(grid=_grid(case), radius=case["radius"], warm=case["mode"] == "warm", local=LOCAL,
                       refine={} if case["mode"] == "refine" else None)


def _to_host(t):
    """The host form the library takes: float32, or the bf16 bits."""
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16)
    return t.cpu().numpy()


def prepare(case, seed):
    ctx = _context()
    kind = case["kind"]
    if kind == "residuals":
        I = _images(seed, case["L"], case["M"], case["N"])
        if case["host"]:
            return dict(kind=kind, images=_to_host(I), out=None)
        return dict(kind=kind, images=I, out=torch.empty_like(I))
    if kind == "estimate":
        I, W = _estimate_inputs(seed, case["L"], case["M"], case["N"])
        if case["host"]:
            return dict(kind=kind, images=_to_host(I), residuals=_to_host(W), out=None)
        return dict(kind=kind, images=I, residuals=W, out=torch.empty_like(I[0]))
    if kind == "serve":
        videos = []
        for M, N, R, K, W in _videos(case, seed):
            P.prnu_tune(ctx, M, N, R)
            videos.append((_Fingerprint(K), W, P.make_opts(grid=FULL, radius=R, warm=True, local=LOCAL)))
        return dict(kind=kind, videos=videos)
    K, W = _video(seed, case["M"], case["N"], case["Mf"], case["Nf"], case["F"], case["radius"])
    W, scales = _store(W, case["dtype"])
    if case["host"]:
        W, scales = _to_host(W), None if scales is None else scales.cpu().numpy()
    P.prnu_tune(ctx, case["M"], case["N"], case["radius"], P.PRNU_BF16 if case["dtype"] == "bf16" else P.PRNU_F32)
    state = dict(kind=kind, frames=W, scales=scales, opts=_options(case), radius=case["radius"])
    if kind == "enrol":
        state["K"] = _to_host(K) if case["host"] else K
    else:
        state["fp"] = _Fingerprint(K)
    if kind == "transforms":
        state["T"] = _transforms(seed, case["n_scale"])
    return state


# ---------------------------------------------------------------------------
# One pass.

def _scores(pce, rho, dx, dy):
    return dict(pce=np.asarray(pce, np.float32), rho=np.asarray(rho, np.float32), dx=dx, dy=dy)


def _found(results):
    """The results of a video's frames as arrays."""
    return dict(_scores([r.pce for r in results], [r.rho for r in results],
                        np.array([r.dx for r in results], np.int32), np.array([r.dy for r in results], np.int32)),
                scale=np.array([r.scale for r in results]), rot_deg=np.array([r.rot_deg for r in results]),
                cand_index=np.array([r.cand_index for r in results], np.int32),
                n_evaluated=np.array([r.n_evaluated for r in results], np.int32))


def run(state):
    ctx, kind = _ctx, state["kind"]
    if kind == "score":
        return _scores(*P.prnu_score_grid(ctx, state["fp"].handle, state["frames"], 0, state["opts"],
                                          scales=state["scales"]))
    if kind == "enrol":
        fp = P.prnu_open_fingerprint(ctx, state["K"])
        out = _scores(*P.prnu_score_grid(ctx, fp, state["frames"], 0, state["opts"]))
        P.prnu_close_fingerprint(ctx, fp)
        return out
    if kind == "search":
        return _found(P.prnu_search_frames(ctx, state["fp"].handle, state["frames"], state["opts"],
                                           scales=state["scales"])[0])
    if kind == "transforms":
        return _scores(*P.prnu_score_transforms(ctx, state["fp"].handle, state["frames"], 0, state["T"],
                                                state["radius"], scales=state["scales"]))
    if kind == "serve":
        tickets = [P.prnu_submit_video(ctx, fp.handle, W, o) for fp, W, o in state["videos"]]
        return [_found(P.prnu_poll(ctx, t, len(W))[1]) for t, (_, W, _) in zip(tickets, state["videos"])]
    if kind == "residuals":
        return P.prnu_extract_residuals(ctx, state["images"], 3.0, out=state["out"])
    return P.prnu_estimate_fingerprint(ctx, state["images"], state["residuals"], out=state["out"])


# ---------------------------------------------------------------------------
# What a pass cannot do without.

def _candidate_flops(M, N, Mf, Nf, radius):
    """Warp (two coordinates, three interpolations), real 2-D DFT, product and energy,
    inverse column DFTs, inverse row DFTs of the rows the peak and its block can lie in."""
    band = M - Mf + 2 * radius + 11
    fft = 2.5 * M * N * math.log2(M * N)
    return 14.0 * Mf * Nf + fft + 4.5 * M * N + 2.5 * M * N * math.log2(M) + 2.5 * band * N * math.log2(N)


def work(case):
    kind, M, N = case["kind"], case["M"], case["N"]
    if kind == "residuals":
        # per level: analysis and synthesis (8 taps, both directions), windows and Wiener
        return dict(bytes=8.0 * case["L"] * M * N, flops=4.0 / 3.0 * case["L"] * M * N * (2 * 32 + 40))
    if kind == "estimate":
        return dict(bytes=4.0 * M * N * (2 * case["L"] + 1), flops=4.0 * case["L"] * M * N)
    if kind == "serve":
        b = f = 0.0
        for v in range(case["videos"]):
            m, n = (M, N) if v % 2 == 0 else (case["M2"], case["N2"])
            R = min(case["radius"], (min(m, n) - 11) // 2)
            # the first frame's full grid, then local grids; a foreign video's fall back
            later = 942 if v % 4 >= 2 else 81
            b += 4.0 * m * n * (case["F"] + 1)
            f += (861 + (case["F"] - 1) * later) * _candidate_flops(m, n, m, n, R)
        return dict(bytes=b, flops=f)
    Mf, Nf, F, R = case["Mf"], case["Nf"], case["F"], case["radius"]
    n = case["n_scale"] * case["n_rot"] * F
    if case["mode"] == "warm":
        n = 861 + 81 * (F - 1)
    if case["mode"] == "refine":
        n = (1111 + 121) * F
    return dict(bytes=4.0 * M * N + F * Mf * Nf * (2.0 if case["dtype"] == "bf16" else 4.0) + 24.0 * n,
                flops=n * _candidate_flops(M, N, Mf, Nf, R))


# ---------------------------------------------------------------------------
# The same in 64 bits.

def _bilinear64(pad, bx, by, Mf, Nf):
    """Bilinear samples of the frame behind `pad` (two zero pixels on each side)."""
    bx, by = bx.clamp(-1.0, float(Nf)), by.clamp(-1.0, float(Mf))
    x0, y0 = torch.floor(bx), torch.floor(by)
    fx, fy = bx - x0, by - y0
    i = (y0.long() + 2) * (Nf + 4) + x0.long() + 2
    flat = pad.reshape(-1)
    top = flat[i] * (1 - fx) + flat[i + 1] * fx
    bot = flat[i + Nf + 4] * (1 - fx) + flat[i + Nf + 5] * fx
    return top * (1 - fy) + bot * fy


class _Exact:
    """Candidates of one frame against one fingerprint: Eq. (1) at every circular shift
    by FFT, Eq. (3) with the energy summed directly."""

    def __init__(self, K, W, radius):
        self.M, self.N = K.shape
        self.Mf, self.Nf = W.shape
        K = K.double()
        K = K - K.mean()
        self.norm = torch.sqrt((K * K).sum())
        self.FK = torch.fft.rfft2(K)
        self.pad = torch.nn.functional.pad(W.double(), (2, 2, 2, 2))
        d = dict(device="cuda", dtype=torch.float64)
        self.ux = (torch.arange(self.Nf, **d) - (self.Nf - 1) / 2)[None, :]
        self.uy = (torch.arange(self.Mf, **d) - (self.Mf - 1) / 2)[:, None]
        self.radius = radius
        self.rows = torch.arange(-radius, self.M - self.Mf + radius + 1, device="cuda")
        self.cols = torch.arange(-radius, self.N - self.Nf + radius + 1, device="cuda")
        self.block = torch.arange(-5, 6, device="cuda")

    def similarity(self, s, t):
        c, n = math.cos(math.radians(t)), math.sin(math.radians(t))
        return self.score((c * self.ux - n * self.uy) / s, (n * self.ux + c * self.uy) / s, None)

    def matrix(self, T):
        G = np.linalg.inv(T)
        X, Y, Z = (float(G[k, 0]) * self.ux + float(G[k, 1]) * self.uy + float(G[k, 2]) for k in range(3))
        return self.score(X / Z, Y / Z, Z > 0)

    def score(self, bx, by, valid):
        M, N, Mf, Nf = self.M, self.N, self.Mf, self.Nf
        w = _bilinear64(self.pad, bx + (Nf - 1) / 2, by + (Mf - 1) / 2, Mf, Nf)
        if valid is not None:
            w = torch.where(valid, w, torch.zeros_like(w))
        if (Mf, Nf) != (M, N):
            w = torch.nn.functional.pad(w, (0, N - Nf, 0, M - Mf))
        w = w - w.mean()
        C = torch.fft.irfft2(self.FK * torch.fft.rfft2(w).conj(), s=(M, N))
        win = C[(self.rows % M)[:, None], (self.cols % N)[None, :]].reshape(-1)
        k = torch.argmax(win)
        dy, dx = self.rows[k // len(self.cols)], self.cols[k % len(self.cols)]
        ex = C[((dy + self.block) % M)[:, None], ((dx + self.block) % N)[None, :]]
        off = (C * C).sum() - (ex * ex).sum()
        pk = win[k]
        return torch.stack((pk * pk.abs() * (M * N - 121) / off, pk / (self.norm * torch.sqrt((w * w).sum()))))


def _nodes(n, lo, hi):
    return [(lo + hi) / 2 + (k - (n - 1) / 2) * ((hi - lo) / (n - 1) if n > 1 else 0.0) for k in range(n)]


def _around(n, centre, step):
    return [centre + (k - (n - 1) / 2) * step for k in range(n)]


def _best64(ex, scales, rots, best=None):
    """(pce, rho, scale, rot) of the best candidate of a grid, or `best` if that is higher."""
    cand = [(s, t) for s in scales for t in rots]
    v = torch.stack([ex.similarity(s, t) for s, t in cand]).cpu().numpy()
    k = int(np.argmax(v[:, 0]))
    here = (float(v[k, 0]), float(v[k, 1]), *cand[k])
    return here if best is None or here[0] > best[0] else best


def _search64(K, W, radius, grid, mode):
    full = (_nodes(*grid[:3]), _nodes(*grid[3:]))
    pce, rho, last = [], [], None
    for w in W:
        ex = _Exact(K, w, radius)
        if mode == "refine":
            s, t, best = 1.0, 0.0, None
            for n in range(1, 4):
                f = 10.0 ** (1 - n)
                seg = _best64(ex, _around(11, s, 0.01 * f), _nodes(101, -5.0, 5.0) if n == 1 else _around(11, t, 0.1 * f))
                best = seg if best is None or seg[0] > best[0] else best
                if seg[2:] == (s, t):
                    break
                s, t = seg[2:]
        elif mode == "warm" and last is not None:
            best = _best64(ex, _around(LOCAL[0], last[2], LOCAL[2]), _around(LOCAL[1], last[3], LOCAL[3]))
            if best[0] < 60.0:
                best = _best64(ex, *full, best)
        else:
            best = _best64(ex, *full)
        last = best
        pce.append(best[0])
        rho.append(best[1])
    return dict(pce=np.array(pce), rho=np.array(rho), dx=None, dy=None, scale=None, rot_deg=None, cand_index=None,
                n_evaluated=None)


_H = (0.23037781330889650, 0.71484657055291565, 0.63088076792985890, -0.02798376941685985, -0.18703481171909309,
      0.03084138183556076, 0.03288301166688520, -0.01059740178506903)
_G = tuple((-1) ** k * _H[7 - k] for k in range(8))


def _analyse(x, f, axis):
    n = torch.arange(x.shape[axis] // 2, device="cuda")
    return sum(f[k] * x.index_select(axis, (2 * n + k) % x.shape[axis]) for k in range(8))


def _synthesise(lo, hi, axis):
    n = torch.arange(lo.shape[axis], device="cuda")
    L = 2 * lo.shape[axis]
    shape = list(lo.shape)
    shape[axis] = L
    out = torch.zeros(shape, device="cuda", dtype=torch.float64)
    for k in range(8):
        out.index_add_(axis, (2 * n + k) % L, _H[k] * lo + _G[k] * hi)
    return out


def _window_mean(q, w):
    h = w // 2
    p = torch.nn.functional.pad(q, (h, h, h, h))
    r = sum(p[:, k:k + q.shape[1]] for k in range(w))
    return sum(r[k:k + q.shape[0]] for k in range(w)) / (w * w)


def _residual64(img, s0):
    M, N = img.shape
    M2, N2 = (M + 15) // 16 * 16, (N + 15) // 16 * 16
    iy, ix = torch.arange(M2, device="cuda"), torch.arange(N2, device="cuda")
    x = img.double()[torch.where(iy < M, iy, 2 * (M - 1) - iy)][:, torch.where(ix < N, ix, 2 * (N - 1) - ix)]
    details = []
    for _ in range(4):
        lo, hi = _analyse(x, _H, 1), _analyse(x, _G, 1)
        details.append([_analyse(lo, _G, 0), _analyse(hi, _H, 0), _analyse(hi, _G, 0)])
        x = _analyse(lo, _H, 0)
    x = torch.zeros_like(x)
    for level in reversed(details):
        kept = []
        for c in level:
            m = torch.stack([_window_mean(c * c, w) for w in (3, 5, 7, 9)]).amin(0)
            v = (m - s0 * s0).clamp_min(0.0)
            kept.append(c * (s0 * s0 / (v + s0 * s0)))
        x = _synthesise(_synthesise(x, kept[0], 0), _synthesise(kept[1], kept[2], 0), 1)
    return x[:M, :N]


def exact(case, seed):
    kind = case["kind"]
    if kind == "residuals":
        return torch.stack([_residual64(i, 3.0) for i in _images(seed, case["L"], case["M"], case["N"])])
    if kind == "estimate":
        I, W = (x.double() for x in _estimate_inputs(seed, case["L"], case["M"], case["N"]))
        return (I * W).sum(0) / (I * I).sum(0)
    if kind == "serve":
        return [_search64(K, W, R, FULL, "warm") for M, N, R, K, W in _videos(case, seed)]
    K, W = _video(seed, case["M"], case["N"], case["Mf"], case["Nf"], case["F"], case["radius"])
    W, scales = _store(W, case["dtype"])
    if scales is not None:
        W = W.double() * scales[:, None, None].double()
    if kind == "search":
        return _search64(K, W, case["radius"], _grid(case), case["mode"])
    ex = _Exact(K, W[0], case["radius"])
    if kind == "transforms":
        v = [ex.matrix(T) for T in _transforms(seed, case["n_scale"])]
    else:
        g = _grid(case)
        v = [ex.similarity(s, t) for s in _nodes(*g[:3]) for t in _nodes(*g[3:])]
    v = torch.stack(v).cpu().numpy()
    return dict(pce=v[:, 0], rho=v[:, 1], dx=None, dy=None)
