"""The work that programs built on this framework have it do, as measurable
cases: one pass of a public entry point on inputs made from a seed.

listed() names twelve of them, draw() gives more of the same ranges, prepare()
makes what a program holds before the call (descriptors in GPU memory, a
parameter set, measured times, a reused workspace), run() is one pass, work()
the bytes and operations a pass cannot do without, and exact() the same results
from plain torch in float64, written from the model's formulas alone.

Inputs follow the distributions of the seeded generators in synth.py; they are
drawn here on the GPU, since a sweep of 2^24 rows takes seconds on the host.
"""
import math

import numpy as np
import torch

from paper_2605_04178_amd import synth
from paper_2605_04178_amd import wavemodel as wm

DEV = "cuda"
MIB = float(1 << 20)


def listed():
    return [
        # a scheduler asks for the times of a handful of candidate kernels: the
        # smallest call, where only its latency counts
        {"name": "few_kernels", "path": "predict", "n": 48, "levels": 4, "combine": 0, "occ": True},
        # the headline sweep: every point of a design-space study
        {"name": "predict_sweep", "path": "predict", "n": 1 << 24, "levels": 4, "combine": 0, "occ": True},
        # one step of a torch training loop over a ragged set of measurements,
        # three-level hierarchy and the occupancy-overlap combine: forward and
        # backward through the autograd function
        {"name": "autograd_step", "path": "autograd", "n": 50_021, "levels": 3, "combine": 1},
        # loss and gradient over the headline sweep (forward and adjoint)
        {"name": "loss_grad_sweep", "path": "loss_grad", "n": 1 << 24, "levels": 4, "combine": 0, "exact": False},
        # the tiles of every GEMM shape of a library's tuning table
        {"name": "tile_sweep", "path": "tiles", "shapes": 1 << 16, "cmax": 96},
        # a calibration with the default step count
        {"name": "calibrate", "path": "calibrate", "n": 1 << 20, "levels": 4, "combine": 0, "steps": 500},
        # six architectures fitted together, hierarchies and sizes mixed
        {"name": "calibrate_sets", "path": "sets", "sets": 6, "lo": 1 << 18, "hi": 1 << 22, "steps": 120},
        # the application times of one benchmark suite
        {"name": "suite_totals", "path": "totals", "apps": 31, "smax": 12},
        # application-level loss and gradient over a large corpus of applications
        {"name": "app_loss_grad", "path": "app_grad", "apps": 1 << 20, "smax": 12},
        # fusion plans of every operator chain of a compiler's corpus
        {"name": "fusion_plan", "path": "plan", "chains": 1 << 16, "lmax": 16, "R": 8},
        # per-case multipliers with a training / held-out split
        {"name": "multipliers", "path": "multipliers", "groups": 1 << 16, "gmax": 40},
        # the second model family: loss and gradient over its sweep
        {"name": "blackwell_loss_grad", "path": "bw_loss_grad", "n": 1 << 24},
    ]


def draw(rng):
    """One more case: any of the paths, sizes spread over their logarithm."""
    def logi(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    model = {"levels": rng.choice([3, 4]), "combine": rng.choice([0, 1])}
    path = rng.choice(["predict", "predict", "loss_grad", "loss_grad", "autograd", "tiles", "tiles", "calibrate",
                       "sets", "totals", "totals", "app_grad", "app_grad", "plan", "plan", "multipliers",
                       "multipliers", "bw_predict", "bw_loss_grad"])
    if path == "predict":
        return {"path": path, "n": logi(1, 1 << 24), **model, "occ": rng.random() < 0.7}
    if path == "loss_grad":
        return {"path": path, "n": logi(64, 1 << 24), **model, "exact": rng.random() < 0.25}
    if path == "autograd":
        return {"path": path, "n": logi(64, 1 << 22), **model}
    if path == "tiles":
        cmax = logi(12, 384)
        return {"path": path, "shapes": logi(1, (1 << 16) * 96 // max(96, cmax)), "cmax": cmax}
    if path == "calibrate":
        return {"path": path, "n": logi(1 << 12, 1 << 20), **model, "steps": logi(20, 400)}
    if path == "sets":
        hi = logi(1 << 14, 1 << 21)
        return {"path": path, "sets": rng.randrange(2, 8), "lo": max(1 << 12, hi // 16), "hi": hi,
                "steps": logi(20, 120)}
    if path in ("totals", "app_grad"):
        return {"path": path, "apps": logi(4, 1 << 20), "smax": rng.choice([4, 8, 12])}
    if path == "plan":
        R, lmax = rng.choice([2, 4, 6, 8, 8, 16]), rng.choice([4, 8, 12, 16, 24, 40])
        most = (1 << 16) * 72 // (min(R, lmax) * (lmax // 2 + 1))
        return {"path": path, "chains": logi(1, min(1 << 16, most)), "lmax": lmax, "R": R}
    if path == "multipliers":
        gmax = logi(6, 150)
        return {"path": path, "groups": logi(1, min(1 << 16, (1 << 16) * 40 // gmax)), "gmax": gmax}
    return {"path": path, "n": logi(1, 1 << 24) if path == "bw_predict" else logi(64, 1 << 24)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Draws:
    """Seeded draws on the GPU, with the shorthands the distributions need."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 2 + 1)

    def u(self, n, lo=0.0, hi=1.0):
        return lo + (hi - lo) * torch.rand(n, generator=self.g, device=DEV, dtype=torch.float64)

    def logu(self, n, lo, hi):
        return torch.exp(self.u(n, math.log(lo), math.log(hi)))

    def i(self, n, lo, hi):
        """Integers in [lo, hi)."""
        return torch.randint(lo, hi, (n,), generator=self.g, device=DEV)

    def pick(self, n, values):
        return torch.tensor(values, device=DEV)[self.i(n, 0, len(values))]

    def chance(self, n, p):
        return self.u(n) < p

    def noise(self, n, sigma):
        return torch.exp(sigma * torch.randn(n, generator=self.g, device=DEV, dtype=torch.float64))


def f32(x):
    return x.to(torch.float32).contiguous()


def i32(x):
    return x.to(torch.int32).contiguous()


def descriptors(r, n, vmax=512):
    """The general kernel sweep (synth.descriptors)."""
    zero = torch.zeros(n, device=DEV, dtype=torch.float64)
    one = torch.ones(n, device=DEV, dtype=torch.int64)
    gp = (r.pick(n, [64, 128, 256, 512, 1024]) | (r.i(n, 0, 5) << 11)
          | ((torch.where(r.chance(n, 0.5), one, r.i(n, 2, 9)) - 1) << 14)
          | ((torch.where(r.chance(n, 0.5), one, r.i(n, 2, 9)) - 1) << 17)
          | (r.chance(n, 0.25).to(torch.int64) << 20)
          | (torch.where(r.chance(n, 0.5), one * 0, r.i(n, 1, 16)) << 21))
    return {"F": f32(r.logu(n, 1e6, 1e13)), "B": f32(r.logu(n, 1e4, 1e11)),
            "r1": f32(r.u(n)), "r2": f32(r.u(n)), "r3": f32(r.u(n)),
            "K": f32(torch.round(r.logu(n, 1.0, 4096.0))), "u": f32(r.u(n, 0.4, 0.7)),
            "W": f32(torch.where(r.chance(n, 0.5), zero, r.logu(n, MIB, 4096.0 * MIB))),
            "vgpr": i32(r.i(n, 16, vmax + 1)), "lds": i32(r.i(n, 0, 65537)), "gpack": i32(gp),
            "grid": i32(torch.round(r.logu(n, 1.0, float(1 << 20))))}


def calibration_descriptors(r, n):
    """Half general sweep, half memory-streaming kernels over the working-set
    regimes (synth.calibration_descriptors)."""
    ns = n // 2
    a, s = descriptors(r, n - ns), descriptors(r, ns, 128)
    B = r.logu(ns, 1e8, 1e11)
    sel = r.u(ns)
    W = torch.where(sel < 0.3, torch.zeros_like(B),
                    torch.where(sel < 0.5, r.u(ns, 205.5, 255.5) * MIB, r.logu(ns, 8.0 * MIB, 2048.0 * MIB)))
    s.update(B=f32(B), F=f32(B * r.logu(ns, 1e-3, 1e-1)), r1=f32(r.u(ns, 0.0, 0.2)), r2=f32(r.u(ns, 0.0, 0.2)),
             W=f32(W), grid=i32(torch.round(r.logu(ns, 4096.0, float(1 << 20)))), lds=i32(r.i(ns, 0, 16385)),
             K=f32(torch.round(r.logu(ns, 1.0, 64.0))))
    return {k: torch.cat([a[k], s[k]]) for k in a}


def counts(r, n, lo, hi):
    """List lengths uniform over [lo, hi], in an order of the seed's: a case
    has the same number of rows whatever the seed."""
    return (lo + torch.arange(n, device=DEV) % (hi - lo + 1))[torch.randperm(n, generator=r.g, device=DEV)]


def offsets(counts):
    return i32(torch.cat([torch.zeros(1, device=DEV, dtype=torch.int64), torch.cumsum(counts, 0)]))


def bw_descriptors(r, n):
    """Blackwell tile kernels (synth.bw_descriptors)."""
    one = torch.ones(n, device=DEV, dtype=torch.int64)
    comp = r.chance(n, 0.25)
    fl = (r.i(n, 0, 5) | (r.i(n, 0, 2) << 3) | (r.i(n, 0, 2) << 4)
          | ((torch.where(r.chance(n, 0.5), one, r.pick(n, [1, 2, 4])) - 1) << 5)
          | ((torch.where(r.chance(n, 0.5), one, r.pick(n, [1, 2, 4])) - 1) << 9)
          | (r.i(n, 1, 3) << 13) | (comp.to(torch.int64) << 16))
    return {"bM": i32(r.pick(n, [64, 128, 256])), "bN": i32(r.pick(n, [64, 128, 256])),
            "bK": i32(r.pick(n, [16, 32, 64, 128])), "G": i32(torch.round(r.logu(n, 1.0, 65536.0))),
            "flags": i32(fl), "Kt": f32(torch.round(r.logu(n, 1.0, 1024.0))),
            "CR": f32(torch.where(comp, r.u(n, 1.0, 4.0), torch.ones(n, device=DEV, dtype=torch.float64))),
            "ob": f32(r.pick(n, [2.0, 4.0]))}


def inputs(case, seed):
    """The case's data: tensors on the GPU and parameter sets.  Measured times
    are the float64 model's under a true parameter set, times noise; the
    program's own set is off by up to 1.5 in every fitted slot."""
    r = Draws(seed)
    path = case["path"]
    if path in ("predict", "loss_grad", "autograd", "calibrate"):
        n = case["n"]
        true = synth.param_set(seed % 1000, n_levels=case["levels"], combine=case["combine"])
        d = calibration_descriptors(r, n) if path == "calibrate" else descriptors(r, n)
        if path == "predict":
            return {"p": true, "d": d}
        mask = synth.fit_mask(case["levels"])
        p = synth.perturb_theta(true, seed % 1000 + 1, mask=mask)
        m = f32(cdna_times(d, true, theta_of(true)) * r.noise(n, 0.02))
        if path == "autograd":
            T = cdna_times(d, p, theta_of(p))
            w = torch.where(torch.isfinite(T) & torch.isfinite(m), torch.sign(T - m) / (m * n), torch.zeros_like(T))
            return {"p": p, "d": d, "w": f32(w)}
        return {"p": p, "d": d, "m": m, "mask": mask}
    if path == "sets":
        out = []
        for k, true in enumerate(synth.multi_arch_sets(seed % 1000, case["sets"])):
            lo, hi = math.log(case["lo"]), math.log(case["hi"])
            # the sizes are the case's own, spread over its range
            n = int(round(math.exp(lo + (hi - lo) * ((k * 0.618034 + 0.37) % 1.0))))
            d = calibration_descriptors(r, n)
            mask = synth.fit_mask(true.n_levels)
            out.append({"d": d, "m": f32(cdna_times(d, true, theta_of(true)) * r.noise(n, 0.02)), "mask": mask,
                        "p": synth.perturb_theta(true, seed % 1000 + 140 + k, mask=mask)})
        return {"sets": out}
    if path == "tiles":
        n, cmax = case["shapes"], case["cmax"]
        cnt = counts(r, n, min(8, cmax), cmax)
        # candidates drawn without replacement: the first cnt of a random
        # order of the 384 tiles, shapes in slices to bound the memory
        codes = torch.from_numpy(synth.all_tile_codes().astype(np.int32)).to(DEV)
        parts = []
        for a in range(0, n, 8192):
            c = cnt[a:a + 8192]
            order = torch.argsort(torch.rand((len(c), len(codes)), generator=r.g, device=DEV), dim=1)
            keep = torch.arange(len(codes), device=DEV)[None, :] < c[:, None]
            parts.append(codes[order[keep]])
        dim = lambda: i32(torch.round(r.logu(n, 128.0, 16384.0)))
        return {"p": synth.param_set(seed % 1000), "M": dim(), "N": dim(), "K": dim(), "dtype": i32(r.i(n, 0, 4)),
                "off": offsets(cnt), "code": torch.cat(parts).contiguous()}
    if path in ("totals", "app_grad"):
        na = case["apps"]
        cnt = counts(r, na, 1, case["smax"])
        off = offsets(cnt)
        n = int(off[-1])
        zero = torch.zeros(n, device=DEV, dtype=torch.float64)
        sg = {"app_off": off, "n_exec": f32(torch.round(r.logu(n, 1.0, 1e4))), "n_kern": i32(r.i(n, 1, 5)),
              "cls": i32(r.i(n, 0, 4)), "h2d": f32(torch.where(r.chance(n, 0.5), zero, r.logu(n, 1e3, 1e9))),
              "d2h": f32(torch.where(r.chance(n, 0.5), zero, r.logu(n, 1e3, 1e9)))}
        p, q = synth.param_set(seed % 1000), synth.seg_params(seed % 1000 + 7)
        x = {"p": p, "q": q, "d": descriptors(r, n, 128), "sg": sg}
        if path == "app_grad":
            x["m"] = f32(app_times(x, theta_of(p), segvec_of(q))[0] * r.noise(na, 0.05))
            x["p"] = synth.perturb_theta(p, seed % 1000 + 152, factor=1.2)
        return x
    if path == "plan":
        cnt = counts(r, case["chains"], 2, case["lmax"])
        off = offsets(cnt)
        n = int(off[-1])
        d = descriptors(r, n, 128)
        B = d["B"].to(torch.float64)
        nxt = torch.cat([B[1:], torch.zeros(1, device=DEV, dtype=torch.float64)])
        edge = r.u(n, 0.05, 0.45) * torch.minimum(B, nxt)
        edge[off[1:].to(torch.int64) - 1] = 0.0
        return {"p": synth.param_set(seed % 1000), "d": d, "edge": f32(edge), "off": off}
    if path == "multipliers":
        ng = case["groups"]
        cnt = counts(r, ng, 1, case["gmax"])
        off = offsets(cnt)
        n = int(off[-1])
        p = synth.param_set(seed % 1000)
        T = f32(cdna_times(descriptors(r, n, 128), p, theta_of(p)))
        factor = torch.repeat_interleave(r.logu(ng, 0.5, 2.0), cnt)
        return {"T": T, "m": f32(T.to(torch.float64) * factor * r.noise(n, 0.05)), "off": off,
                "train": (~r.chance(n, 1.0 / 3.0)).to(torch.uint8).contiguous()}
    n = case["n"]
    p = synth.bw_param_set(seed % 1000)
    d = bw_descriptors(r, n)
    if path == "bw_predict":
        return {"p": p, "d": d}
    true = synth.bw_param_set(seed % 1000 + 1)
    return {"p": p, "d": d, "m": f32(bw_times(d, true, theta_of(true)) * r.noise(n, 0.02))}


def prepare(case, seed):
    """What a program has in hand before the call."""
    x = inputs(case, seed)
    path = case["path"]
    s = {"path": path, "case": dict(case)}
    if path == "sets":
        s["descs"] = [wm.DeviceDescriptors(k["d"]) for k in x["sets"]]
        s["meas"] = [k["m"] for k in x["sets"]]
        s["p0"] = [k["p"] for k in x["sets"]]
        s["opts"] = [wm.calib_opts(steps=case["steps"], free_mask=k["mask"]) for k in x["sets"]]
        return s
    if path == "tiles":
        s["shapes"] = wm.DeviceShapes(x["M"], x["N"], x["K"], x["dtype"], x["off"], x["code"])
        s["p"] = x["p"]
        return s
    if path.startswith("bw"):
        s["desc"] = wm.DeviceBwDescriptors(x["d"])
        if path == "bw_loss_grad":
            s["ws"] = wm._workspace(wm.bw_workspace_bytes(wm.BW_OP_GRAD, case["n"]), DEV)
    elif path != "multipliers":
        s["desc"] = wm.DeviceDescriptors(x["d"])
    if path in ("totals", "app_grad"):
        s["segs"] = wm.DeviceSegments(x["sg"])
        if path == "app_grad":
            s["ws"] = wm._workspace(wm.apps_workspace_bytes(s["segs"].n, s["segs"].n_apps), DEV)
    elif path == "loss_grad":
        s["ws"] = wm._workspace(wm.workspace_bytes(wm.OP_LOSS_GRAD, case["n"]), DEV)
    elif path == "calibrate":
        s["ws"] = wm._workspace(wm.workspace_bytes(wm.OP_CALIBRATE, case["n"], 1, case["steps"]), DEV)
    elif path == "plan":
        s["ws"] = wm._workspace(wm.plan_workspace_bytes(s["desc"].n, case["R"]), DEV)
    elif path == "multipliers":
        s["ws"] = wm._workspace(wm.workspace_bytes(wm.OP_FIT_MULTIPLIERS, x["T"].numel()), DEV)
    elif path == "autograd":
        s["theta"] = torch.tensor(x["p"].theta, dtype=torch.float64)
    for k in ("p", "q", "m", "w", "mask", "edge", "off", "T", "train"):
        if k in x:
            s[k] = x[k]
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    path, case = state["path"], state["case"]
    if path == "predict":
        return wm.predict(state["desc"], state["p"], want_occ=case["occ"])
    if path == "loss_grad":
        return wm.loss_grad(state["desc"], state["m"], state["p"], ws=state["ws"], exact=case["exact"])
    if path == "autograd":
        theta = state["theta"].clone().requires_grad_()
        T = wm.WMPredict.apply(state["desc"], theta, state["p"])
        T.backward(state["w"])
        return T.detach(), theta.grad
    if path == "tiles":
        return wm.select_tile(state["shapes"], state["p"])
    if path == "calibrate":
        return wm.calibrate(state["desc"], state["m"], state["p"], steps=case["steps"], free_mask=state["mask"],
                            ws=state["ws"])
    if path == "sets":
        return wm.calibrate_batched(state["descs"], state["meas"], state["p0"], state["opts"])
    if path == "totals":
        return wm.predict_apps(state["desc"], state["segs"], state["p"], state["q"])[0]
    if path == "app_grad":
        return wm.apps_loss_grad(state["desc"], state["segs"], state["m"], state["p"], state["q"], ws=state["ws"])
    if path == "plan":
        return wm.plan_fusion(state["desc"], state["edge"], state["off"], state["p"], case["R"], ws=state["ws"])
    if path == "multipliers":
        return wm.fit_multipliers(state["T"], state["m"], state["off"], state["train"], ws=state["ws"])
    if path == "bw_predict":
        return wm.bw_predict(state["desc"], state["p"])
    return wm.bw_loss_grad(state["desc"], state["m"], state["p"], ws=state["ws"])


# One evaluation of the model is about 60 float operations, with its adjoint
# about 130; a descriptor is 48 bytes (Blackwell: 32), a segment row 20 more.
EVAL, ADJ = 60, 130


def work(case):
    path = case["path"]
    if path == "predict":
        n = case["n"]
        return {"bytes": n * (52 + 4 * case["occ"]), "flops": n * EVAL}
    if path == "loss_grad":
        return {"bytes": case["n"] * 52 + 208, "flops": case["n"] * ADJ}
    if path == "autograd":    # forward reads 48 and writes 4, backward reads 52
        return {"bytes": case["n"] * 104 + 192, "flops": case["n"] * (EVAL + ADJ)}
    if path == "calibrate":   # every step looks at every measurement
        return {"bytes": case["steps"] * case["n"] * 52, "flops": case["steps"] * case["n"] * ADJ}
    if path == "sets":
        lo, hi = math.log(case["lo"]), math.log(case["hi"])
        n = sum(int(round(math.exp(lo + (hi - lo) * ((k * 0.618034 + 0.37) % 1.0)))) for k in range(case["sets"]))
        return {"bytes": case["steps"] * n * 52, "flops": case["steps"] * n * ADJ}
    if path == "tiles":
        cand = case["shapes"] * (min(8, case["cmax"]) + case["cmax"]) / 2
        return {"bytes": case["shapes"] * 33 + cand * 4, "flops": cand * 90}
    if path in ("totals", "app_grad"):
        rows = case["apps"] * (1 + case["smax"]) / 2
        return {"bytes": rows * 68 + case["apps"] * 8, "flops": rows * ((EVAL if path == "totals" else ADJ) + 20)}
    if path == "plan":
        L, R = (2 + case["lmax"]) / 2, case["R"]
        runs = case["chains"] * sum(max(0.0, L - k) for k in range(R))
        return {"bytes": case["chains"] * (L * 53 + 20), "flops": runs * (EVAL + 30)}
    if path == "multipliers":
        rows = case["groups"] * (1 + case["gmax"]) / 2
        return {"bytes": rows * 13 + case["groups"] * 12, "flops": rows * (6 + 2 * math.log2(case["gmax"]))}
    return {"bytes": case["n"] * (40 if path == "bw_predict" else 36), "flops": case["n"] * 100}


# ---------------------------------------------------------------------------
# the same results from plain torch in float64
# ---------------------------------------------------------------------------
def theta_of(p):
    return torch.tensor(p.theta, dtype=torch.float64, device=DEV)


def segvec_of(q):
    return torch.tensor(list(q.kappa) + [q.bw_h2d, q.bw_d2h, q.tau_memcpy], dtype=torch.float64, device=DEV)


def ceil_div(a, b):
    return torch.div(a + b - 1, b, rounding_mode="floor")


def cdna_times(d, p, th):
    """Kernel times of the CDNA wavefront-centric model in float64 (+inf for a
    kernel that does not fit), differentiable in th."""
    x = {k: v.to(torch.int64 if k in ("vgpr", "lds", "gpack", "grid") else torch.float64) for k, v in d.items()}
    gp, G = x["gpack"], x["grid"]
    dt = (gp >> 11) & 7
    # occupancy and rounds
    k = ceil_div(gp & 2047, p.wave)
    va = ceil_div(x["vgpr"], p.vgpr_gran) * p.vgpr_gran
    w = torch.where(va <= p.vgpr_simd, torch.clamp(p.vgpr_simd // va, max=p.waves_simd), torch.zeros_like(va))
    o = torch.div(p.n_simd * w, k, rounding_mode="floor")
    sa = ceil_div(x["lds"], p.lds_gran) * p.lds_gran
    o = torch.where(x["lds"] > 0, torch.minimum(o, p.lds_cu // torch.clamp(sa, min=1)), o)
    fits = o > 0
    o1 = torch.clamp(o, min=1)
    nr = ceil_div(G, p.n_cu * o1).to(torch.float64)
    # traffic
    h3, W = x["r3"], x["W"]
    if p.n_levels == 4:
        Wm = torch.where(W > 0, W, torch.full_like(W, MIB)) / MIB
        tr = ((p.c_llc_mib - Wm) / (p.c_llc_mib - p.w_lo_mib)).clamp(min=1e-300)
        h = torch.where(Wm < p.w_lo_mib, torch.ones_like(W),
                        torch.where(Wm <= p.c_llc_mib, tr ** th[20], (p.c_llc_mib / Wm) ** th[21]))
        h3 = torch.where(W > 0, h, h3)
    m1 = 1.0 - x["r1"]
    s1, s2, a12 = x["r1"], m1 * x["r2"], m1 * (1.0 - x["r2"])
    s3, sh = (a12 * h3, a12 * (1.0 - h3)) if p.n_levels == 4 else (torch.zeros_like(a12), a12)
    e = torch.where(W > 0, torch.exp(-W / th[22]), torch.zeros_like(W))
    bwh = th[3] + (th[23] - th[3]) * e
    S = s1 * th[0] + s2 * th[1] + s3 * th[2] + sh * bwh
    lat = (s1 * th[4] + s2 * th[5] + s3 * th[6] + sh * th[7]) / p.f_clk
    # stages
    Tc = x["F"] / (x["u"] * th[8:13][dt])
    Tb = x["B"] / S
    Tl = nr * x["B"] / (G.to(torch.float64) * k * p.bytes_inflight_wave) * lat
    Tm = torch.where(Tb >= Tl, Tb, Tl)
    if p.combine == 0:
        step = torch.where(Tc >= Tm, Tc, Tm)
    else:
        a = (o1 * k - 1).to(torch.float64)
        sat = a * Tc >= Tm
        eta = torch.where(sat, torch.ones_like(Tc), a * Tc / Tm)
        eta = torch.where(a == 0, torch.zeros_like(Tc), eta)
        step = (Tm + Tc) / (1.0 + eta)
    cnt = [((gp >> 14) & 7), ((gp >> 17) & 7), ((gp >> 20) & 1), ((gp >> 21) & 15)]
    Tov = th[13] + th[14] * G + th[15] * nr * x["K"]
    for j, c in enumerate(cnt):
        Tov = Tov + th[16 + j] * c
    return torch.where(fits, Tov + step, torch.full_like(step, math.inf))


def bw_times(d, p, th):
    """Kernel times of the Blackwell stage-centric model in float64."""
    x = {k: v.to(torch.float64 if k in ("Kt", "CR", "ob") else torch.int64) for k, v in d.items()}
    fl = x["flags"]
    dt, pair, sb = fl & 7, ((fl >> 3) & 1) == 1, ((fl >> 4) & 1) == 1
    PA, PB = (((fl >> 5) & 15) + 1).double(), (((fl >> 9) & 15) + 1).double()
    nbar, comp = ((fl >> 13) & 7).double(), ((fl >> 16) & 1) == 1
    f = p.f_clk
    acc = x["bM"] * x["bN"] * torch.where(dt == 0, 8, 4)
    cta = torch.clamp(p.tmem_bytes // acc, max=p.max_cta)
    fits = cta > 0
    nr = ceil_div(x["G"], p.n_sm * torch.clamp(cta, min=1)).double()
    e = 2.0 ** (3 - dt).double()
    bM, bN, bK, Kt = x["bM"].double(), x["bN"].double(), x["bK"].double(), x["Kt"]
    MA, MB, D = bM * bK * e, bN * bK * e, acc.double()
    zero = torch.zeros_like(MA)
    tmem = (D + torch.where(sb, MA, zero)) / th[0] + th[2] / f + D / th[1]
    Tc = 2.0 * bM * bN * bK / (th[3:8][dt] * torch.where(pair, th[8], torch.ones_like(th[8]))) + tmem + th[20] / f / Kt
    tma = th[9] / f + (MA / PA + torch.where(pair, 0.5 * MB, MB) / PB) / th[10]
    dsm = torch.where(pair, 0.5 * MB / th[23], zero)
    de = torch.where(comp, (MA + MB) / (x["CR"] * th[13] * th[14]), zero)
    up = torch.where(dt == 4, (MA + MB) / th[15] + th[16] / f, zero)
    sync = nbar * th[11] / f + torch.where(pair, th[12] / f, zero)
    Tio = th[17] * (tma + de + up + dsm) + sync
    step = torch.where(Tc >= Tio, Tc, Tio) + sync + th[21]
    store = bM * bN * x["ob"] / th[18] + th[19] / f
    T = th[22] + nr * (Kt * step + store)
    return torch.where(fits, T, torch.full_like(T, math.inf))


def app_times(x, th, sv):
    """(application times, rows' finite mask) in float64."""
    sg = {k: v.to(torch.int64 if k in ("app_off", "n_kern", "cls") else torch.float64) for k, v in x["sg"].items()}
    T = cdna_times(x["d"], x["p"], th)
    t = sv[:4][sg["cls"]] * T + (sg["n_kern"] - 1) * th[13]
    for b, s in (("h2d", sv[4]), ("d2h", sv[5])):
        t = t + torch.where(sg[b] > 0, sg[b] / s + sv[6], torch.zeros_like(t))
    t = sg["n_exec"] * t
    na = sg["app_off"].numel() - 1
    owner = torch.repeat_interleave(torch.arange(na, device=DEV), sg["app_off"][1:] - sg["app_off"][:-1])
    return torch.zeros(na, dtype=torch.float64, device=DEV).index_add(0, owner, t), t


def loss_of(T, m):
    """(loss, count): mean |T - m| / m over finite times and measurements."""
    m = m.to(torch.float64)
    ok = torch.isfinite(T) & torch.isfinite(m) & (m > 0)
    z = torch.where(ok, (T - m).abs() / m, torch.zeros_like(T))
    n = int(ok.sum())
    return z.sum() / max(n, 1), n


def grad_call(times, m, th, *more):
    """[loss, count, gradients] as one float64 vector."""
    leaves = [v.clone().requires_grad_() for v in (th,) + more]
    loss, n = loss_of(times(*leaves), m)
    g = torch.autograd.grad(loss, leaves, allow_unused=True)
    g = [torch.zeros_like(v) if q is None else q for v, q in zip(leaves, g)]
    return torch.cat([loss.detach().reshape(1), torch.tensor([float(n)], dtype=torch.float64, device=DEV)] + g)


def adam(times, m, p, mask, steps, lr=0.05, lr_final=1e-3, b1=0.9, b2=0.999, eps=1e-8):
    """(theta, losses) of Adam on log(theta) over the mean relative error."""
    fit = torch.tensor([(mask >> j) & 1 for j in range(24)], dtype=torch.bool, device=DEV)
    th = theta_of(p)
    phi = torch.where(fit, torch.log(torch.where(fit, th, torch.ones_like(th))), torch.zeros_like(th))
    mo, ve, hist = torch.zeros_like(th), torch.zeros_like(th), []
    for k in range(steps):
        v = grad_call(times, m, th)
        hist.append(v[0])
        g = th * v[2:]
        mo, ve = b1 * mo + (1.0 - b1) * g, b2 * ve + (1.0 - b2) * g * g
        rate = lr * (lr_final / lr) ** (k / (steps - 1)) if steps > 1 else lr
        step = rate * (mo / (1.0 - b1 ** (k + 1))) / (torch.sqrt(ve / (1.0 - b2 ** (k + 1))) + eps)
        phi = torch.where(fit, phi - step, phi)
        th = torch.where(fit, torch.exp(phi), th)
    return th.cpu().numpy(), torch.stack(hist).cpu().numpy()


def tile_best(x):
    """The smallest float64 cost of each shape's candidate tiles."""
    off = x["off"].to(torch.int64)
    n = off.numel() - 1
    sh = torch.repeat_interleave(torch.arange(n, device=DEV), off[1:] - off[:-1])
    M, N, K, t = (x[k].to(torch.int64)[sh] for k in ("M", "N", "K", "dtype"))
    c = x["code"].to(torch.int64)
    mt, nt, kd = 32 << (c & 3), 32 << ((c >> 2) & 3), 16 << ((c >> 4) & 3)
    g = (((c >> 6) & 7) + 1) * x["p"].wave
    e = 8 >> t
    eo = torch.where(t == 3, 2 * torch.ones_like(e), e)
    gm, gn, Ks = ceil_div(M, mt), ceil_div(N, nt), ceil_div(K, kd)
    pan = (mt + nt) * kd * e
    Bi = (gm * gn * Ks * pan + M * N * eo).double()
    Ui = ((M * K + K * N) * e + M * N * eo).double()
    v = ceil_div(torch.where(t == 0, 2, 1) * mt * nt, g) + ceil_div(pan, 4 * g) + 16
    zero = torch.zeros_like(Bi)
    d = {"F": 2.0 * (gm * mt).double() * (gn * nt).double() * (Ks * kd).double(), "B": Bi, "r1": zero,
         "r2": (1.0 - Ui / Bi).clamp(min=0.0), "r3": zero, "K": Ks.double(), "u": zero + 1.0, "W": zero,
         "vgpr": v, "lds": 2 * pan, "gpack": g | (t << 11), "grid": gm * gn}
    T = cdna_times(d, x["p"], theta_of(x["p"]))
    T = torch.where((g <= 1024) & (gm * gn < 1 << 31), T, torch.full_like(T, math.inf))
    best = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
    return best.scatter_reduce(0, sh, T, "amin")


def plan_totals(x, R):
    """(planned, unfused) chain times: the prefix programme over every run of
    at most R kernels, all chains side by side."""
    p, th = x["p"], theta_of(x["p"])
    off = x["off"].to(torch.int64)
    a, L = off[:-1], off[1:] - off[:-1]
    d = {k: v.to(torch.int64 if k in ("vgpr", "lds", "gpack", "grid") else torch.float64) for k, v in x["d"].items()}
    edge, peak = x["edge"].to(torch.float64), th[8:13]
    inf = torch.full((len(a),), math.inf, dtype=torch.float64, device=DEV)
    best, unfused = [torch.zeros_like(inf)], torch.zeros_like(inf)
    for j in range(int(L.max())):
        here = j < L
        bj = inf
        s = None
        for ln in range(1, min(R, j + 1) + 1):
            at = torch.where(here, a + j - ln + 1, torch.zeros_like(a))
            y = {k: v[at] for k, v in d.items()}
            gp, dt = y["gpack"], (y["gpack"] >> 11) & 7
            f = [gp & 2047, (gp >> 14) & 7, (gp >> 17) & 7, (gp >> 21) & 15]
            tc = y["F"] / (y["u"] * peak[dt])
            # the run grows at its front; the dtype is the first row's with the most flops
            if s is None:
                s = {"F": y["F"], "B": y["B"], "E": torch.zeros_like(inf), "K": y["K"], "W": y["W"], "tc": tc,
                     "r": [y[k] * y["B"] for k in ("r1", "r2", "r3")], "top": y["F"], "dt": dt, "v": y["vgpr"],
                     "s": y["lds"], "G": y["grid"], "f": f}
                T = cdna_times(y, p, th)
                unfused = unfused + torch.where(here, T, torch.zeros_like(T))
            else:
                s["dt"] = torch.where(y["F"] >= s["top"], dt, s["dt"])
                s["top"] = torch.maximum(y["F"], s["top"])
                s.update(F=s["F"] + y["F"], B=s["B"] + y["B"], E=s["E"] + edge[at], K=s["K"] + y["K"],
                         W=s["W"] + y["W"], tc=s["tc"] + tc, v=torch.maximum(s["v"], y["vgpr"]),
                         s=torch.maximum(s["s"], y["lds"]), G=torch.maximum(s["G"], y["grid"]),
                         r=[q + y[k] * y["B"] for q, k in zip(s["r"], ("r1", "r2", "r3"))],
                         f=[torch.maximum(q, z) for q, z in zip(s["f"][:3], f[:3])] + [s["f"][3] + f[3]])
                z = {"F": s["F"], "B": (s["B"] - 2.0 * s["E"]).clamp(min=0.0), "K": s["K"],
                     "W": (s["W"] - s["E"]).clamp(min=0.0), "u": (s["F"] / (peak[s["dt"]] * s["tc"])).clamp(max=1.0),
                     "vgpr": s["v"], "lds": s["s"], "grid": s["G"],
                     "gpack": s["f"][0] | (s["dt"] << 11) | (s["f"][1] << 14) | (s["f"][2] << 17) | (1 << 20)
                     | (s["f"][3].clamp(max=15) << 21)}
                z.update({k: q / s["B"] for k, q in zip(("r1", "r2", "r3"), s["r"])})
                T = cdna_times(z, p, th)
            bj = torch.minimum(bj, best[j + 1 - ln] + T)
        best.append(torch.where(here, bj, best[-1]))
    return best[-1], unfused


def multipliers(x):
    """(multipliers, scaled times, [training error, rows, held-out error, rows])."""
    T, m = x["T"].to(torch.float64), x["m"].to(torch.float64)
    off = x["off"].to(torch.int64)
    ng = off.numel() - 1
    grp = torch.repeat_interleave(torch.arange(ng, device=DEV), off[1:] - off[:-1])
    ok = (T > 0) & torch.isfinite(T) & (m > 0) & torch.isfinite(m)
    use = torch.nonzero(ok & (x["train"] != 0)).reshape(-1)
    r, w, g = (m / T)[use], (T / m)[use], grp[use]
    o = torch.argsort(r, stable=True)
    o = o[torch.argsort(g[o], stable=True)]
    r, w, g = r[o], w[o], g[o]
    tot = torch.zeros(ng, dtype=torch.float64, device=DEV).index_add(0, g, w)
    c = torch.cumsum(w, 0)
    first = torch.searchsorted(g, torch.arange(ng, device=DEV))
    start = torch.cat([torch.zeros(1, dtype=torch.float64, device=DEV), c])[first]
    hit = torch.where(c - start[g] >= 0.5 * tot[g] * (1.0 - 1e-13), r, torch.full_like(r, math.inf))
    mult = torch.full((ng,), math.inf, dtype=torch.float64, device=DEV).scatter_reduce(0, g, hit, "amin")
    mult = torch.where(torch.isfinite(mult), mult, torch.ones_like(mult))
    Ts = mult[grp] * T
    err = torch.where(ok, (Ts - m).abs() / m, torch.zeros_like(T))
    tr = ok & (x["train"] != 0)
    held = ok & (x["train"] == 0)
    stats = torch.stack([err[tr].sum(), tr.sum().double(), err[held].sum(), held.sum().double()])
    return mult, Ts, stats


def exact(case, seed):
    x = inputs(case, seed)
    path = case["path"]
    if path == "predict":
        T = cdna_times(x["d"], x["p"], theta_of(x["p"]))
        return (T, None)
    if path == "loss_grad":
        return grad_call(lambda th: cdna_times(x["d"], x["p"], th), x["m"], theta_of(x["p"]))
    if path == "autograd":
        th = theta_of(x["p"]).requires_grad_()
        T = cdna_times(x["d"], x["p"], th)
        fin = torch.isfinite(T)
        torch.where(fin, T, torch.zeros_like(T)).backward(torch.where(fin, x["w"].double(), torch.zeros_like(T)))
        return T.detach(), th.grad.cpu()
    if path == "tiles":
        return None, tile_best(x), None
    if path == "calibrate":
        th, h = adam(lambda t: cdna_times(x["d"], x["p"], t), x["m"], x["p"], x["mask"], case["steps"])
        return None, th, h
    if path == "sets":
        got = [adam(lambda t, k=k: cdna_times(k["d"], k["p"], t), k["m"], k["p"], k["mask"], case["steps"])
               for k in x["sets"]]
        return None, np.stack([g[0] for g in got]), np.stack([g[1] for g in got])
    if path == "totals":
        return app_times(x, theta_of(x["p"]), segvec_of(x["q"]))[0]
    if path == "app_grad":
        return grad_call(lambda th, sv: app_times(x, th, sv)[0], x["m"], theta_of(x["p"]), segvec_of(x["q"]))
    if path == "plan":
        total, unfused = plan_totals(x, case["R"])
        return total, unfused, None
    if path == "multipliers":
        return multipliers(x)
    if path == "bw_predict":
        return bw_times(x["d"], x["p"], theta_of(x["p"])), None
    return grad_call(lambda th: bw_times(x["d"], x["p"], th), x["m"], theta_of(x["p"]))
