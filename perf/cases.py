"""The calls whose speed counts: one pass each through the public entry points
of paper_2103_00571_amd.ops, on synthetic SU(3) links held on the GPU.

A case is a dict:

    op      the call (below)
    form    storage form of the lattice: f64, f32, bf16, r12_f32, r12c_f32, r12_f64
    sites   lattice sites
    pitch   SoA calls: "dense" (plane pitch = sites) or "padded" (ops.soa_pitch)
    wrt     autograd calls: the inputs that need a gradient, "ab", "a" or "b"
    out     products: True where the program keeps its output buffer and passes
            it in, as a loop over passes does; False where the call allocates it

and op is one of

    nn, na, an       the site-major products a b, a b^H, a^H b
    mat_vec          links times the site's colour vector
    soa              the product on structure-of-arrays planes
    to_soa, to_aos   the layout transforms
    pack, unpack     FP64 links to a storage form, and back
    bwd              the adjoint, its outputs and workspace kept by the program
    train            SU3MultNN forward and backward through torch.autograd
"""

import torch

from paper_2103_00571_amd import ops

FORMS = {"f64": ops.SU3_F64, "f32": ops.SU3_F32, "bf16": ops.SU3_BF16, "r12_f32": ops.SU3_R12_F32,
         "r12c_f32": ops.SU3_R12C_F32, "r12_f64": ops.SU3_R12_F64}
# bytes per site of the lattice in each form, and of the product
A_BYTES = {"f64": 576, "f32": 288, "bf16": 144, "r12_f32": 192, "r12c_f32": 192, "r12_f64": 384}
C_BYTES = {"f64": 576, "f32": 288, "bf16": 144, "r12_f32": 288, "r12c_f32": 192, "r12_f64": 576}


def listed():
    return [
        # the smallest lattice that is timed here (L=8): one call's latency
        {"name": "nn_f64_L8", "op": "nn", "form": "f64", "sites": 8 ** 4, "out": False},
        # the headline: FP64 on L=48, output buffer kept over the passes
        {"name": "nn_f64_L48", "op": "nn", "form": "f64", "sites": 48 ** 4, "out": True},
        # the paper's lattice in its single precision
        {"name": "nn_f32_L32", "op": "nn", "form": "f32", "sites": 32 ** 4, "out": True},
        # one GPU's share of L=48 over eight, in the smallest storage form
        {"name": "nn_bf16_shard8", "op": "nn", "form": "bf16", "sites": 48 ** 4 // 8, "out": True},
        # compressed links in, full product out, a mid-sized lattice
        {"name": "nn_r12_f32_L24", "op": "nn", "form": "r12_f32", "sites": 24 ** 4, "out": True},
        # data remapped to planes, as the paper suggests, on its larger lattice
        {"name": "soa_f64_L32", "op": "soa", "form": "f64", "sites": 32 ** 4, "pitch": "dense", "out": True},
        # the same on a site count that no power of two divides
        {"name": "soa_f32_odd", "op": "soa", "form": "f32", "sites": 31 ** 4, "pitch": "dense", "out": True},
        # the remapping itself
        {"name": "to_soa_f64_L40", "op": "to_soa", "form": "f64", "sites": 40 ** 4, "pitch": "dense"},
        # stored links widened for a program that computes in FP64
        {"name": "unpack_bf16_L32", "op": "unpack", "form": "bf16", "sites": 32 ** 4},
        # both gradients with buffers kept by the program
        {"name": "bwd_f64_L32", "op": "bwd", "form": "f64", "sites": 32 ** 4},
        # a training step in single precision on the paper's smaller lattice
        {"name": "train_f32_L16", "op": "train", "form": "f32", "sites": 16 ** 4, "wrt": "ab"},
        # the four shared matrices fitted to a lattice that is data
        {"name": "train_f64_L24_b", "op": "train", "form": "f64", "sites": 24 ** 4, "wrt": "b"},
    ]


# most sites a drawn case of each op has (its bytes then stay below those of
# the FP64 product on L=48)
MOST_SITES = {"nn": 48 ** 4, "na": 48 ** 4, "an": 48 ** 4, "mat_vec": 48 ** 4, "soa": 46 ** 4, "to_soa": 42 ** 4,
              "to_aos": 44 ** 4, "pack": 46 ** 4, "unpack": 46 ** 4, "bwd": 40 ** 4, "train": 36 ** 4}


def draw(rng):
    op = rng.choice(["nn", "nn", "nn", "na", "an", "mat_vec", "soa", "soa", "to_soa", "to_aos", "pack", "unpack",
                     "bwd", "train", "train"])
    most = MOST_SITES[op]
    if rng.random() < 0.4:
        # L^3 x T lattices, L and T even, L <= T <= 2 L
        sites = rng.choice([L ** 3 * T for L in range(4, 49, 2) for T in range(L, 2 * L + 1, 2) if L ** 3 * T <= most])
    else:
        # any count, spread over its logarithm, odd ones included
        sites = min(most, int(256 * (most / 256.0) ** rng.random()) | (rng.random() < 0.5))
    case = {"op": op, "sites": sites}
    if op == "nn":
        case["form"] = rng.choice(list(FORMS))
    elif op in ("pack", "unpack"):
        case["form"] = rng.choice(["f32", "bf16", "r12_f32", "r12_f64"])
    else:
        case["form"] = rng.choice(["f64", "f32"])
    if op in ("soa", "to_soa", "to_aos"):
        case["pitch"] = rng.choice(["dense", "padded"])
    if op == "train":
        case["wrt"] = rng.choice(["ab", "ab", "a", "b"])
    if op in ("nn", "na", "an", "mat_vec", "soa"):
        case["out"] = rng.random() < 0.5
    return case


# ---- inputs ---------------------------------------------------------------

def _haar(n, gen):
    """n Haar-random SU(3) matrices, complex128 (n, 3, 3) on the GPU."""
    g = torch.randn((n, 2, 3), dtype=torch.complex128, device="cuda", generator=gen)
    r0 = g[:, 0]
    r0 = r0 / torch.linalg.vector_norm(r0, dim=-1, keepdim=True)
    r1 = g[:, 1]
    for _ in range(2):
        r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj().resolve_conj()], dim=1)


def _links(sites, gen):
    return _haar(4 * sites, gen).view(sites, 4, 3, 3)


def _store(a64, form):
    """FP64 site-major links in a storage form."""
    if form == "f32":
        return a64.to(torch.complex64)
    if form == "bf16":
        return torch.view_as_real(a64).to(torch.float32).to(torch.bfloat16)
    if form in ("r12_f32", "r12c_f32"):
        return a64[:, :, :2].to(torch.complex64).contiguous()
    if form == "r12_f64":
        return a64[:, :, :2].contiguous()
    return a64


def _real_form(form):
    return torch.complex128 if form in ("f64", "r12_f64") else torch.complex64


def _planes(x, pitch):
    """Site-major links as (4, 3, 3, pitch) planes; the padding is zero."""
    out = torch.zeros((4, 3, 3, pitch), dtype=x.dtype, device=x.device)
    out[..., :x.shape[0]] = x.permute(1, 2, 3, 0)
    return out


def _pitch(case):
    n = case["sites"]
    return n if case["pitch"] == "dense" else ops.soa_pitch(n, FORMS[case["form"]])


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, form, op = case["sites"], case["form"], case["op"]
    s = {"a64": _links(n, gen)}
    s["b"] = _haar(4, gen).to(_real_form(form))
    if op == "mat_vec":
        s["v"] = torch.randn((n, 3), dtype=torch.complex128, device="cuda", generator=gen).to(_real_form(form))
    if op in ("bwd", "train"):
        s["dc"] = torch.randn((n, 4, 3, 3), dtype=torch.complex128, device="cuda", generator=gen).to(_real_form(form))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    a64 = s.pop("a64")
    n, form, op = case["sites"], case["form"], case["op"]
    s["case"], s["sites"], s["form"] = case, n, FORMS[form]
    if op == "pack":
        s["a"] = a64
    elif op in ("soa", "to_aos"):
        s["a"] = _planes(_store(a64, form), _pitch(case))
    else:
        s["a"] = _store(a64, form)
    if op == "to_soa":
        s["pitch"] = _pitch(case)
    if op == "train":
        s["wrt"] = []
        for name in case["wrt"]:
            s[name].requires_grad_(True)
            s["wrt"].append(s[name])
    if op == "bwd":
        s["da"] = torch.empty_like(s["a"])
        s["db"] = torch.empty((4, 3, 3), dtype=torch.complex128, device="cuda")
        s["ws"] = ops.mult_nn_bwd_workspace(n, s["form"], s["a"].device)
    s["out"] = None
    if case.get("out"):
        if op == "mat_vec":
            s["out"] = torch.zeros((n, 4, 3), dtype=s["a"].dtype, device="cuda")
        elif op == "nn" and form in ("r12_f32", "r12_f64"):
            s["out"] = torch.zeros((n, 4, 3, 3), dtype=s["a"].dtype, device="cuda")
        else:
            s["out"] = torch.zeros_like(s["a"])
    return s


def run(s):
    op = s["case"]["op"]
    if op == "nn":
        return ops.mult_nn(s["a"], s["b"], out=s["out"], form=s["form"])
    if op == "na":
        return ops.mult_na(s["a"], s["b"], out=s["out"])
    if op == "an":
        return ops.mult_an(s["a"], s["b"], out=s["out"])
    if op == "mat_vec":
        return ops.mat_vec(s["a"], s["v"], out=s["out"])
    if op == "soa":
        # the lattice part of the planes; padding belongs to nobody
        return ops.mult_nn_soa(s["a"], s["b"], out=s["out"], sites=s["sites"])[..., :s["sites"]]
    if op == "to_soa":
        return ops.aos_to_soa(s["a"], s["pitch"])[..., :s["sites"]]
    if op == "to_aos":
        return ops.soa_to_aos(s["a"], s["sites"])
    if op == "pack":
        return ops.pack(s["a"], s["form"])
    if op == "unpack":
        return ops.unpack(s["a"], s["form"])
    if op == "bwd":
        da, db = ops.mult_nn_bwd(s["a"], s["b"], s["dc"], da=s["da"], db=s["db"], ws=s["ws"])
        return {"da": da, "db": db}
    c = ops.SU3MultNN.apply(s["a"], s["b"])
    grads = torch.autograd.grad(c, s["wrt"], s["dc"])
    return {"c": c, **{"d" + name: g for name, g in zip(s["case"]["wrt"], grads)}}


def work(case):
    n, form, op = case["sites"], case["form"], case["op"]
    a, c = A_BYTES[form], C_BYTES[form]
    b = 576 if form in ("f64", "r12_f64") else 288
    if op in ("nn", "na", "an", "soa"):
        return {"bytes": n * (a + c) + b, "flops": 864 * n}
    if op == "mat_vec":
        return {"bytes": n * (a + a // 12 + a // 3), "flops": 288 * n}
    if op in ("to_soa", "to_aos"):
        return {"bytes": n * 2 * a, "flops": 0}
    if op in ("pack", "unpack"):
        return {"bytes": n * (576 + a), "flops": 0}
    if op == "bwd":
        return {"bytes": n * 3 * a + b + 576, "flops": 2 * 864 * n}
    # forward: a in, c out; backward: dc in, and a in (for db), da out (for da)
    grads = case["wrt"]
    return {"bytes": n * a * (3 + len(grads)) + 3 * b, "flops": 864 * n * (1 + len(grads))}


# ---- the same in 64 bits, by torch alone -----------------------------------

def _wide(x, form):
    """A stored lattice (or b, v, dc) in complex128, site-major; compressed links
    get their third row."""
    if x.dtype == torch.bfloat16:
        return torch.view_as_complex(x.to(torch.float64))
    x = x.to(torch.complex128)
    if form in ("r12_f32", "r12_f64") and x.dim() == 4 and x.shape[2] == 2:
        x = torch.cat([x, torch.linalg.cross(x[:, :, 0], x[:, :, 1]).conj().resolve_conj()[:, :, None]], dim=2)
    return x


def _mm(x, y):
    """Products of 3x3 (or 2x3) complex matrices over the leading dimensions."""
    z = x[..., :, 0, None] * y[..., 0, None, :]
    for m in (1, 2):
        z = z + x[..., :, m, None] * y[..., m, None, :]
    return z


def _h(x):
    return x.transpose(-1, -2).conj().resolve_conj()


def exact(case, seed):
    s = _inputs(case, seed)
    n, form, op = case["sites"], case["form"], case["op"]
    if op == "pack":
        a64 = s["a64"]
        if form == "bf16":
            return torch.view_as_real(a64)
        return a64[:, :, :2].contiguous() if form in ("r12_f32", "r12_f64") else a64
    stored = _store(s["a64"], form)
    a, b = _wide(stored, form), s["b"].to(torch.complex128)
    if op == "unpack":
        return a
    if op == "to_aos":
        return a
    if op == "to_soa":
        return a.permute(1, 2, 3, 0).contiguous()
    if op == "nn":
        c = _mm(a, b)
        return torch.view_as_real(c) if form == "bf16" else c
    if op == "na":
        return _mm(a, _h(b))
    if op == "an":
        return _mm(_h(a), b)
    if op == "soa":
        return _mm(a, b).permute(1, 2, 3, 0).contiguous()
    if op == "mat_vec":
        v = s["v"].to(torch.complex128)
        return _mm(a, v[:, None, :, None])[..., 0]
    dc = s["dc"].to(torch.complex128)
    grads = {"da": _mm(dc, _h(b)), "db": _mm(_h(a), dc).sum(0)}
    if op == "bwd":
        return grads
    return {"c": _mm(a, b), **{"d" + name: grads["d" + name] for name in case["wrt"]}}
