"""The work that users of this framework have it do, as cases that can be timed and compared: optimizer steps
through the public entry points (`MonaOptimizer.step`, `mona_step_noalloc`, `AdamWOptimizer.step`).

A case is a dict of plain values:
  path       "mona" (a list of matrices behind one state), "noalloc" (one matrix, caller-kept state arrays) or
             "adamw" (the tensors that are not matrices)
  shapes     "count*m*n, ..." (matrices) or "count*n, ..." (tensors of AdamW)
  w, g       dtype of parameters and gradients: "f32" or "bf16"
  state      dtype of the stored G_{k-1} and A: "f32" or "bf16" (the low-precision state variant)
  accel      how the acceleration term is carried: "two" buffers, "one" buffer, or the caller's "slot"
  precision  0: bf16 products, 1: fp32 products
  steps      Newton-Schulz iterations
"""
import ctypes as C
import math

import torch

from paper_2605_26842_amd import binding as B
from paper_2605_26842_amd import workloads as wl

_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
_ACCEL = {"two": B.MONA_ACCEL_TWO_BUFFER, "one": B.MONA_ACCEL_ONE_BUFFER, "slot": B.MONA_ACCEL_CALLER_SLOT}


def _mona(name, shapes, w="bf16", g="f32", state="f32", accel="two", precision=0, steps=5, path="mona"):
    case = {"name": name, "path": path, "shapes": shapes, "w": w, "g": g, "state": state, "accel": accel,
            "precision": precision, "steps": steps}
    return case


def _adamw(name, shapes, w="bf16", g="f32"):
    return {"name": name, "path": "adamw", "shapes": shapes, "w": w, "g": g}


def listed():
    return [
        # one fp32 matrix: the smallest step, a chain of small dependent launches
        _mona("single_256x512", "1*256*512", w="f32"),
        # one matrix of a caller that cannot allocate (graph capture, serving loops)
        _mona("noalloc_512x1408", "1*512*1408", path="noalloc"),
        # ragged shapes: rows and columns off every tile size, a row, a column, a 3 x 5
        _mona("ragged_mix", "1*100*300, 1*333*130, 1*257*257, 1*3*5, 1*1*64, 1*70*1, 3*192*136", w="f32"),
        # attention and feed-forward matrices of one dense block of hidden size 2048
        _mona("dense_block_h2048", "4*2048*2048, 1*2048*8192, 1*8192*2048"),
        # the same kind of block with sides that are no multiple of a tile (hidden 1000, feed-forward 8/3 of it)
        _mona("dense_block_h1000", "4*1000*1000, 2*1000*2666, 1*2666*1000"),
        # fp32-class products: a block of hidden size 1024, fp32 parameters
        _mona("block_h1024_fp32_products", "4*1024*1024, 1*1024*4096, 1*4096*1024", w="f32", precision=1),
        # many small experts: hidden 768, feed-forward 256
        _mona("moe_1b_experts", "128*768*256, 128*256*768"),
        # 64 experts of hidden 2048, feed-forward 1024
        _mona("moe_bank_e64", "128*2048*1024, 64*1024*2048"),
        # the memory-saving options together: bf16 gradients, one bf16 acceleration buffer
        _mona("moe_6b_experts_lite", "128*1536*1024, 128*1024*1536", g="bf16", state="bf16", accel="one"),
        # the largest: attention and 128 experts of one MoE layer of hidden size 4096
        _mona("moe_layer_h4096_e128", "4*4096*4096, 256*4096*1536, 128*1536*4096"),
        # norm gains and small vectors of a model, fp32
        _adamw("adamw_small_vectors", "49*4096, 1*1000, 1*3", w="f32"),
        # input embedding, output head and norm gains of hidden size 4096, vocabulary 128 k
        _adamw("adamw_embeddings_h4096_v128k", "2*536870912, 49*4096"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A side of a matrix: as often any number at all as a multiple of 64 or 256."""
    v = _log_int(rng, lo, hi)
    unit = rng.choice((1, 1, 64, 256))
    return max(unit, (v + unit // 2) // unit * unit) if v >= unit else v


# The largest listed case is the bound of the drawn ones: elements (memory) and products (time).
_MOST_ELEMENTS, _MOST_FLOPS = 1.2e9, 2.0e13


def draw(rng):
    kind = rng.choice(("one", "block", "bank", "bank", "mix", "noalloc", "adamw"))
    if kind == "adamw":
        total = _log_int(rng, 3, 500_000_000)
        parts = [f"1*{total}", f"{rng.randint(1, 60)}*{_log_int(rng, 1, 8192)}"]
        return dict(_adamw("", ", ".join(parts), w=rng.choice(("f32", "bf16")), g=rng.choice(("f32", "bf16"))))
    w, g = rng.choice(("f32", "bf16", "bf16")), rng.choice(("f32", "f32", "bf16"))
    state = rng.choice(("f32", "f32", "bf16"))
    accel = rng.choice(("two", "two", "one", "slot"))
    if kind == "noalloc":
        p = _side(rng, 16, 512)
        q = min(_side(rng, p, 4 * p), 1408)
        m, n = (p, q) if rng.random() < 0.5 else (q, p)
        return dict(_mona("", f"1*{m}*{n}", w=w, g=g, state=state, path="noalloc"))
    precision = 1 if rng.random() < 0.15 else 0
    specs = []
    for _ in range({"one": 1, "block": 3, "bank": rng.randint(1, 3), "mix": rng.randint(3, 8)}[kind]):
        p = _side(rng, 1 if kind == "mix" else 64, {"one": 4096, "block": 2048, "bank": 1536, "mix": 700}[kind])
        q = _side(rng, p, 4 * p)
        most = max(1, int(min(_MOST_ELEMENTS / 3 / (p * q), _MOST_FLOPS / 3 / (15.0 * p * p * q + 5.0 * p ** 3))))
        if precision == 1:
            most = max(1, most // 20)
        count = {"one": 1, "block": rng.choice((1, 2, 4)), "bank": _log_int(rng, 8, 256), "mix": rng.randint(1, 3)}[kind]
        m, n = (p, q) if rng.random() < 0.5 else (q, p)
        specs.append(f"{min(count, most)}*{m}*{n}")
    return dict(_mona("", ", ".join(specs), w=w, g=g, state=state, accel=accel, precision=precision))


def _specs(case):
    return [tuple(int(v) for v in part.split("*")) for part in case["shapes"].split(",")]


def _bank(spec, std, dtype, gen):
    """`count` tensors of one shape in one allocation, each 16-byte aligned: (the whole as count x elements, the list)."""
    count, shape = spec[0], spec[1:]
    n = math.prod(shape)
    room = torch.zeros((count, (n + 7) // 8 * 8), dtype=dtype, device="cuda")
    whole = room[:, :n]
    whole.normal_(0.0, std, generator=gen)
    return whole, [whole[i].view(shape) for i in range(count)]


def _gradients(specs, dtype, gen, sets=2, rho=wl.GRAD_RHO):
    """`sets` consecutive gradients of every tensor: a stationary AR(1) stream, as consecutive steps of a training run."""
    out, before = [], None
    for _ in range(sets):
        wholes, tensors = [], []
        for j, spec in enumerate(specs):
            whole, each = _bank(spec, wl.GRAD_SIGMA, dtype, gen)
            if before is not None:
                whole.mul_(math.sqrt(1.0 - rho * rho)).add_(before[j], alpha=rho)
            wholes.append(whole)
            tensors += each
        before = wholes
        out.append(tensors)
    return out


def _state_bank(views):
    """Equal-shape pieces of a state, evenly spaced in the arena, as one strided tensor (no copy)."""
    v = views[0]
    if len(views) == 1:
        return v
    step = (views[1].data_ptr() - v.data_ptr()) // v.element_size()
    return torch.as_strided(v, (len(views),) + tuple(v.shape), (step,) + tuple(v.stride()))


def _state_views(specs, kinds, view):
    """The whole arrays the state keeps of every tensor: one output for each shape and kind."""
    out, at = [], 0
    for spec in specs:
        out += [_state_bank([view(i, kind) for i in range(at, at + spec[0])]) for kind in kinds]
        at += spec[0]
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(wl.BASE_SEED + int(seed))
    specs = _specs(case)
    w_dtype, g_dtype = _DTYPE[case["w"]], _DTYPE[case["g"]]
    params, wholes = [], []
    for spec in specs:
        whole, each = _bank(spec, wl.WEIGHT_STD, w_dtype, gen)
        wholes.append(whole)
        params += each
    grads = _gradients(specs, g_dtype, gen)
    s = {"path": case["path"], "grads": grads, "turn": 0, "k": 0}
    if case["path"] == "adamw":
        s["opt"] = opt = B.AdamWOptimizer(params, g_dtype=g_dtype)
        s["hp"] = B.mona_adamw_hparams(1e-3, 0.9, 0.95, 1e-8, 0.1)
        s["out"] = wholes + _state_views(specs, (B.MONA_ADAMW_VIEW_M, B.MONA_ADAMW_VIEW_V), opt.view)
        return s
    hp = wl.HParams(ns_steps=case["steps"])
    state_dtype = _DTYPE[case["state"]]
    if case["path"] == "noalloc":
        w = params[0]
        g_prev, acc = (torch.zeros(w.shape, dtype=state_dtype, device="cuda") for _ in range(2))
        mom = torch.zeros(w.shape, dtype=torch.float32, device="cuda")
        s["hp"] = B.make_hparams(hp)
        s["opts"] = B.mona_options(case["precision"], B._dtype_code(state_dtype), B.MONA_ACCEL_TWO_BUFFER, 0, 0, 0,
                                   (C.c_int32 * 2)())
        s["mats"] = [B.make_matrices([w], g) for g in grads]
        s["arrays"] = (g_prev, acc, mom)
        s["out"] = [w, g_prev, acc, mom]
        return s
    accel = case["accel"]
    s["hp"] = hp
    s["opt"] = opt = B.MonaOptimizer(params, ns_precision=case["precision"], state_dtype=state_dtype, g_dtype=g_dtype,
                                     accel_form=_ACCEL[accel])
    kinds = {"two": (B.MONA_VIEW_G_PREV, B.MONA_VIEW_A, B.MONA_VIEW_M), "one": (B.MONA_VIEW_C, B.MONA_VIEW_M),
             "slot": (B.MONA_VIEW_A, B.MONA_VIEW_M)}[accel]
    s["out"] = wholes + _state_views(specs, kinds, opt.view)
    s["slots"] = None
    if accel == "slot":
        s["slots"] = []
        for count, m, n in specs:
            room = torch.zeros((count, (m * n + 7) // 8 * 8), dtype=state_dtype, device="cuda")
            s["slots"] += [room[i, :m * n].view(m, n) for i in range(count)]
            s["out"].append(room)
    return s


def run(s):
    """One optimizer step with the next gradients; returns the parameters and the state arrays it has updated."""
    turn = s["turn"]
    s["turn"] = turn ^ 1
    if s["path"] == "noalloc":
        g_prev, acc, mom = s["arrays"]
        B.mona_step_noalloc(s["mats"][turn], s["opts"], g_prev.data_ptr(), acc.data_ptr(), mom.data_ptr(), s["hp"],
                            s["k"], torch.cuda.current_stream().cuda_stream)
        s["k"] += 1
    elif s["path"] == "adamw":
        s["opt"].step(s["grads"][turn], s["hp"])
    else:
        s["opt"].step(s["grads"][turn], s["hp"], slots=s["slots"])
    return s["out"]


def _f32(v):
    """A hyper-parameter as the C structures carry it."""
    return torch.tensor(v, dtype=torch.float32).item()


def _orthogonalise(mom, steps, hp):
    """`steps` Newton-Schulz iterations on a batch of matrices in 64 bits."""
    a, b, c = _f32(hp.ns_a), _f32(hp.ns_b), _f32(hp.ns_c)
    x = mom / mom.flatten(1).norm(dim=1)[:, None, None]
    tall = x.shape[1] > x.shape[2]
    if tall:
        x = x.transpose(1, 2).contiguous()
    for _ in range(steps):
        s = torch.matmul(x, x.transpose(1, 2).contiguous())
        x = a * x + torch.matmul(b * s + c * torch.matmul(s, s), x)
    return x.transpose(1, 2).contiguous() if tall else x


def exact(case, seed):
    """What the first pass on these inputs gives, in 64 bits (all state arrays start from zero)."""
    gen = torch.Generator(device="cuda").manual_seed(wl.BASE_SEED + int(seed))
    specs = _specs(case)
    params = [_bank(spec, wl.WEIGHT_STD, _DTYPE[case["w"]], gen)[0] for spec in specs]
    grads = _gradients(specs, _DTYPE[case["g"]], gen, sets=1)[0]
    out, state, slots, at = [], [], [], 0
    for spec, whole in zip(specs, params):
        count, shape = spec[0], spec[1:]
        g = torch.stack([t.double() for t in grads[at:at + count]])
        at += count
        w = whole.double().reshape((count,) + shape)
        if case["path"] == "adamw":
            lr, b1, b2, eps, wd = (_f32(v) for v in (1e-3, 0.9, 0.95, 1e-8, 0.1))
            # first step: the bias corrections make the corrected moments g and g^2
            out.append(w * (1.0 - lr * wd) - lr * g / (g.abs() + eps))
            state += [(1.0 - b1) * g, (1.0 - b2) * g * g]
            continue
        hp = wl.HParams(ns_steps=case["steps"])
        lr, beta = _f32(hp.lr), _f32(hp.beta_a)
        a = (1.0 - beta) * g
        m = g + _f32(hp.alpha) * a
        keep, scale = 1.0 - lr * _f32(hp.weight_decay), lr * _f32(hp.gamma_coeff) * math.sqrt(max(shape))
        each = max(1, 2 ** 26 // math.prod(shape))
        for i in range(0, count, each):
            w[i:i + each].mul_(keep).sub_(_orthogonalise(m[i:i + each], case["steps"], hp), alpha=scale)
        out.append(w)
        if case["accel"] == "one":
            state += [beta * a - (1.0 - beta) * g, m]
        elif case["accel"] == "slot":
            state += [a, m]
            room = torch.zeros((count, (math.prod(shape) + 7) // 8 * 8), dtype=torch.float64, device="cuda")
            room[:, :math.prod(shape)] = g.flatten(1)
            slots.append(room)
        else:
            state += [g, a, m]
    # one output for each output of run(): whole tensors, then the state arrays
    return out + state + slots


def work(case):
    size = {"f32": 4, "bf16": 2}
    specs = _specs(case)
    elements = float(sum(math.prod(spec) for spec in specs))
    if case["path"] == "adamw":
        # g read; w, m and v read and written
        return {"bytes": elements * (size[case["g"]] + 2 * size[case["w"]] + 16), "flops": 15.0 * elements}
    # g read; w, M and the acceleration's arrays read and written
    arrays = 1 if case["accel"] == "one" else 2
    nbytes = elements * (size[case["g"]] + 2 * size[case["w"]] + 2 * arrays * size[case["state"]] + 8)
    flops = 0.0
    for count, m, n in specs:
        p, q, t = float(min(m, n)), float(max(m, n)), case["steps"]
        # symmetric products on one triangle; iterations one by one, or (long sides well above the short one)
        # the first three and then pairs of them taken on the p x p side
        one_by_one = t * (3 * p * p * q + p ** 3)
        chunks = ([3] if t >= 3 else []) + [2] * ((t - 3 if t >= 3 else t) // 2)
        left = t - sum(chunks)
        taken = sum(3 * p * p * q + (4 * c - 3) * p ** 3 for c in chunks) + left * (3 * p * p * q + p ** 3)
        flops += count * min(one_by_one, taken)
    return {"bytes": nbytes, "flops": flops + 10.0 * elements}


def tolerance(case):
    if case["path"] == "adamw":
        # fp32 moments and parameters; a bf16 parameter may round to the neighbouring value
        return {"rel": 1e-5} if case["w"] == "f32" else {"rel": 1e-3}
    if case["precision"] == 1:
        # fp32 products: the orthogonalised matrix is right to about 3e-6, a fifth of which reaches W
        return {"rel": 1e-5} if case["w"] == "f32" else {"rel": 1e-3}
    # bf16 products: one layout of the iterations against another, or against fp32 products, moves W by 2e-3 to
    # 4e-3 of its norm in one step and by 3e-3 to 7e-3 in three
    return {"rel": 1e-2}
