"""The calls whose speed this library is judged by: what a program that does
arithmetic on batches of big integers asks of it, from one small batch to the
full ragged workloads, each through the public Python entry points.

A case is a dict of plain values: ``op`` names the entry point, ``batch`` the
instances, ``na`` / ``nb`` the u32 limbs of the operands (dividend and divisor
for a division; ``lo`` / ``hi`` bounds of the dividend or operand limbs of a
ragged batch), ``data`` the limb distribution (``uniform``, or ``mixed``: half
the rows carry-adversarial, runs of 0xFFFFFFFF with isolated random limbs) and
``limb`` the width of the tensors' limbs (32, or 64 for int64 tensors).
"""
import math

import numpy as np
import torch

import paper_2607_28897_amd as bi


def listed():
    return [
        # 64 pairs of 2^15 bits: the smallest workload, launch latency
        dict(name="add_64x1024", op="add", batch=64, na=1024, nb=1024, data="uniform", limb=32),
        # a large odd-sized batch through HBM: no 16-byte alignment between rows
        dict(name="sub_4096x8191", op="sub", batch=4096, na=8191, nb=8191, data="mixed", limb=32),
        # the same 64 pairs multiplied: fewer instances than compute units
        dict(name="mul_64x1024", op="mul", batch=64, na=1024, nb=1024, data="uniform", limb=32),
        # many short operands (2^13 bits), the small rows of the paper's tables
        dict(name="mul_16384x256", op="mul", batch=16384, na=256, nb=256, data="uniform", limb=32),
        # 1024 pairs of 2^17 bits, half of them carry-adversarial
        dict(name="mul_1024x4096", op="mul", batch=1024, na=4096, nb=4096, data="mixed", limb=32),
        # 256 pairs of 2^19 bits, the benchmark's workload
        dict(name="mul_256x16384", op="mul", batch=256, na=16384, nb=16384, data="uniform", limb=32),
        # a few large products alone: one caller waiting for its result
        dict(name="mul_3x16384", op="mul", batch=3, na=16384, nb=16384, data="uniform", limb=32),
        # operands of unequal and odd sizes
        dict(name="mul_300x5003x2777", op="mul", batch=300, na=5003, nb=2777, data="uniform", limb=32),
        # the paper's fixed-precision product (mod B^n) on 64-bit limb tensors
        dict(name="mullo_512x8192_u64", op="mullo", batch=512, na=8192, nb=8192, data="uniform", limb=64),
        # 4096 products of 2^15..2^19 bits, each pair its own size, planned once
        dict(name="mul_ragged_4096", op="mul_ragged", batch=4096, lo=1024, hi=16384, data="uniform", limb=32),
        # 4096 divisions of 2^16-bit dividends by 2^15-bit divisors
        dict(name="divmod_4096x2048", op="divmod", batch=4096, na=2048, nb=1024, data="uniform", limb=32),
        # 512 divisions of 2^16..2^18-bit dividends, divisors half as long
        dict(name="div_ragged_512", op="div_ragged", batch=512, lo=2048, hi=8192, data="uniform", limb=32),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Sizes log-uniform over the ranges the listed cases span, odd ones
    included; batches such that no case costs more than the listed ones."""
    op = rng.choice(["add", "sub", "mul", "mul", "mul", "mullo", "mul_ragged", "divmod", "div_ragged"])
    data = rng.choice(["uniform", "mixed"])
    limb = rng.choice([32, 32, 64])
    if op in ("add", "sub"):
        n = _log_int(rng, 256, 16384)
        batch = _log_int(rng, 64, max(64, min(65536, (1 << 25) // n)))
        nb = n
    elif op == "mul_ragged":
        lo = _log_int(rng, 512, 4096)
        return dict(op=op, batch=_log_int(rng, 64, 2048), lo=lo, hi=_log_int(rng, 2 * lo, 16384), data=data, limb=32)
    elif op == "div_ragged":
        lo = _log_int(rng, 512, 4096)
        return dict(op=op, batch=_log_int(rng, 32, 512), lo=lo, hi=_log_int(rng, lo + 64, 8192), data=data, limb=32)
    elif op == "divmod":
        n = _log_int(rng, 256, 8192)
        batch = _log_int(rng, 16, max(16, min(16384, (1 << 22) // n)))
        nb = max(2, int(n * rng.choice([0.5, 0.5, 0.3, 0.75])))
    else:
        n = _log_int(rng, 256, 16384)
        batch = _log_int(rng, 1, max(1, min(16384, (1 << 22) // n)))
        nb = n if op == "mullo" or rng.random() < 0.6 else _log_int(rng, max(64, n // 4), n)
    if limb == 64:
        n, nb = n + n % 2, nb + nb % 2
    return dict(op=op, batch=batch, na=n, nb=nb, data=data, limb=limb)


def _limbs(case, rows, n, g):
    """[rows, n] int32 limbs on the GPU; ``mixed``: the second half of the
    rows is all ones but for isolated random limbs (one in 2048 on average)."""
    x = torch.randint(-2**31, 2**31, (rows, n), dtype=torch.int32, device="cuda", generator=g)
    if case["data"] == "mixed" and rows > 1:
        h = rows // 2
        keep = torch.rand((rows - h, n), device="cuda", generator=g) < 1.0 / 2048
        x[h:] = torch.where(keep, x[h:], torch.full_like(x[h:], -1))
    return x


def _flat(case, lens, g):
    """The flat limbs of a ragged batch and their offsets."""
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    flat = _limbs(dict(data="uniform"), 1, int(off[-1]), g).view(-1)
    if case["data"] == "mixed":
        h = int(off[len(lens) // 2])
        keep = torch.rand(flat.numel() - h, device="cuda", generator=g) < 1.0 / 2048
        flat[h:] = torch.where(keep, flat[h:], torch.full_like(flat[h:], -1))
    return flat, torch.from_numpy(off).cuda(), off


def _lens(case, seed):
    """Log-uniform limb counts of a ragged batch.  They are the case's, the
    same for every seed: a plan is made for sizes, then fed many inputs."""
    r = np.random.default_rng(case["batch"] * 1000003 + case["lo"] * 4099 + case["hi"])
    n = np.ceil(np.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]), case["batch"])))
    return np.clip(n, case["lo"], case["hi"]).astype(np.int64)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def prepare(case, seed):
    g = _generator(seed)
    op = case["op"]
    if op in ("mul_ragged", "div_ragged"):
        la = _lens(case, seed)
        lb = la if op == "mul_ragged" else np.maximum(la // 2, 1)
        a, a_off, _ = _flat(case, la, g)
        b, b_off, hb = _flat(case, lb, g)
        s = dict(op=op, a=a, a_off=a_off, b=b, b_off=b_off)
        if op == "mul_ragged":
            s["plan"] = bi.MulPlan(la, lb)
            off = np.zeros(len(la) + 1, np.int64)
            np.cumsum(la + lb, out=off[1:])
            s["out_off"] = torch.from_numpy(off).cuda()
            s["out"] = torch.empty(int(off[-1]), dtype=torch.int32, device="cuda")
        else:
            tops = torch.from_numpy(hb[1:] - 1).cuda()   # divisors with a nonzero top limb
            b[tops] = b[tops] | 1
            s["plan"] = bi.DivPlan(la, lb)
        return s
    a = _limbs(case, case["batch"], case["na"], g)
    b = _limbs(case, case["batch"], case["nb"], g)
    if op == "divmod":
        b[:, -1] |= 1
    if case["limb"] == 64:
        a, b = a.view(torch.int64), b.view(torch.int64)
    return dict(op=op, a=a, b=b)


def run(s):
    op = s["op"]
    if op == "add":
        return bi.add(s["a"], s["b"])
    if op == "sub":
        return bi.sub(s["a"], s["b"])
    if op == "mul":
        return bi.mul(s["a"], s["b"])
    if op == "mullo":
        return bi.mullo(s["a"], s["b"])
    if op == "divmod":
        return bi.divmod(s["a"], s["b"])
    if op == "mul_ragged":
        return s["plan"](s["a"], s["a_off"], s["b"], s["b_off"], out=s["out"], out_off=s["out_off"])[0]
    return s["plan"](s["a"], s["a_off"], s["b"], s["b_off"])


def _product_ops(na, nb):
    """Operations of one product by transforms: three of na + nb points."""
    n = na + nb
    return 6.0 * n * math.log2(max(n, 2))


def work(case):
    op = case["op"]
    if op in ("mul_ragged", "div_ragged"):
        la = _lens(case, 0).astype(np.float64)
        lb = la if op == "mul_ragged" else np.maximum(la // 2, 1)
    else:
        la = np.full(case["batch"], float(case["na"]))
        lb = np.full(case["batch"], float(case["nb"]))
    ta, tb = float(la.sum()), float(lb.sum())
    if op in ("add", "sub"):
        return {"bytes": 4.0 * 3 * ta + 4.0 * len(la), "flops": 2.0 * ta}
    if op in ("mul", "mul_ragged"):
        return {"bytes": 8.0 * (ta + tb), "flops": float(sum(_product_ops(x, y) for x, y in zip(la, lb)))}
    if op == "mullo":
        return {"bytes": 12.0 * ta, "flops": float(sum(_product_ops(x, y) for x, y in zip(la, lb)))}
    # a division reads u and v, writes q (as long as u) and r (as long as v) and
    # cannot do with less than the quotient's and the remainder's product
    return {"bytes": 8.0 * (ta + tb) + 4.0 * len(la),
            "flops": float(sum(2 * _product_ops(x - y + 1, y) for x, y in zip(la, lb)))}


def _ints(rows):
    return [int.from_bytes(r.tobytes(), "little") for r in rows]


def _back(xs, n):
    """Integers as rows of n u32 limbs (mod 2^(32n)), int32."""
    m = (1 << (32 * n)) - 1
    buf = b"".join((x & m).to_bytes(4 * n, "little") for x in xs)
    return torch.from_numpy(np.frombuffer(buf, np.int32).reshape(len(xs), n).copy())


def exact(case, seed):
    """The same outputs by Python's integers (None where that takes long)."""
    op, batch = case["op"], case["batch"]
    if op in ("mul_ragged", "div_ragged"):
        return None
    na, nb = case["na"], case["nb"]
    cost = batch * (na * nb if op == "divmod" else (na + nb) * 8 if op in ("add", "sub") else (na * nb) ** 0.8)
    if cost > 4e8:
        return None
    s = prepare(case, seed)
    a = s["a"].view(torch.int32).cpu().numpy().view(np.uint32)
    b = s["b"].view(torch.int32).cpu().numpy().view(np.uint32)
    xs, ys = _ints(a), _ints(b)
    wide = torch.int64 if case["limb"] == 64 else torch.int32
    if op in ("add", "sub"):
        zs = [x + y if op == "add" else x - y for x, y in zip(xs, ys)]
        flag = [z >> (32 * na) & 1 for z in zs]
        return _back(zs, na).view(wide), torch.tensor(flag, dtype=torch.int32)
    if op in ("mul", "mullo"):
        return _back([x * y for x, y in zip(xs, ys)], na + nb if op == "mul" else na).view(wide)
    qr = [divmod(x, y) for x, y in zip(xs, ys)]
    return (_back([q for q, _ in qr], na).view(wide), _back([r for _, r in qr], nb).view(wide),
            torch.zeros(batch, dtype=torch.int32))
