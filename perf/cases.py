"""Timing cases of the protected product: what a program does with `gecc.Context`, over the range it is used on.

A case is one configuration of the context and one of four ways to use it:

  clean    gecc_protected_gemm on intact operands: encode, multiply, verify and the decoder that finds
           nothing to do.  What nearly every step of a training run is.
  correct  encode, errors strike, multiply, verify, correct: the campaign and scenario trials, two wrong
           symbols per product (one of A or B overwritten after encoding, or of C inside the product).
  blocked  `clean` with the blocked grid code (one codeword per block of C).
  stored   a product that has been lying in memory: re-verified from memory (gecc_verify(fused=0)) and
           corrected, two symbols of it having been overwritten.

Layouts: NN (both operands row-major), NT (B stored m x k), TN (A stored k x n), TT.
"""
import ctypes
import math

import torch

from paper_2508_04355_amd import gecc

_U = 3.0 ** -0.5                       # standard deviation of U(-1, 1)
_REPORT_INTS = ctypes.sizeof(gecc.Report) // 4


def _case(name, use, dtype, n, k, m, layout="NN", batch=1, law="layer", block_n=0, block_m=0):
    c = {"use": use, "dtype": dtype, "n": n, "k": k, "m": m, "layout": layout, "batch": batch, "law": law,
         "block_n": block_n, "block_m": block_m}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest product: nothing but launches and latencies
        _case("clean-128-f32", "clean", "f32", 128, 128, 128, law="normal"),
        # a single fp32 product of ordinary size
        _case("clean-1024-f32", "clean", "f32", 1024, 1024, 1024, law="uniform"),
        # odd sizes in fp32: rows that are not 16-byte aligned, tiles that hang over every edge
        _case("clean-ragged-f32", "clean", "f32", 1000, 1031, 777, law="uniform"),
        # 256 small fp32 problems, two errors in each: the code at its limit everywhere at once
        _case("correct-batch-f32", "correct", "f32", 512, 512, 512, batch=256, law="uniform"),
        # odd sizes in bf16: one operand with aligned rows, one without
        _case("clean-ragged-bf16", "clean", "bf16", 1500, 1000, 1100, law="small"),
        # the square bf16 product of the error campaigns, without and with errors
        _case("clean-4096-bf16", "clean", "bf16", 4096, 4096, 4096, law="small"),
        _case("correct-4096-bf16", "correct", "bf16", 4096, 4096, 4096, law="small"),
        # the three products of a transformer layer in training: forward, gradient of the input,
        # gradient of the weight (the largest cases)
        _case("clean-forward-bf16", "clean", "bf16", 16384, 4096, 14336, law="layer"),
        _case("clean-dgrad-bf16", "clean", "bf16", 16384, 14336, 4096, layout="NT", law="layer"),
        _case("clean-wgrad-bf16", "clean", "bf16", 4096, 16384, 14336, layout="TN", law="normal"),
        # the forward product in 1024 x 1024 codewords: two errors in every block can be put right
        _case("blocked-forward-bf16", "blocked", "bf16", 16384, 4096, 14336, law="layer", block_n=1024, block_m=1024),
        # the forward product's C checked again in memory
        _case("stored-forward-bf16", "stored", "bf16", 16384, 4096, 14336, law="layer"),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, lo, hi, most_flops, step):
    """Three sizes spread over the logarithm of lo..hi, as they come or rounded to a multiple of `step`."""
    while True:
        n, k, m = (_log_size(rng, lo, hi) for _ in range(3))
        if step > 1:
            n, k, m = (max(step, (x + step // 2) // step * step) for x in (n, k, m))
        if 2.0 * n * k * m <= most_flops:
            return n, k, m


def draw(rng):
    kind = rng.choice(["f32", "f32", "batch", "bf16", "bf16", "layer", "layer", "correct", "blocked", "stored"])
    layout = rng.choice(["NN", "NN", "NT", "TN", "TT"])
    step = rng.choice([1, 8, 64, 128])
    if kind == "f32":
        n, k, m = _shape(rng, 48, 2048, 8e9, step)
        return _case(None, "clean", "f32", n, k, m, layout, law=rng.choice(["normal", "uniform"]))
    if kind == "batch":
        n, k, m = _shape(rng, 96, 640, 3e8, step)
        batch = max(2, min(256, int(rng.uniform(0.2, 1.0) * 6.8e10 / (2.0 * n * k * m))))
        return _case(None, rng.choice(["clean", "correct"]), "f32", n, k, m, layout, batch=batch, law="uniform")
    if kind == "bf16":
        n, k, m = _shape(rng, 200, 6144, 2e11, step)
        return _case(None, "clean", "bf16", n, k, m, layout, law="small")
    if kind == "layer":
        # tokens x hidden x intermediate, in one of the three products of a step
        t, h, f = rng.randrange(8, 129) * 128, rng.randrange(8, 33) * 128, rng.randrange(16, 113) * 128
        n, k, m, lay = rng.choice([(t, h, f, "NN"), (t, f, h, "NT"), (h, t, f, "TN")])
        return _case(None, "clean", "bf16", n, k, m, lay, law="normal" if lay == "TN" else "layer")
    if kind == "correct":
        n, k, m = _shape(rng, 512, 6144, 2e11, max(8, step))
        return _case(None, "correct", "bf16", n, k, m, layout, law="small")
    if kind == "blocked":
        bn, bm = rng.choice([512, 1024, 2048]), rng.choice([512, 1024, 2048])
        n, m, k = bn * rng.randrange(2, 9), bm * rng.randrange(2, 8), rng.randrange(16, 65) * 64
        return _case(None, "blocked", "bf16", n, k, m, rng.choice(["NN", "NT", "TN"]), law="layer", block_n=bn, block_m=bm)
    n, m, k = (_log_size(rng, 1024, hi) // step * step for hi in (16384, 14336, 4096))
    return _case(None, "stored", "bf16", n, k, m, law="layer")


# ---- inputs ----------------------------------------------------------------------------------------
# law: (how A is drawn, how B is drawn, standard deviations)
_LAWS = {"normal": (1.0, 1.0), "small": (0.02, 0.02), "layer": (1.0, 0.02), "uniform": (_U, _U)}


def _draw_matrix(gen, batch, rows, cols, law, sigma, dtype):
    x = torch.empty((batch, rows, cols), dtype=torch.float32, device="cuda:0")
    if law == "uniform":
        x.uniform_(-1.0, 1.0, generator=gen)
    else:
        x.normal_(0.0, sigma, generator=gen)
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _operands(case, gen):
    """A and B as stored (batch, rows, columns)."""
    n, k, m, b = case["n"], case["k"], case["m"], case["batch"]
    sa, sb = _LAWS[case["law"]]
    ra, ca = (k, n) if case["layout"][0] == "T" else (n, k)
    rb, cb = (m, k) if case["layout"][1] == "T" else (k, m)
    return (_draw_matrix(gen, b, ra, ca, case["law"], sa, case["dtype"]),
            _draw_matrix(gen, b, rb, cb, case["law"], sb, case["dtype"]))


def _logical(case, A, B):
    """The operands as (batch, n, k) and (batch, k, m), whatever way they are stored."""
    return (A.transpose(1, 2) if case["layout"][0] == "T" else A,
            B.transpose(1, 2) if case["layout"][1] == "T" else B)


def _two_faults(case, gen):
    """Two wrong symbols per item at places uniform over A, B and C (drawn again where both fall into one
    column of A or one row of B, which two parities cannot tell apart); additive, magnitude U[1, 100], either
    sign.  The campaign's law.  Returns [(matrix, item, row, col, offset)], logical coordinates."""
    n, k, m = case["n"], case["k"], case["m"]
    sizes, cols = (n * k, k * m, n * m), (k, m, m)
    u = torch.rand((case["batch"], 8, 6), generator=gen, device="cuda:0", dtype=torch.float64).cpu().tolist()
    out = []
    for b in range(case["batch"]):
        for v in u[b]:
            got = []
            for x in range(2):
                f = int(v[x] * sum(sizes))
                mat = 0 if f < sizes[0] else (1 if f < sizes[0] + sizes[1] else 2)
                f -= (0, sizes[0], sizes[0] + sizes[1])[mat]
                e = (1.0 + 99.0 * v[2 + x]) * (1.0 if v[4 + x] < 0.5 else -1.0)
                got.append((mat, b, f // cols[mat], f % cols[mat], e))
            p, q = got
            if p[0] == q[0] and (p[2:4] == q[2:4] or (p[0] == 0 and p[3] == q[3]) or (p[0] == 1 and p[2] == q[2])):
                continue
            break
        out += got
    return out


def _strike(case, X, matrix, faults):
    """(flat indices, wrong values) of the faults in one operand as stored."""
    t = case["layout"][matrix] == "T"
    rows, cols = X.shape[1], X.shape[2]
    mine = [f for f in faults if f[0] == matrix]
    if not mine:
        return None
    at = torch.tensor([b * rows * cols + (j * cols + i if t else i * cols + j) for (_, b, i, j, _) in mine], device="cuda:0")
    off = torch.tensor([f[4] for f in mine], dtype=torch.float32, device="cuda:0")
    return at, (X.view(-1)[at].float() + off).to(X.dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda:0").manual_seed(int(seed))
    n, k, m = case["n"], case["k"], case["m"]
    A, B = _operands(case, gen)
    sa, sb = _LAWS[case["law"]]
    bn, bm = case["block_n"], case["block_m"]
    tau = gecc.noise_thresholds(bn or n, k, bm or m, sa, sb)
    ctx = gecc.Context(n, k, m, gecc.BF16 if case["dtype"] == "bf16" else gecc.F32, tau, batch=case["batch"],
                       trans_a=int(case["layout"][0] == "T"), trans_b=int(case["layout"][1] == "T"), block=(bn, bm))
    A_par, B_par, C_par = ctx.alloc_parities()
    s = {"use": case["use"], "ctx": ctx, "A": A, "B": B, "C": ctx.alloc_c(), "A_par": A_par, "B_par": B_par,
         "C_par": C_par, "report": ctx.alloc_report()}
    if case["use"] == "correct":
        faults = _two_faults(case, gen)
        s["strike_a"], s["strike_b"] = _strike(case, A, 0, faults), _strike(case, B, 1, faults)
        s["faults"] = gecc.make_faults([f[1:] for f in faults if f[0] == 2])
    if case["use"] == "stored":
        ctx.protected_gemm(A, B, s["C"], A_par, B_par, C_par, s["report"])
        u = torch.rand(4, generator=gen, device="cuda:0", dtype=torch.float64).tolist()
        i, j = sorted((int(u[0] * n), (int(u[0] * n) + 1 + n // 3) % n)), (int(u[1] * m), (int(u[1] * m) + 1 + m // 3) % m)
        at = torch.tensor([i[0] * m + j[0], i[1] * m + j[1]], device="cuda:0")
        off = torch.tensor([1.0 + 99.0 * u[2], -1.0 - 99.0 * u[3]], dtype=torch.float32, device="cuda:0")
        s["strike_c"] = at, s["C"].view(-1)[at] + off
    return s


# ---- one pass --------------------------------------------------------------------------------------
def _decisions(s, flagged):
    """What the reports say in whole numbers (views of the device records, nothing is launched): status and
    number of errors, the located positions, and on request the counts of flagged rows and columns (not where
    an operand is hit: then they depend on products that lie below the threshold)."""
    r = s["report"].view(torch.int32).view(-1, _REPORT_INTS)
    d = {"status": r[:, 0], "n_err": r[:, 3], "positions": r[:, 4:4 + 6 * gecc.MAX_ERR].view(-1, gecc.MAX_ERR, 6)[:, :, :3]}
    if flagged:
        d["flagged"] = r[:, 1:3]
    return d


def run(s):
    ctx, use = s["ctx"], s["use"]
    A, B, C, A_par, B_par, C_par, rep = (s[x] for x in ("A", "B", "C", "A_par", "B_par", "C_par", "report"))
    if use in ("clean", "blocked"):
        ctx.protected_gemm(A, B, C, A_par, B_par, C_par, rep)
        return {"C": C, "A_par": A_par, "B_par": B_par, "C_par": C_par, "report": _decisions(s, True)}
    if use == "stored":
        C.view(-1).index_copy_(0, *s["strike_c"])
        ctx.verify(C, C_par, rep, fused=False)
        ctx.correct(A, A_par, B, B_par, C, C_par, rep)
        return {"C": C, "report": _decisions(s, True)}
    ctx.encode_a(A, A_par)
    ctx.encode_b(B, B_par)
    if s["strike_a"]:
        A.view(-1).index_copy_(0, *s["strike_a"])
    if s["strike_b"]:
        B.view(-1).index_copy_(0, *s["strike_b"])
    ctx.multiply(A, A_par, B, B_par, C, C_par, *s["faults"])
    ctx.verify(C, C_par, rep, fused=True)
    ctx.correct(A, A_par, B, B_par, C, C_par, rep)
    return {"A": A, "B": B, "C": C, "A_par": A_par, "B_par": B_par, "C_par": C_par, "report": _decisions(s, False)}


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    n, k, m, b = case["n"], case["k"], case["m"], case["batch"]
    e = 2 if case["dtype"] == "bf16" else 4
    if case["use"] == "stored":        # every symbol of C read once, into two row sums and two column sums
        return {"bytes": 4.0 * n * m + 16.0 * (n + m), "flops": 8.0 * n * m}
    par = 8.0 * (4 * k + 2 * n + 2 * m + 4)
    # the product, and two weighted sums along each axis of both operands
    return {"bytes": b * (e * (float(n) * k + float(k) * m) + 4.0 * n * m + par),
            "flops": b * (2.0 * n * k * m + 8.0 * (float(n) * k + float(k) * m))}


def tolerance(case):
    """fp32 sums over k terms, in whatever order: measured against 64 bits, C is 1e-7 (k = 136) to 8e-7
    (k = 16384) off, and the stated limit is two to four times what two such results may differ by.  (The
    parities are sums in 64 bits and far closer; in blocked mode the parity blocks of the product go through
    32-bit sums, 1e-9 off.)  A line of C that was repaired after an operand error keeps the rounding noise of
    the wrong terms f that passed through its running sums, about 0.2 |f| 2^-24 sqrt(k): with magnitudes up
    to 100 against operands of 0.02 that is 1e-4 of C's root mean square in that line (up to 1e-3 at its worst
    symbol), 5e-6 of C as a whole where the line is one of 512."""
    if case["use"] == "correct":
        return {"rel": 2e-5, "max": 5e-3}
    r = 2e-6 * max(1.0, math.sqrt(case["k"] / 4096.0))
    return {"rel": r, "max": 40 * r}


# ---- the same in 64 bits -----------------------------------------------------------------------------
def _parities(X, dim):
    """Plain and index-weighted sums of X over `dim` (1 or 2 of 3) -> (batch, 2, rest)."""
    w = torch.arange(1, X.shape[dim] + 1, dtype=torch.float64, device=X.device)
    w = w.view(1, -1, 1) if dim == 1 else w.view(1, 1, -1)
    return torch.stack([X.sum(dim), (X * w).sum(dim)], 1)


def exact(case, seed):
    if 2.0 * case["n"] * case["k"] * case["m"] * case["batch"] > 2.5e12:
        return None
    s = prepare(case, seed)            # (`stored`: only the inputs of it are used)
    A0, B0 = s["A"], s["B"]
    A, B = (x.double().contiguous() for x in _logical(case, A0, B0))
    C = torch.stack([A[i] @ B[i] for i in range(case["batch"])])
    n, m, bn, bm = case["n"], case["m"], case["block_n"] or case["n"], case["block_m"] or case["m"]
    a_par = [_parities(A[:, i:i + bn], 1) for i in range(0, n, bn)]
    b_par = [_parities(B[:, :, j:j + bm], 2) for j in range(0, m, bm)]
    c_par = []
    for i, ap in enumerate(a_par):
        for j, bp in enumerate(b_par):
            bt = bp.transpose(1, 2).contiguous()
            blocks = (torch.matmul(A[:, i * bn:(i + 1) * bn], bt).transpose(1, 2), torch.matmul(ap, B[:, :, j * bm:(j + 1) * bm].contiguous()),
                      torch.matmul(ap, bt))
            c_par.append(torch.cat([x.reshape(case["batch"], -1) for x in blocks], 1))
    if case["use"] == "stored":
        return {"C": C, "report": None}
    out = {"C": C, "A_par": torch.cat(a_par).reshape(-1), "B_par": torch.cat(b_par).reshape(-1),
           "C_par": torch.cat(c_par, 0 if case["block_n"] else 1).reshape(-1), "report": None}
    if case["use"] == "correct":
        out["A"], out["B"] = A0.double(), B0.double()
    return out
