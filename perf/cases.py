"""The work that users of this library have it do, as cases that can be timed and checked.

Three kinds of call, each through the public binding:
  dense   all singular values of a dense matrix (`svdvals`, the library's main call): every storage
          type, square, tall and wide, whole tiles and ragged, the caller's tile size or the library's;
  band    a matrix that is banded to begin with: `svb_gb2bd`, then `svb_bdsvals_dev`, asynchronous, on
          buffers the program keeps (the band is consumed, so the program copies it first);
  bidiag  the singular values of a bidiagonal (`svb_bdsvals_dev`).
"""
import math

import torch

import paper_2508_06339_amd as svb

_TYPES = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def _dense(dtype, m, n, nb, values):
    return {"kind": "dense", "dtype": dtype, "m": m, "n": n, "nb": nb, "values": values}


def listed():
    return [
        # the smallest call in use: a single small f64 matrix, where launches and latency count
        dict(_dense("f64", 256, 256, 32, "gauss"), name="dense_f64_256"),
        # an ordinary small f32 matrix with a decaying spectrum
        dict(_dense("f32", 1024, 1024, 32, "geometric"), name="dense_f32_1024"),
        # ordinary f64 work
        dict(_dense("f64", 4096, 4096, 64, "gauss"), name="dense_f64_4096"),
        # half precision storage
        dict(_dense("f16", 4096, 4096, 64, "uniform"), name="dense_f16_4096"),
        # ordinary f32 work, clustered spectrum
        dict(_dense("f32", 8192, 8192, 64, "clustered"), name="dense_f32_8192"),
        # the largest f64 matrix in use
        dict(_dense("f64", 16384, 16384, 128, "gauss"), name="dense_f64_16384"),
        # the largest f32 matrix in use (4 GiB)
        dict(_dense("f32", 32768, 32768, 128, "gauss"), name="dense_f32_32768"),
        # a ragged rectangular matrix, tile size left to the library: staged copy
        dict(_dense("f32", 5000, 3001, 0, "gauss"), name="dense_f32_5000x3001"),
        # a data matrix: many rows, few columns, f64, ragged
        dict(_dense("f64", 20000, 500, 0, "gauss"), name="dense_f64_20000x500"),
        # a wide bf16 matrix (transposed problem)
        dict(_dense("bf16", 1537, 2500, 0, "gauss"), name="dense_bf16_1537x2500"),
        # a banded matrix, odd order
        {"kind": "band", "dtype": "f32", "n": 6007, "nb": 64, "name": "band_f32_6007_64"},
        # the bidiagonal solver by itself
        {"kind": "bidiag", "dtype": "f64", "n": 6000, "name": "bidiag_f64_6000"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["dense", "band", "bidiag"], [8, 2, 1])[0]
    if kind == "bidiag":
        return {"kind": kind, "dtype": rng.choice(["f32", "f64"]), "n": _log_uniform(rng, 64, 12000)}
    if kind == "band":
        return {"kind": kind, "dtype": rng.choice(["f32", "f64"]), "n": _log_uniform(rng, 64, 12000),
                "nb": rng.choice([8, 32, 64, 128])}
    dtype = rng.choices(["f32", "f64", "f16", "bf16"], [4, 3, 1, 1])[0]
    k = _log_uniform(rng, 64, 12000 if dtype == "f32" else 8000)
    shape = rng.choices(["square", "tall", "wide"], [5, 3, 2])[0]
    nb = 0 if rng.random() < 0.6 else rng.choice([32, 64, 128])
    m = n = k
    if shape == "square":
        if rng.random() < 0.5:      # whole tiles: worked on in place
            m = n = max(128, k // 128 * 128)
    else:
        long = min(int(k * math.exp(rng.uniform(0.0, math.log(40.0)))) + 1, 40000, max(k, 100_000_000 // k))
        m, n = (long, k) if shape == "tall" else (k, long)
    values = rng.choice(["gauss", "gauss", "geometric", "uniform", "clustered"]) if min(m, n) >= 128 else "gauss"
    return _dense(dtype, m, n, nb, values)


def _spectrum(values, k, gen):
    if values == "geometric":       # 1 down to 1e-3
        return 1e-3 ** (torch.arange(k, dtype=torch.float64, device="cuda") / max(k - 1, 1))
    u = torch.rand(k, dtype=torch.float64, device="cuda", generator=gen)
    if values == "uniform":         # uniform in [1e-2, 1]
        return 1e-2 + 0.99 * u
    centres = 10.0 ** (-0.5 * (torch.arange(k, device="cuda") * 8 // k).double())   # 8 clusters, relative spread 1e-4
    return centres * (1.0 + 1e-4 * (2.0 * u - 1.0))


def _rotate_rows(a, gen):
    """Random orthogonal transformation of the rows: block reflectors with permutations between them."""
    r = a.shape[0]
    for _ in range(2):
        x = torch.linalg.qr(torch.randn(r, max(1, min(r // 2, 256)), dtype=a.dtype, device="cuda", generator=gen))[0]
        a = a - 2.0 * (x @ (x.T.contiguous() @ a))
        a = a[torch.randperm(r, device="cuda", generator=gen)]
    return a


def _matrix(case, seed):
    """The matrix, column-major: a contiguous n x m tensor whose row j is column j."""
    m, n = case["m"], case["n"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    wide = torch.float64 if case["dtype"] == "f64" else torch.float32
    if case["values"] == "gauss":
        a = torch.randn(n, m, dtype=wide, device="cuda", generator=gen).mul_(1.0 / math.sqrt(max(m, n)))
    else:
        k = min(m, n)
        a = torch.zeros(n, m, dtype=wide, device="cuda")
        a.diagonal().copy_(_spectrum(case["values"], k, gen))
        a = _rotate_rows(_rotate_rows(a, gen).T.contiguous(), gen).T.contiguous()
    return a.to(_TYPES[case["dtype"]]).contiguous()


def _band(case, seed):
    """Upper band of nb super-diagonals, packed: row j of the tensor is column j, ldab = 3 nb."""
    n, nb = case["n"], case["nb"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ty = _TYPES[case["dtype"]]
    band = torch.zeros(n, 3 * nb, dtype=ty, device="cuda")
    # entry (i, j) at [j, i - j + 2 nb - 1], j - nb <= i <= j
    part = torch.randn(n, nb + 1, dtype=ty, device="cuda", generator=gen) / math.sqrt(nb)
    i = torch.arange(n, device="cuda")[:, None] + torch.arange(-nb, 1, device="cuda")[None, :]
    band[:, nb - 1:2 * nb] = torch.where(i >= 0, part, torch.zeros_like(part))
    return band


def _bidiagonal(case, seed):
    """Diagonal and super-diagonal as the reduction of a Gaussian matrix leaves them (chi distributed)."""
    n = case["n"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ty = _TYPES[case["dtype"]]
    left = torch.arange(n, 0, -1, dtype=torch.float64, device="cuda")
    g = torch.randn(2, n, dtype=torch.float64, device="cuda", generator=gen)
    d = (left.sqrt() + 0.7 * g[0]) / math.sqrt(n)
    e = ((left - 1.0).clamp(min=0.0).sqrt() + 0.7 * g[1]) / math.sqrt(n)
    e[n - 1] = 0.0
    return d.to(ty), e.to(ty)


def _scratch(rc_bytes):
    assert rc_bytes[0] == svb.SVB_OK
    return torch.empty(max(rc_bytes[1], 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    state = {"case": case}
    code = svb.dtype_code(_TYPES[case["dtype"]])
    if case["kind"] == "dense":
        state["a"] = _matrix(case, seed)
        state["work"] = _scratch(svb.svb_workspace_bytes(code, case["m"], case["n"], case["nb"])[:2])
        return state
    n = case["n"]
    state["code"] = code
    if case["kind"] == "band":
        state["band0"] = _band(case, seed)
        state["band"] = torch.empty_like(state["band0"])
        state["work2"] = _scratch(svb.svb_gb2bd_workspace_bytes(n, case["nb"]))
        state["d"] = torch.empty(n, dtype=_TYPES[case["dtype"]], device="cuda")
        state["e"] = torch.empty(n, dtype=_TYPES[case["dtype"]], device="cuda")
    else:
        state["d"], state["e"] = _bidiagonal(case, seed)
    state["sigma"] = torch.empty(n, dtype=_TYPES[case["dtype"]], device="cuda")
    state["work3"] = _scratch(svb.svb_bdsvals_dev_workspace_bytes(n))
    return state


def _ok(rc):
    if rc != svb.SVB_OK:
        raise svb.SvbError(rc, "cases")


def run(state):
    case = state["case"]
    if case["kind"] == "dense":
        return svb.svdvals(state["a"], nb=case["nb"], work=state["work"])
    n = case["n"]
    if case["kind"] == "band":
        state["band"].copy_(state["band0"])     # the reduction consumes the band
        _ok(svb.svb_gb2bd(state["code"], n, case["nb"], state["band"], 3 * case["nb"], state["d"], state["e"],
                          state["work2"], state["work2"].numel()))
    _ok(svb.svb_bdsvals_dev(state["code"], n, state["d"], state["e"], state["sigma"], 0.0, state["work3"],
                            state["work3"].numel()))
    return state["sigma"]


def work(case):
    cs = _BYTES[case["dtype"]]
    out = 8 if case["dtype"] == "f64" else 4
    if case["kind"] == "dense":
        k, long = min(case["m"], case["n"]), max(case["m"], case["n"])
        # bidiagonalisation of the matrix, or of the triangular factor of its QR where that is less
        flops = min(4.0 * long * k * k - 4.0 / 3.0 * k ** 3, 2.0 * long * k * k + 2.0 * k ** 3)
        return {"bytes": case["m"] * case["n"] * cs + k * out, "flops": flops}
    n = case["n"]
    if case["kind"] == "band":      # about n^2 / (2 nb) steps of two reflectors on 2 nb lines of nb entries
        return {"bytes": (case["nb"] + 1) * n * cs + n * out, "flops": 8.0 * n * n * case["nb"]}
    return {"bytes": 2 * n * cs + n * out, "flops": 6.0 * n * n}    # about three passes over the rest per value


def tolerance(case):
    # about four times the distance from 64 bits that the path shows, over types, kinds and orders: 64-bit
    # errors grow with the order (6e-15 at 256, 1.0e-13 at 4096, 1.8e-13 at 5532), 32-bit ones are 1e-7 to
    # 3.4e-7, f16 3e-5 to 7e-5, bf16 1.0e-4 to 1.5e-4 at orders up to 1537
    k = case["n"] if case["kind"] != "dense" else min(case["m"], case["n"])
    rel0, rel1, max0, max1 = {"f64": (1e-14, 1e-16, 3e-14, 2.5e-16), "f32": (4e-7, 1.2e-10, 1.5e-6, 6e-10),
                              "f16": (1.2e-4, 4e-8, 5e-4, 2e-7), "bf16": (6e-4, 4e-7, 2.5e-3, 1.5e-6)}[case["dtype"]]
    # (clusters are far below the storage rounding of the largest values: 16-bit errors there are four times as large)
    f = 4.0 if case.get("values") == "clustered" and case["dtype"] in ("f16", "bf16") else 1.0
    return {"rel": f * (rel0 + rel1 * k), "max": f * (max0 + max1 * k)}


def exact(case, seed):
    if case["kind"] == "dense":
        a = _matrix(case, seed)
        k, long = sorted(a.shape)
        if k > 8192 or long * k * k > 5.6e11:
            return None
    else:
        n = case["n"]
        if n > 8192:
            return None
        a = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        if case["kind"] == "band":
            band, nb = _band(case, seed).double(), case["nb"]
            for t in range(min(nb, n - 1) + 1):     # super-diagonal t
                a.diagonal(t).copy_(band[t:, 2 * nb - 1 - t])
        else:
            d, e = _bidiagonal(case, seed)
            a.diagonal().copy_(d.double())
            a.diagonal(1).copy_(e.double()[:n - 1])
    s = torch.linalg.svdvals(a.double().cpu())
    return s.numpy() if case["kind"] == "dense" else s
