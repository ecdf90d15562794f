"""The attention kernels by themselves, through the library's internal entry
points, against softmax attention in fp64 on the same operands: what a whole
pass cannot show, since its other bf16 roundings are as large."""
import ctypes
import math

import pytest
import torch

import paper_2607_17572_amd as pk

pytestmark = pytest.mark.gpu

P, I = ctypes.c_void_p, ctypes.c_int


class RowMap(ctypes.Structure):
    _fields_ = [("B", I), ("nt", I), ("ni", I)]


class Fwd(ctypes.Structure):
    _fields_ = [("Q", P), ("K", P), ("V", P), ("O", P), ("ld_o", I), ("lse", P), ("B", I), ("H", I), ("N", I),
                ("Dh", I), ("dt", I), ("rm", RowMap)]


class Bwd(ctypes.Structure):
    _fields_ = [("Q", P), ("K", P), ("V", P), ("O", P), ("ld_o", I), ("dO", P), ("ld_do", I), ("lse", P),
                ("delta", P), ("dQ", P), ("dK", P), ("dV", P), ("dt_d", I), ("B", I), ("H", I), ("N", I), ("Dh", I),
                ("dt", I), ("rm", RowMap), ("dS", P), ("ld_ds", I), ("nk_pad", I)]


def call(name, args):
    """jg::attention_<name>(args, null stream)"""
    f = getattr(pk.lib(), f"_ZN2jg13attention_{name}ERKNS_7Attn{name.capitalize()}EP12ihipStream_t")
    f.argtypes, f.restype = [P, P], I
    assert f(ctypes.addressof(args), None) == 0, pk.api.lib().jagg_last_error()


def rows_of_tokens(B, nt, ni):
    """[B][N] rows of the stream-major layout"""
    b = torch.arange(B, device="cuda")[:, None]
    j = torch.arange(nt + ni, device="cuda")[None]
    return torch.where(j < nt, b * nt + j, B * nt + b * ni + (j - nt))


def token_major(x, rows, ld):
    """[B][H][N][Dh] -> rows of ld elements, head h at columns h * Dh; the rest NaN"""
    B, H, N, Dh = x.shape
    out = torch.full((B * N, ld), float("nan"), dtype=x.dtype, device="cuda")
    out[rows.reshape(-1), :H * Dh] = x.permute(0, 2, 1, 3).reshape(B * N, H * Dh)
    return out


def run(dt, Dh, B, H, nt, ni, extra=0):
    """{name: (kernel's result, fp64 result)}; extra: columns of the rows of O beyond the heads'"""
    N, ld = nt + ni, H * Dh + extra
    g = torch.Generator(device="cuda").manual_seed(100 * Dh + N)
    q, k, v, do = (torch.randn((B, H, N, Dh), generator=g, device="cuda", dtype=torch.float32).to(dt) for _ in range(4))
    q64, k64, v64, do64 = (x.double() for x in (q, k, v, do))
    s = torch.stack([torch.stack([q64[b, h] @ k64[b, h].t().contiguous() for h in range(H)]) for b in range(B)]) / math.sqrt(Dh)
    lse64 = torch.logsumexp(s, -1)
    p = torch.exp(s - lse64[..., None])
    mm = lambda a, b: torch.stack([torch.stack([a[i, j] @ b[i, j] for j in range(H)]) for i in range(B)])
    t = lambda a: a.transpose(-1, -2).contiguous()
    o64 = mm(p, v64)
    rows, code = rows_of_tokens(B, nt, ni), pk.BF16 if dt == torch.bfloat16 else pk.F32
    rm = RowMap(B, nt, ni)
    O = torch.full((B * N, ld), float("nan"), dtype=dt, device="cuda")
    lse = torch.empty((B, H, N), device="cuda", dtype=torch.float32)
    call("fwd", Fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), O.data_ptr(), ld, lse.data_ptr(), B, H, N, Dh, code, rm))
    out = {"O": (O[rows][..., :H * Dh].reshape(B, N, H, Dh).permute(0, 2, 1, 3), o64), "lse": (lse, lse64)}
    # the backward from the stored O and log-sum-exp, as the pass has them
    o, lse32 = o64.to(dt), lse64.float()
    p = torch.exp(s - lse32.double()[..., None])
    ds = p * (mm(do64, t(v64)) - (do64 * o.double()).sum(-1, keepdim=True)) / math.sqrt(Dh)
    ref = {"dQ": mm(ds, k64), "dK": mm(t(ds), q64), "dV": mm(t(p), do64)}
    got = {n: torch.full_like(q, float("nan")) for n in ref}
    Or, dOr = token_major(o, rows, ld), token_major(do, rows, H * Dh)
    delta = torch.empty((2, B, H, N), device="cuda", dtype=torch.float32)
    call("bwd", Bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), Or.data_ptr(), ld, dOr.data_ptr(), H * Dh,
                    lse32.data_ptr(), delta.data_ptr(), got["dQ"].data_ptr(), got["dK"].data_ptr(),
                    got["dV"].data_ptr(), code, B, H, N, Dh, code, rm, None, 0, 0))
    torch.cuda.synchronize()
    out.update({n: (got[n], ref[n]) for n in ref})
    return out


def err(x, y):
    return float((x.double() - y).norm() / y.norm())


TOKENS = [(1, 4), (28, 100), (29, 100), (77, 256)]


# Products of bf16 operands with probabilities and dS in (at least) 17 bits and fp32 sums: the results are those of
# fp64 rounded to bf16, so their error is the rounding's (a bf16 rounding of P or dS on the way adds 20% and more).
@pytest.mark.parametrize("nt,ni", TOKENS)
@pytest.mark.parametrize("Dh", [16, 32, 64])
def test_bf16_results_are_rounded_once(Dh, nt, ni):
    for name, (x, y) in run(torch.bfloat16, Dh, 2, 3, nt, ni).items():
        e = err(x, y)
        once = err(y.to(torch.bfloat16), y) if name != "lse" else 1e-6
        print(f"{Dh} {nt}+{ni} {name}: {e:.3e}, rounding alone {once:.3e}", flush=True)
        assert e <= 1.01 * once, name


# Rows of O that are not a multiple of four elements (a single block of such an MLP width), and fp32 sums of fp32
# operands: every term carries a few roundings of 2^-24, the exponential one of its argument (below 8 here)
# (bf16 head dim 128 takes the fp32-arithmetic kernels at such widths only)
@pytest.mark.parametrize("dt,Dh,extra", [(dt, Dh, extra) for dt in (torch.float32, torch.bfloat16)
                                         for Dh in (16, 32, 64, 128) for extra in (0, 1, 170)
                                         if (dt, Dh, extra) != (torch.bfloat16, 128, 0)])
def test_row_widths(dt, Dh, extra):
    for name, (x, y) in run(dt, Dh, 2, 2, 29, 40, extra).items():
        e = err(x, y)
        bar = 1.01 * err(y.to(dt), y) if dt == torch.bfloat16 and name != "lse" else 2e-6
        print(f"{dt} {Dh} +{extra} {name}: {e:.3e}, bar {bar:.3e}", flush=True)
        assert e <= bar, name
