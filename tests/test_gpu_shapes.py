"""GPU parity of the kernels chosen by size and type, at the sizes where their
rules and tile edges lie.  Whole passes (pair forward and JAGG group backward)
against the oracle in fp64; bars as in test_gpu_parity: fp32 1e-4, bf16 2e-2,
globally and per tensor."""
import numpy as np
import pytest
import torch

import paper_2607_17572_amd as pk
import synth
from harness import Case, compare_grads, rel_l2, rounded, to_dev
from oracle import mmdit

pytestmark = pytest.mark.gpu


def block(heads, head_dim, n_txt, lat_h, lat_w, act=pk.F32, **over):
    d = heads * head_dim
    k = dict(n_double=1, n_single=0, hidden=d, heads=heads, head_dim=head_dim, mlp_hidden=4 * d, in_ch=16, patch=2,
             lat_h=lat_h, lat_w=lat_w, n_txt=n_txt, txt_dim=d, t_freq_dim=256, block_only=1, act_dtype=act,
             grad_dtype=pk.F32)
    k.update(over)
    return pk.Config(**k)


def check_pass(c, B, W, tol):
    cs = Case(c, B=B, W=W)
    eg, worst = compare_grads(cs, cs.gpu_jagg(), cs.oracle_jagg(), tol, report=True)
    print(f"rel L2 {eg:.2e}, worst tensor {worst}", flush=True)


# fp32 products: 64 x 64 tiles from 480 of them on (4 x 517 rows: 528 tiles for the MLP's first layer), 32 x 32 tiles
# below, ragged rows in both; rows that are not 16-byte aligned (3-wide patches, 30-wide text embeddings)
@pytest.mark.parametrize("c,B", [
    (block(4, 64, 77, 40, 44), 2),
    (block(3, 16, 5, 6, 10), 1),
    (block(2, 32, 7, 6, 5, block_only=0, in_ch=3, patch=1, txt_dim=30, n_single=1), 1),
], ids=["tiles64", "tiles32", "unaligned"])
def test_fp32_products(c, B):
    check_pass(c, B, 3, 1e-4)


# bf16 operands whose rows are not 16-byte aligned, at 64 x 64 tiles of the fp32 kernel (32 x 32 of them)
def test_unaligned_bf16_products():
    rows, n_out, n_in = 2001, 2004, 516
    dY = rounded(synth.normal((rows, n_out), 1), torch.bfloat16)
    X = rounded(synth.normal((rows, n_in), 2), torch.bfloat16)
    W = rounded(synth.normal((n_out, n_in), 3, scale=0.02), torch.bfloat16)
    ctx = pk.Context(pk.config("tiny"))
    dX = torch.empty(rows, n_in, dtype=torch.float32, device="cuda")
    ctx.linear_grad(pk.DGRAD, to_dev(dY, torch.bfloat16), to_dev(W, torch.bfloat16), dX)
    dW = torch.ones(n_out, n_in, dtype=torch.float32, device="cuda")
    ctx.linear_grad(pk.WGRAD, to_dev(dY, torch.bfloat16), to_dev(X, torch.bfloat16), dW, beta=1.0)
    # fp32 sums of exact products: 2000 terms, relative error below sqrt(2000) 2^-24 = 3e-6
    assert rel_l2(dX.double().cpu().numpy(), dY @ W) <= 1e-5
    assert rel_l2(dW.double().cpu().numpy(), 1.0 + mmdit.wgrad(dY, X)) <= 1e-5


# bf16 products of 64 x 64 and 128 x 128 direct-to-LDS tiles: one row below and above a tile edge, one k tile, ragged k in the weight gradient (rows), K = 96 (not a multiple of 64), an odd number of
# k tiles over two k groups (1057 rows: 34 with a ragged last one; K = 1056: 33)
@pytest.mark.parametrize("rows,n_out,n_in", [(8, 64, 64), (63, 96, 72), (65, 64, 136), (129, 768, 200), (1057, 72, 96), (200, 1056, 136), (127, 2048, 1024),
                                             (1089, 1536, 768), (2500, 1544, 1536)])
def test_bf16_product_tiles(rows, n_out, n_in):
    dY = rounded(synth.normal((rows, n_out), 5), torch.bfloat16)
    X = rounded(synth.normal((rows, n_in), 6), torch.bfloat16)
    W = rounded(synth.normal((n_out, n_in), 7, scale=0.02), torch.bfloat16)
    ctx = pk.Context(pk.config("tiny"))
    dX = torch.empty(rows, n_in, dtype=torch.float32, device="cuda")
    dYd, Xd, Wd = (to_dev(x, torch.bfloat16) for x in (dY, X, W))
    ctx.linear_grad(pk.DGRAD, dYd, Wd, dX)
    # rows past the last one of X and of dY must not reach the sums: each the first rows of a larger allocation, the
    # rest NaN (both, since a NaN of one times a zero read for the other shows, and a finite value would not)
    def within_nan(x):
        big = torch.full((rows + 64, x.shape[1]), float("nan"), dtype=torch.bfloat16, device="cuda")
        big[:rows] = x
        return big[:rows]

    dYn, Xn = within_nan(dYd), within_nan(Xd)
    dW = torch.ones(n_out, n_in, dtype=torch.float32, device="cuda")
    ctx.linear_grad(pk.WGRAD, dYn, Xn, dW, beta=1.0)
    dWb = torch.ones(n_out, n_in, dtype=torch.bfloat16, device="cuda")
    ctx.linear_grad(pk.WGRAD, dYn, Xn, dWb, beta=1.0)
    want = 1.0 + mmdit.wgrad(dY, X)
    # fp32 sums of exact products (K <= 2500: below 1e-5); one bf16 rounding is 2^-9 at most
    assert rel_l2(dX.double().cpu().numpy(), dY @ W) <= 1e-5
    assert rel_l2(dW.double().cpu().numpy(), want) <= 1e-5
    assert rel_l2(dWb.double().cpu().numpy(), want) <= 8e-3


@pytest.mark.parametrize("c,B", [
    (block(6, 128, 77, 10, 14, act=pk.BF16), 1),   # 64 x 64 tiles
    # 128 x 128 (register-staged in the forward) and 64 x 64
    (block(6, 128, 77, 34, 38, act=pk.BF16, block_only=0, n_single=1), 2),
    (block(3, 32, 9, 6, 6, act=pk.BF16), 1),  # K = 96 and 288
    # forward products on 128 x 128 direct-to-LDS tiles: K = 480 is not a multiple of 64, 168 to 351 tiles with all
    # three epilogues (bias; bias + GELU; both in one launch for the single block)
    (block(15, 32, 77, 34, 38, act=pk.BF16, block_only=0, n_single=1), 2),
], ids=["tiles64", "tiles128", "k96", "k480"])
def test_bf16_products_of_a_pass(c, B):
    check_pass(c, B, 3, 2e-2)


# forward products on 192 x 192 and 256 x 192 tiles, ragged in both streams' rows: the MLP's first layer of a double
# block and a single block's whole input projection (24192-wide MLP: 252 and 254 tiles in one round of the CUs), and a
# q/k/v projection (252 tiles of 192 x 192; 204 of 256 x 192)
@pytest.mark.parametrize("c,B", [
    (block(1, 64, 75, 38, 10, act=pk.BF16, mlp_hidden=24192, block_only=0, n_single=1), 1),
    (block(1, 64, 100, 50, 10, act=pk.BF16, mlp_hidden=24192, block_only=0, n_single=1), 1),
    (block(3, 128, 40, 58, 66, act=pk.BF16, mlp_hidden=64), 4),
    (block(3, 128, 43, 62, 66, act=pk.BF16, mlp_hidden=64), 4),
], ids=["mlp192", "mlp256x192", "qkv192", "qkv256x192"])
def test_bf16_forward_tiles(c, B):
    check_pass(c, B, 2, 2e-2)


# time MLP and modulations at each samples-per-thread form of their backward (batch 2, 4, 8, 16, 32 of the pair), rows
# that are not a multiple of the 8-row tiles, and a frequency width without 16-byte rows
@pytest.mark.parametrize("B,over", [(1, {}), (2, {}), (3, {}), (6, {}), (13, {}), (2, dict(t_freq_dim=250))],
                         ids=["pair2", "pair4", "pair6", "pair12", "pair26", "unaligned"])
def test_modulation_batches(B, over):
    check_pass(block(3, 16, 2, 4, 4, **over), B, 2, 1e-4)
    check_pass(block(2, 32, 2, 4, 4, act=pk.BF16, grad_dtype=pk.BF16, **over), B, 2, 2e-2)


# attention: bf16 head dim 64 and 128 (128-query and 128-key blocks, 64-row tiles) and the fp32-arithmetic kernels (32
# queries or keys per workgroup, four waves taking every fourth 32-row tile): one tile, one row beyond, several
@pytest.mark.parametrize("act,head_dim,n_txt,lat_h,lat_w", [
    (pk.BF16, 64, 3, 4, 4), (pk.BF16, 64, 28, 12, 12), (pk.BF16, 64, 29, 12, 12), (pk.BF16, 64, 65, 16, 16),
    (pk.BF16, 64, 77, 24, 26), (pk.BF16, 128, 65, 16, 16), (pk.BF16, 32, 9, 6, 8), (pk.BF16, 16, 21, 12, 14),
    (pk.F32, 16, 28, 4, 4), (pk.F32, 32, 29, 4, 4), (pk.F32, 64, 33, 12, 16), (pk.F32, 128, 77, 10, 12),
])
def test_attention_shapes(act, head_dim, n_txt, lat_h, lat_w):
    check_pass(block(2, head_dim, n_txt, lat_h, lat_w, act=act), 1, 2, 2e-2 if act == pk.BF16 else 1e-4)


# group scores: 16-byte and element loads, a last incomplete step, fewer elements than threads; fp64 sums of exact
# products differ from numpy's by their order only (n <= 3e5: below n 2^-53)
@pytest.mark.parametrize("n,off", [(5, 0), (8, 0), (4099, 0), (300007, 0), (4099, 1)])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("W", [2, 5, 8])
def test_group_score_forms(n, off, dt, W):
    x = [to_dev(synth.normal((n + off,), 50 + j) + synth.normal((n + off,), 9), dt)[off:] for j in range(W)]
    ctx = pk.Context(pk.config("tiny"))
    v = [t.double().cpu().numpy() for t in x]
    cos = [float(v[i] @ v[j] / np.sqrt((v[i] @ v[i]) * (v[j] @ v[j]))) for i in range(W) for j in range(i + 1, W)]
    assert abs(ctx.group_score(x) - np.mean(cos)) <= 1e-12


# LayerNorm and q/k norm kernels: hidden sizes whose last 512-column run is incomplete, exact, and the widest (4096);
# every head dim with fewer, as many and more heads than one step of a wave takes (512 / head dim)
@pytest.mark.parametrize("heads,head_dim", [(3, 16), (33, 16), (16, 32), (21, 32), (9, 64), (12, 64), (5, 128), (32, 128)])
@pytest.mark.parametrize("act", [pk.F32, pk.BF16])
def test_norm_widths(heads, head_dim, act):
    check_pass(block(heads, head_dim, 3, 4, 6, act=act, mlp_hidden=64), 1, 2, 2e-2 if act == pk.BF16 else 1e-4)


# a single block whose rows of q, k, v and MLP (3 hidden + MLP) and of attention output and MLP (hidden + MLP) are not
# multiples of four elements: products, attention and q/k norm on their element loads
@pytest.mark.parametrize("heads,head_dim", [(4, 16), (2, 64), (1, 128)])
@pytest.mark.parametrize("act", [pk.F32, pk.BF16])
def test_mlp_widths_of_a_single_block(heads, head_dim, act):
    check_pass(block(heads, head_dim, 9, 4, 6, act=act, block_only=0, n_single=1, mlp_hidden=170), 1, 2,
               2e-2 if act == pk.BF16 else 1e-4)


# hidden sizes that are not multiples of 8: a network without blocks (its final LayerNorm on the element-wise kernels;
# the text embedding then has no gradient), and with blocks refused for their head dim
@pytest.mark.parametrize("act", [pk.F32, pk.BF16])
def test_hidden_sizes_without_attention(act):
    none = dict(n_double=0, block_only=0, in_ch=3, patch=1, txt_dim=20)
    check_pass(block(5, 4, 9, 4, 6, act=act, **none), 2, 2, 2e-2 if act == pk.BF16 else 1e-4)
    check_pass(block(3, 100, 2, 5, 7, act=act, **none), 1, 2, 2e-2 if act == pk.BF16 else 1e-4)
    for over in (dict(), dict(block_only=0)):
        for heads, head_dim in ((5, 4), (2, 20)):
            with pytest.raises(pk.api.JaggError, match="head_dim must be 16, 32, 64 or 128") as e:
                Case(block(heads, head_dim, 9, 4, 6, act=act, **over), B=1, W=2).saved_pair()
            assert e.value.status == 4
