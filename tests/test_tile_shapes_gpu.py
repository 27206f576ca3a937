"""The tiled GEMM's tile shapes (8-bit: 256 x 128, 128 x 128, 64 x 128 and
64 x 64 outputs per workgroup; 4-bit: the last three) and their split plans, at sizes that take each
(tile_sizes.py): one row past a tile, half tiles of columns, all tiles split along
K, a last round of whole tiles with split ones beside them.  Integer codes and
power-of-two steps make every sum exact (|sum| < 2^24 steps), so the outputs
must EQUAL the integer product in every order of the sums; guard rows around
the output must stay as they were."""
import pytest
import torch
from tile_sizes import EIGHT, FOUR, GELU_EIGHT, GELU_FOUR

from paper_2609_39056_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def random_weight(K, N, group, gen):
    """Random packed codes in [-7, 7], power-of-two steps; (Weight, codes [N, K] fp64, steps [K/group, N] fp64)."""
    codes = torch.randint(-7, 8, (N, K), generator=gen, device="cuda", dtype=torch.int32)
    lo = codes.view(N, K // 8, 2, 4)
    qw = ((lo[:, :, 0] & 15) | ((lo[:, :, 1] & 15) << 4)).to(torch.uint8).reshape(N, K // 2).contiguous()
    step = torch.exp2(torch.randint(-1, 1, (K // group, N), generator=gen, device="cuda").float())
    return B.Weight(qw=qw, w_scale=step.half().contiguous(), w_group=group), codes.double(), step.double()


@pytest.mark.parametrize("group", [128, 0])
@pytest.mark.parametrize("with_ws", [True, False])
@pytest.mark.parametrize("M,K,N", EIGHT)
def test_tile_shapes_exact(M, K, N, with_ws, group):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * 7 + K + N)
    G = group or K
    W, codes, step = random_weight(K, N, G, gen)
    qx = torch.randint(-31, 32, (M, K), generator=gen, device="cuda", dtype=torch.int32).to(torch.int8)
    r = torch.exp2(torch.randint(-2, 3, (M,), generator=gen, device="cuda").float())
    buf = torch.full((M + 2, N), -7.5, dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(B.SQ_VARIANT_GEMM, M, K, N, 8) if with_ws else None
    B.sq_gemm_w4a8(qx, r, W, buf[1:M + 1], B.SQ_OUT_F32, ws)
    wd = (codes.view(N, K // G, G) * step.t().unsqueeze(2)).view(N, K)
    want = qx.double() @ wd.t()
    assert float((qx.double().abs() @ wd.abs().t()).max()) < 2.0**23  # in units of the smallest step, 1/2: < 2^24
    assert torch.equal(buf[1:M + 1].double(), want * r.double().unsqueeze(1))
    assert bool((buf[0] == -7.5).all()) and bool((buf[M + 1] == -7.5).all())


@pytest.mark.parametrize("group", [128, 0])
@pytest.mark.parametrize("M,K,N", GELU_EIGHT)
def test_tile_shapes_gelu_epilogue(M, K, N, group):
    """The fused up projection's codes and row scales against the three
    separate calls, bit for bit, on the same shapes."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K + N)
    W, _, _ = random_weight(K, N, group or K, gen)
    W = B.Weight(qw=W.qw, w_scale=(W.w_scale.float() * 2.0**-7).half(), w_group=W.w_group,
                 bias=(torch.randn((N,), generator=gen, device="cuda") * 0.1).to(torch.bfloat16))
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    t2s = torch.randint(0, 3, (M,), generator=gen, device="cuda", dtype=torch.int32)
    gamma = torch.exp(torch.randn((2, 3), generator=gen, device="cuda") * 0.3)
    dinv = torch.rand((N,), generator=gen, device="cuda") + 0.5
    act = B.ActParams(tok2stream=t2s, gamma=gamma, step=1)
    nxt = B.ActParams(tok2stream=t2s, gamma=gamma, step=0, range_mode=B.SQ_RANGE_STATIC,
                      clip=torch.tensor([2.5, 3.0], device="cuda"), dinv=dinv)
    ws = B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, 8)
    qx, r = B.act_buffers(M, N, 8)
    B.sq_linear_w4a8_gelu_quant(x, act, W, nxt, qx, r, ws)
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    B.sq_linear_w4a8(x, act, W, y, B.SQ_OUT_BF16, ws)
    B.sq_gelu_bf16(y, y)
    qx2, r2 = B.act_buffers(M, N, 8)
    B.sq_quantize_act(y, nxt, qx2, r2)
    assert torch.equal(qx, qx2)
    assert torch.equal(r.view(torch.int32), r2.view(torch.int32))


@pytest.mark.parametrize("with_ws", [True, False])
@pytest.mark.parametrize("M,K,N", FOUR)
def test_tile_shapes_exact_4bit(M, K, N, with_ws):
    """Codes as fp8 bytes of code * 2^-9, power-of-two group steps, kc from its definition."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M * 5 + K + N)
    W, codes, step = random_weight(K, N, 128, gen)
    q = torch.randint(-7, 8, (M, K), generator=gen, device="cuda", dtype=torch.int32)
    qx = (q.abs() | ((q < 0).int() << 7)).to(torch.uint8)
    sigma = torch.exp2(torch.randint(-1, 2, (M, K // 64), generator=gen, device="cuda").float())
    kc = -8.0 * q.view(M, K // 64, 64).sum(2).float() * sigma * 2.0**-18
    act = B.ActParams(tok2stream=torch.zeros(M, dtype=torch.int32, device="cuda"),
                      gamma=torch.full((1, 1), 0.5, device="cuda"), step=0, act_bits=4)
    buf = torch.full((M + 2, N), -7.5, dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(B.SQ_VARIANT_GEMM, M, K, N, 4) if with_ws else None
    B.sq_gemm_w4a4_fp8(qx, sigma, kc, act, W, buf[1:M + 1], B.SQ_OUT_F32, ws)
    xd = (q.view(M, K // 64, 64).double() * sigma.double().unsqueeze(2)).view(M, K)
    wd = (codes.view(N, K // 128, 128) * step.t().unsqueeze(2)).view(N, K)
    assert float((xd.abs() @ wd.abs().t()).max()) < 2.0**22  # in units of the smallest step, 1/4: < 2^24
    assert torch.equal(buf[1:M + 1].double(), (xd @ wd.t()) * 2.0)
    assert bool((buf[0] == -7.5).all()) and bool((buf[M + 1] == -7.5).all())


@pytest.mark.parametrize("M,K,N", GELU_FOUR)
def test_tile_shapes_gelu_epilogue_4bit(M, K, N):
    """The fused up projection followed by the down GEMM against the three
    separate calls, bit for bit, on the same shapes."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + K + N)
    W, _, _ = random_weight(K, N, 128, gen)
    W = B.Weight(qw=W.qw, w_scale=(W.w_scale.float() * 2.0**-5).half(), w_group=W.w_group,
                 bias=(torch.randn((N,), generator=gen, device="cuda") * 0.1).to(torch.bfloat16))
    D, _, _ = random_weight(N, 64, 128, gen)
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    t2s = torch.randint(0, 3, (M,), generator=gen, device="cuda", dtype=torch.int32)
    gamma = torch.exp(torch.randn((2, 3), generator=gen, device="cuda") * 0.3)
    act = B.ActParams(tok2stream=t2s, gamma=gamma, step=1, act_bits=4)
    nxt = B.ActParams(tok2stream=t2s, gamma=gamma, step=0, act_bits=4, range_mode=B.SQ_RANGE_STATIC,
                      clip=torch.tensor([2.5, 3.0], device="cuda"),
                      dinv=torch.rand((N,), generator=gen, device="cuda") + 0.5)
    ws = B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, 4)
    wd = B.alloc_workspace(B.SQ_VARIANT_FUSED, M, N, 64, 4)
    qx = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    sg, kc = (torch.empty((M, N // 64), dtype=torch.float32, device="cuda") for _ in range(2))
    out = torch.empty((M, 64), dtype=torch.float32, device="cuda")
    want = torch.empty_like(out)
    B.sq_linear_w4a4_gelu_quant(x, act, W, nxt, qx, sg, kc, ws)
    B.sq_gemm_w4a4_fp8(qx, sg, kc, nxt, D, out, B.SQ_OUT_F32, wd)
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    B.sq_linear_w4a4(x, act, W, y, B.SQ_OUT_BF16, ws)
    B.sq_gelu_bf16(y, y)
    B.sq_linear_w4a4(y, nxt, D, want, B.SQ_OUT_F32, wd)
    assert torch.equal(out, want)
