"""The batched decode launches (tm_tgemv_rms16, tm_mixer_gate_part, tm_tgemv):
the projections against float64 over the batches, group sizes and edges of its
blocks, and whole tokens against the unfused decode, eager and replayed."""

import pytest

torch = pytest.importorskip("torch")

from paper_2606_18114_amd import ops  # noqa: E402
from paper_2606_18114_amd.stack import Mamba2Decoder  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _packed(gen, N, K, g):
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    codes, s, s16, _ = ops.ternarize_pack(w, g, 1e-5)
    tau = (s + 1e-5).repeat_interleave(g, dim=1)
    q = (torch.sign(w) * (w.abs() > 0.5 * tau)).double()
    return codes, s16, q * s16.double().repeat_interleave(g, 1)


# (B, N, K, g): one row and all sixteen, one block and one output, blocks of
# two and ragged ones, fewer groups than waves, several rounds of chunks
@pytest.mark.parametrize("B,N,K,g", [(1, 1, 64, 64), (5, 130, 256, 256), (16, 2048, 4096, 128),
                                     (9, 8512, 2048, 128), (12, 8500, 512, 64),
                                     (16, 17, 4096, 256), (7, 6170, 320, 64)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_projection(B, N, K, g, accumulate):
    print(f"[decode16] B={B} N={N} K={K} g={g} accumulate={accumulate}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B + N)
    codes, s16, what = _packed(gen, N, K, g)
    src = torch.randn((B, K), generator=gen, device="cuda")
    nw = 1 + 0.1 * torch.randn(K, generator=gen, device="cuda")
    P = 3
    cuts = [0, K // 4, K // 2, K]
    part = torch.stack([src[:, a:b].square().sum(1) for a, b in zip(cuts, cuts[1:])], 1)
    y0 = torch.randn((B, N), generator=gen, device="cuda")
    y = y0.clone()
    part_out = torch.full((B, (N + 15) // 16), float("nan"), device="cuda")
    pos = torch.tensor([3], dtype=torch.int32, device="cuda")
    ops.tgemv_rms16(src, part.contiguous(), codes, s16, g, nw, 1e-5, y, accumulate=accumulate,
                    part_out=part_out, advance=pos)
    assert P == part.shape[1] and int(pos) == 0
    r = 1 / torch.sqrt(part.sum(1) / K + 1e-5)
    x = (src * r[:, None] * nw).to(torch.bfloat16).double()
    ref = x @ what.t() + (y0.double() if accumulate else 0)
    mag = x.abs() @ what.abs().t() + y0.double().abs()
    # float32 sums of exact products; an x on the edge of its bfloat16
    # rounding (another order of the sums of squares) may move by 2^-8
    err = (y.double() - ref).abs()
    assert bool((err <= (K ** 0.5 * 2.0 ** -23 + 2.0 ** -9 / K ** 0.5) * mag).all())
    sq = torch.zeros((B, (N + 15) // 16 * 16), device="cuda", dtype=torch.float64)
    sq[:, :N] = y.double().square()
    assert torch.allclose(part_out.double(), sq.view(B, -1, 16).sum(2), rtol=2e-6)


def _bits(t):
    return t.contiguous().view(torch.uint8)


# one in nine rows and all sixteen, fewer groups than waves and several per
# wave, columns that are no multiple of 256, rows that end inside a block
@pytest.mark.parametrize("B,N,K,g", [(9, 17, 64, 64), (16, 8512, 2048, 128), (16, 2048, 4096, 64),
                                     (12, 8500, 3904, 64), (16, 12400, 4096, 64),
                                     (11, 530, 1280, 256), (10, 8200, 1088, 64),
                                     (13, 6170, 2176, 128)])
def test_projection_has_the_bits_of_the_unfused_launches(B, N, K, g):
    print(f"[decode16] bits B={B} N={N} K={K} g={g}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B + N)
    codes, s16, _ = _packed(gen, N, K, g)
    src = torch.randn((B, K), generator=gen, device="cuda")
    nw = 1 + 0.1 * torch.randn(K, generator=gen, device="cuda")
    y0 = torch.randn((B, N), generator=gen, device="cuda")
    x = torch.empty((1, B, K), dtype=torch.bfloat16, device="cuda")
    ops.residual_rmsnorm(src.clone(), None, nw, 1e-5, x=x[0])
    ref = ops.tgemv(x, codes[None], s16[None], g)[0]
    for accumulate in (False, True):
        y = y0.clone()
        ops.tgemv_rms16(src, None, codes, s16, g, nw, 1e-5, y, accumulate=accumulate)
        assert torch.equal(_bits(y), _bits(y0 + ref if accumulate else ref))


@pytest.mark.parametrize("B,d_model,heads,g", [(5, 256, 8, 64), (16, 512, 16, 128),
                                               (12, 768, 24, 256), (8, 2048, 64, 128),
                                               (9, 1024, 64, 64), (16, 2048, 64, 128)])
def test_token_matches_the_unfused_decode(B, d_model, heads, g):
    print(f"[decode16] token B={B} d_model={d_model} heads={heads} g={g}", flush=True)
    L, di = 3, 64 * heads
    cd = di + 256

    def build(**kw):
        def weight(side, l):
            n, k = (2 * di + 256 + heads, d_model) if side == "in" else (d_model, di)
            gw = torch.Generator(device="cuda").manual_seed(100 * l + (side == "in"))
            return torch.randn((n, k), generator=gw, device="cuda") * 0.02

        def mixer(l):
            gm = torch.Generator(device="cuda").manual_seed(1000 + l)
            u = lambda *s: torch.rand(s, generator=gm, device="cuda")  # noqa: E731
            return dict(conv_w=u(cd, 4) - 0.5, conv_b=u(cd) - 0.5, dt_bias=u(heads) - 4,
                        A_log=torch.log(1 + 15 * u(heads)), D=u(heads), norm_w=0.5 + u(di))
        return Mamba2Decoder(weight, mixer, lambda l: torch.full((d_model,), 1.0 + 0.1 * l), L,
                             d_model, heads, g=g, batch=B, **kw)
    a, b = build(), build(fused=False)
    assert a.fused16 and not a.fused and not b.fused16 and not b.stack
    gen = torch.Generator(device="cuda").manual_seed(7)
    for step in range(5):
        e = torch.randn((B, d_model), generator=gen, device="cuda")
        a.emb.copy_(e)
        b.emb.copy_(e)
        if step == 2:  # the state goes on through replays of a capture
            a.capture()
        xa = (a.replay() if step >= 2 else a.token()).float()
        xb = b.token().float()
        if B >= 9:  # the same sums in the same order
            assert torch.equal(_bits(xa), _bits(xb))
            for k in ("ssm_state", "conv_state"):
                assert torch.equal(_bits(a.arena[k]), _bits(b.arena[k]))
        # each of the 2 L activations handed on may round to the other
        # bfloat16 neighbour: 2^-9 each, at most as independent errors
        assert float((xa - xb).norm() / xb.norm()) <= 2.0 ** -8 * (2 * L) ** 0.5
        for la, lb in zip(a.layers, b.layers):
            assert torch.equal(la["pos"], lb["pos"]) and int(la["pos"]) == (step + 1) % 4
            d = (la["ssm"].float() - lb["ssm"].float()).norm() / lb["ssm"].float().norm()
            assert float(d) <= 2.0 ** -8 * (2 * L) ** 0.5


# (matrices, B, N, K, g): past four 16-row blocks per CU x is copied to LDS;
# one, two and four blocks per wave, K below, at and past a window of columns,
# rounds with one group and with sixteen, ragged rows and matrices; g = 64 at K
# past 2048 on both sides of its own line
@pytest.mark.parametrize("count,B,N,K,g", [(3, 9, 5500, 4160, 64), (2, 16, 8500, 4608, 512),
                                           (1, 12, 16500, 64, 64), (1, 16, 262149, 64, 64),
                                           (1, 10, 524300, 128, 128), (4, 16, 4300, 2048, 256),
                                           (4, 11, 4300, 2304, 128), (1, 16, 1000, 8192, 256),
                                           (6, 9, 5500, 4160, 64), (3, 12, 9000, 4480, 128)])
def test_batched_gemv(count, B, N, K, g):
    print(f"[decode16] gemv {count} x B={B} N={N} K={K} g={g}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    packed = [_packed(gen, N, K, g) for _ in range(count)]
    x = torch.randn((count, B, K), generator=gen, device="cuda").to(torch.bfloat16)
    codes = torch.stack([p[0] for p in packed])
    s16 = torch.stack([p[1] for p in packed])
    y = torch.full((count, B, N), float("nan"), device="cuda")
    ops.tgemv(x, codes, s16, g, y=y)
    for i in range(count):
        ref = x[i].double() @ packed[i][2].t()
        mag = x[i].double().abs() @ packed[i][2].abs().t()
        # exact products, float32 sums of at most K of them
        assert bool(((y[i].double() - ref).abs() <= (K + 2) * 2.0 ** -24 * mag + 1e-30).all())
