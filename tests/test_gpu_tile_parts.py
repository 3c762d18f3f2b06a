"""The training products where output tiles are cut along the contraction and
their parts meet in a scratch buffer: dX (both forms, float32 and bfloat16,
from a bfloat16 or a float32 gradient) and dW (stored and accumulated), on
shapes with fewer 256 x 256 tiles than compute units, ragged edges, one part,
the most parts, and a remainder after whole rounds; against float64."""

import pytest

torch = pytest.importorskip("torch")

from paper_2606_18114_amd import ops  # noqa: E402

pytestmark = pytest.mark.gpu

# (M, N, K, g): tokens, out features, in features
SHAPES = [(1, 256, 64, 32), (16, 256, 512, 128), (300, 1032, 768, 64), (257, 4104, 320, 64),
          (1000, 3352, 768, 256), (2050, 2056, 512, 512), (129, 8512, 2048, 128),
          (4352, 4096, 1024, 128)]


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _operands(M, N, K, g, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    dy = torch.randn((M, N), generator=gen, device="cuda") * 0.01
    codes, s, _, _ = ops.ternarize_pack(w, g, 1e-5)
    tau = (s + 1e-5).repeat_interleave(g, dim=1)
    what = (torch.sign(w) * (w.abs() > 0.5 * tau)).double() * s.double().repeat_interleave(g, 1)
    return x, dy, codes, s, what


def _rel(a, ref):
    return float((a.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("M,N,K,g", SHAPES)
@pytest.mark.parametrize("precision", ["f16", "exact"])
def test_input_grad(M, N, K, g, precision):
    print(f"[parts] dX {precision} M={M} N={N} K={K} g={g}", flush=True)
    _, dy, codes, s, what = _operands(M, N, K, g)
    dyb = dy.to(torch.bfloat16)
    ref = dyb.double() @ what
    dX = ops.tgemm_bwd_dx(dyb, codes, s, g, precision=precision)
    # float16 keeps 11 bits of a scale (2^-12 rms of a rounding), the two-pass
    # form 16 bits; the float32 sums add less
    assert _rel(dX, ref) <= (2.0 ** -11 if precision == "f16" else 2.0 ** -15)
    assert torch.equal(dX, ops.tgemm_bwd_dx(dyb, codes, s, g, precision=precision))
    for gy in (dyb, dy):  # a bfloat16 result is the float32 one rounded once
        dX16, gy16 = ops.layer_input_grad(gy, codes, s, g, precision=precision)
        assert dX16.dtype == torch.bfloat16 and torch.equal(dX16, dX.to(torch.bfloat16))
        assert torch.equal(gy16, dyb)


@pytest.mark.parametrize("M,N,K,g", SHAPES)
def test_weight_grad(M, N, K, g):
    print(f"[parts] dW M={M} N={N} K={K}", flush=True)
    x, dy, _, _, _ = _operands(M, N, K, g)
    dyb = dy.to(torch.bfloat16)
    ref = dyb.double().t() @ x.double()
    dW = ops.tgemm_bwd_dw_ste(dyb, x)
    # float32 sums of exact products: random rounding of M terms
    tol = 2.0 ** -23 * max(M, 16) ** 0.5
    assert _rel(dW, ref) <= tol
    assert torch.equal(dW, ops.tgemm_bwd_dw_ste(dyb, x))
    acc = torch.ones_like(dW)
    ops.tgemm_bwd_dw_ste(dyb, x, acc, accumulate=True)
    assert _rel(acc, ref + 1) <= tol + 2.0 ** -24


# More than 256 tiles of dX (dW) and a remainder: without scratch the leftover
# tiles are cleared and their parts add up by atomics; ragged and whole edges,
# parts of few stages
@pytest.mark.parametrize("M,N,K,g", [(4300, 520, 4160, 64), (4352, 1032, 4096, 256),
                                     (4170, 200, 4224, 128)])
@pytest.mark.parametrize("precision", ["f16", "exact"])
def test_input_grad_without_scratch(M, N, K, g, precision):
    print(f"[parts] dX no scratch {precision} M={M} N={N} K={K} g={g}", flush=True)
    _, dy, codes, s, what = _operands(M, N, K, g)
    dyb = dy.to(torch.bfloat16)
    dX = torch.full((M, K), float("nan"), device="cuda")
    head = (dyb.data_ptr(), codes.data_ptr(), s.data_ptr(), M, N, K, g, dX.data_ptr())
    stream = torch.cuda.current_stream().cuda_stream
    if precision == "f16":
        ws = torch.empty(ops.dx_f16_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
        st = ops.lib().tm_tgemm_bwd_dx_f16(*head, ws.data_ptr(), ws.numel(), stream)
    else:
        st = ops.lib().tm_tgemm_bwd_dx(*head, stream)
    assert st == 0
    assert _rel(dX, dyb.double() @ what) <= (2.0 ** -11 if precision == "f16" else 2.0 ** -15)
    # the same products in another order
    with_scratch = ops.tgemm_bwd_dx(dyb, codes, s, g, precision=precision)
    assert _rel(dX, with_scratch.double()) <= 2.0 ** -23 * N ** 0.5


@pytest.mark.parametrize("M,N,K", [(300, 4104, 4160), (1000, 4352, 4096), (65, 4360, 4224)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_weight_grad_without_scratch(M, N, K, accumulate):
    print(f"[parts] dW no scratch M={M} N={N} K={K} accumulate={accumulate}", flush=True)
    x, dy, _, _, _ = _operands(M, N, K, 64)
    dyb = dy.to(torch.bfloat16)
    dW = torch.full((N, K), 1.0 if accumulate else float("nan"), device="cuda")
    st = ops.lib().tm_tgemm_bwd_dw_ste(dyb.data_ptr(), x.data_ptr(), M, N, K, dW.data_ptr(),
                                       accumulate, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    ref = dyb.double().t() @ x.double() + accumulate
    # float32 sums of exact products; a sum that starts at 1 rounds to its step
    # at each of at most 256 parts
    tol = 2.0 ** -23 * max(M, 16) ** 0.5
    assert _rel(dW, ref) <= tol + accumulate * 2.0 ** -20


@pytest.mark.parametrize("M,N,K,g", [(2050, 2056, 512, 512), (300, 8512, 2048, 128)])
def test_no_memory_for_scratch(M, N, K, g, monkeypatch):
    """Where the scratch cannot be allocated the calls do without it."""
    print(f"[parts] no memory for scratch M={M} N={N} K={K} g={g}", flush=True)
    x, dy, codes, s, what = _operands(M, N, K, g)
    dyb = dy.to(torch.bfloat16)
    L, none = ops.lib(), []
    sizes = {L.tm_tgemm_fwd_scratch(M, N, K, g, 0), L.tm_tgemm_fwd_scratch(M, N, K, g, 1),
             L.tm_tgemm_bwd_dx_slots(M, N, K, 0), L.tm_tgemm_bwd_dx_slots(M, N, K, 1),
             L.tm_tgemm_bwd_dw_slots(M, N, K)} - {0, ops.dx_f16_workspace_bytes(M, N)}

    def calls():
        return [ops.tgemm_fwd(x, codes, s, g), ops.tgemm_fwd(x, codes, s, g,
                                                             out_dtype=torch.bfloat16),
                ops.tgemm_bwd_dx(dyb, codes, s, g), ops.tgemm_bwd_dx(dyb, codes, s, g,
                                                                     precision="exact"),
                ops.layer_input_grad(dy, codes, s, g)[0], ops.layer_input_grad(dyb, codes, s, g)[0],
                ops.layer_input_grad(dyb, codes, s, g, precision="exact")[0],
                ops.tgemm_bwd_dw_ste(dyb, x)]
    want = calls()
    real = torch.empty

    def empty(*a, **kw):
        if kw.get("dtype") == torch.uint8 and a[0] in sizes:
            none.append(a[0])
            raise torch.OutOfMemoryError("none left")
        return real(*a, **kw)
    monkeypatch.setattr(torch, "empty", empty)
    got = calls()
    monkeypatch.undo()
    assert len(none) >= 5
    for a, b in zip(got, want):
        assert a.dtype == b.dtype
        # another order of the float32 sums; in bfloat16 a rounding may fall
        # the other way
        assert _rel(a, b.double()) <= (2.0 ** -9 if a.dtype == torch.bfloat16
                                       else 2.0 ** -23 * max(M, N, K) ** 0.5)


# (tokens, out features, in features, g): the forward's three tile shapes, cut
# and whole, with code stages of one and four operand stages
FORWARD = [(1, 64, 64, 32), (16, 256, 512, 128), (70, 1000, 320, 64), (300, 8512, 2048, 128),
           (500, 2048, 4096, 128), (1000, 3351, 768, 64), (129, 513, 1536, 512),
           (2048, 8512, 2048, 128), (4096, 2048, 1024, 256), (3000, 4000, 1024, 32),
           (33, 8512, 4096, 512), (2100, 4097, 192, 64),
           # leftover tiles after whole rounds: 64 and 48 (two parts in Y), 32
           (8192, 8512, 2048, 128), (6000, 8511, 1024, 32), (4096, 8512, 1408, 64),
           (4096, 2048, 4096, 32),
           # K no multiple of 256 (stage times of its own in the plan): two parts in Y
           # (slots in bfloat16), slots of small tiles, whole tiles of two shapes
           (8192, 6344, 1408, 128), (40, 2056, 4160, 64), (2600, 2000, 1344, 64),
           (414, 5377, 2112, 64), (2459, 3875, 832, 32), (1822, 2475, 832, 32),
           (700, 300, 1088, 32)]


@pytest.mark.parametrize("M,N,K,g", FORWARD)
def test_forward(M, N, K, g):
    print(f"[parts] fwd M={M} N={N} K={K} g={g}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    w[:, :g] *= (torch.arange(N, device="cuda") % 3 != 0)[:, None]  # groups of zeros
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    codes, s, _, _ = ops.ternarize_pack(w, g, 1e-5)
    tau = (s + 1e-5).repeat_interleave(g, dim=1)
    what = (torch.sign(w) * (w.abs() > 0.5 * tau)).double() * s.double().repeat_interleave(g, 1)
    ref = x.double() @ what.t()
    Y = torch.full((M, N), float("nan"), device="cuda")
    ops.tgemm_fwd(x, codes, s, g, Y=Y)
    # float32 sums of exact products, a rescale (two roundings) per group
    assert _rel(Y, ref) <= 2.0 ** -24 * (2 * K // g + K ** 0.5)
    assert torch.equal(Y, ops.tgemm_fwd(x, codes, s, g))
    Yb = ops.tgemm_fwd(x, codes, s, g, out_dtype=torch.bfloat16)
    # (a float32 tile may be cut where the bfloat16 one is whole)
    assert _rel(Yb, Y.to(torch.bfloat16).double()) <= 2.0 ** -9
    assert torch.equal(Yb, ops.tgemm_fwd(x, codes, s, g, out_dtype=torch.bfloat16))


def test_float32_gradient_rounding():
    """Ties, infinities, NaN and subnormals round as torch's cast does."""
    _, dy, codes, s, _ = _operands(16, 256, 512, 128)
    bits = torch.arange(16 * 256, device="cuda", dtype=torch.int64) * 1048583 % (1 << 32)
    dy = bits.to(torch.int32).view(torch.float32).reshape(16, 256).contiguous()
    dy[0, :4] = torch.tensor([float("inf"), float("-inf"), float("nan"), 1e-40], device="cuda")
    _, got = ops.layer_input_grad(dy, codes, s, 128)
    ref = dy.to(torch.bfloat16)
    nan = ref.isnan()
    assert torch.equal(got.isnan(), nan)
    assert torch.equal(got[~nan].view(torch.int16), ref[~nan].view(torch.int16))


# whole tiles (more than 256 of them) and cut ones, edges inside a block of 8
# rows x 32 columns and at its end
@pytest.mark.parametrize("M,N,K", [(3, 7648, 2368), (29, 9864, 2560), (90, 6456, 4160),
                                   (129, 8512, 2048), (40, 264, 64)])
def test_weight_grad_accumulates_in_one_sum(M, N, K):
    print(f"[parts] dW accumulate M={M} N={N} K={K}", flush=True)
    x, dy, _, _, _ = _operands(M, N, K, 64)
    dyb = dy.to(torch.bfloat16)
    old = torch.randn((N, K), device="cuda")
    acc = old.clone()
    ops.tgemm_bwd_dw_ste(dyb, x, acc, accumulate=True)
    assert torch.equal(acc, old + ops.tgemm_bwd_dw_ste(dyb, x))


# the forward's parts meet through tickets, and in slots; dX's and dW's in slots
@pytest.mark.parametrize("M,N,K,g", [(4352, 4096, 512, 128), (2048, 8512, 2048, 128)])
def test_scratch_in_graphs_and_on_two_streams(M, N, K, g):
    """The calls' scratch under capture (replayed with eager work between) and
    in use on two streams at once: the bits of the eager run."""
    print(f"[parts] scratch in graphs and streams M={M} N={N} K={K} g={g}", flush=True)
    x, dy, codes, s, _ = _operands(M, N, K, g)
    dyb = dy.to(torch.bfloat16)

    def outputs():
        return [torch.full((M, N), float("nan"), device="cuda"),
                torch.full((M, K), float("nan"), device="cuda"),
                torch.full((N, K), float("nan"), device="cuda")]

    def run(Y, dX, dW):
        ops.tgemm_fwd(x, codes, s, g, Y=Y)
        ops.tgemm_bwd_dx(dyb, codes, s, g, dX=dX)
        ops.tgemm_bwd_dw_ste(dyb, x, dW)
        return Y, dX, dW
    want = run(*outputs())
    torch.cuda.synchronize()
    sides = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [outputs(), outputs()]
    torch.cuda.synchronize()
    for _ in range(3):
        for side, out in zip(sides, outs):
            with torch.cuda.stream(side):
                run(*out)
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(a, b) for a, b in zip(out, want))
    graph = torch.cuda.CUDAGraph()
    out = outs[0]
    with torch.cuda.graph(graph):
        run(*out)
    for rep in range(3):
        for t in out:
            t.fill_(float("nan"))
        run(*outs[1])  # eager work in scratch of its own
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want)), f"replay {rep}"
