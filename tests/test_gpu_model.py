"""GPU model-level prefill (PrefillModel over ris_*) vs the oracle stack.

float32 end to end: every kernel accumulates in float32, the GEMMs are
float32 library GEMMs (contraction length K <= 640 here), so a layer's
outputs move by at most about K float32 ulps (640 x 2^-24 ~ 4e-5 relative)
of their inputs, and the final RMSNorm'd states (values of order 1, below 5)
stay within 5e-5 of the float64 oracle.
bfloat16: each layer rounds its activations to bf16 R = 13 times on the way
from its input to its output (the normed input, the QKV projection, the
rotated Q and K, the softmax weights, the attention output, the O
projection, the residual sum, the second norm, the gate/up projection, the
SwiGLU product, the down projection, the second residual sum, the next
norm), each a relative error of at most u = 2^-9.  Independent roundings add
in quadrature, so over L layers the relative error of the final states is of
order sqrt(R L) u; the bars allow twice that: ||got - want|| / ||want|| <=
2 sqrt(R L) u and max |got - want| <= 2 sqrt(R L) u max|want| (0.020 and
about 0.09 for the two-layer stacks here, against measured 0.008 and 0.045),
plus agreement in direction (cosine > 0.999).
"""

import numpy as np
import pytest

from gpu_common import need_gpu, say, torch
from oracle import geometry as o_geo
from oracle import model as o_model
from oracle import rope as o_rope
from synth import MODELS, model_weights, tokens

pytestmark = pytest.mark.gpu

CASES = [
    # model, N, mode, ppm, seeds, block, window, anchor, rope kind, factor
    ("tiny_qwen2", 300, 0, 50_000, 3, 0, 32, 2, o_rope.YARN, 0.0),
    ("tiny_qwen2", 300, 0, 50_000, 3, 0, 32, 2, o_rope.LINEAR, 0.0),
    ("tiny_llama", 257, 1, 100_000, 4, 16, 0, 0, o_rope.YARN, 4.0),
    ("tiny_llama", 200, 0, 10**6, 1, 0, 0, 0, o_rope.PLAIN, 0.0),      # dense causal
]


def run(case, dtype):
    ris = need_gpu()
    from paper_2607_21927_amd.model import PrefillModel
    name, N, mode, ppm, S, block, window, anchor, kind, factor = case
    cfg = MODELS[name]
    W = model_weights(cfg, seed=7)
    ids = tokens(N, cfg.vocab, seed=8)
    spec = o_geo.MaskSpec(mode=mode, density_ppm=ppm, seed=0, n_seeds=S, layer=0, N=N,
                          heads=cfg.kv_heads, block=block, window=window, anchor=anchor)
    want = o_model.prefill(ids, W, cfg, spec, kind, factor)
    model = PrefillModel(cfg, W, "cuda", dtype)
    rd = ris.rope_desc(kind, cfg.rope_base, orig_max_pos=cfg.native_len, factor=factor)
    mask = dict(mode=mode, density_ppm=ppm, n_seeds=S, block=block, window=window, anchor=anchor)
    got = model.prefill(torch.tensor(ids, device="cuda"), mask, rd).float().cpu().numpy()
    return got, want


@pytest.mark.parametrize("case", CASES)
def test_model_prefill_float32_matches_oracle(case):
    say(f"model parity f32 {case}")
    got, want = run(case, torch.float32)
    err = float(np.abs(got - want).max())
    say(f"  max err {err:.3e} (max |want| {np.abs(want).max():.2f})")
    assert err <= 5e-5


@pytest.mark.parametrize("case", CASES[:1] + CASES[2:3])
def test_model_prefill_bf16_close_to_oracle(case):
    got, want = run(case, torch.bfloat16)
    layers = MODELS[case[0]].layers
    bound = 2.0 * np.sqrt(13 * layers) * 2.0**-9
    err = float(np.abs(got - want).max())
    rel = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    cos = float((got * want).sum() / (np.linalg.norm(got) * np.linalg.norm(want)))
    say(f"  bf16 max err {err:.3e} (bar {bound * np.abs(want).max():.3e}), relative L2 {rel:.3e} "
        f"(bar {bound:.3e}), cosine {cos:.6f}")
    assert np.isfinite(got).all() and cos > 0.999
    assert rel <= bound
    assert err <= bound * float(np.abs(want).max())


def test_host_layers_match_closed_forms():
    """ris_rmsnorm (with and without the residual add) and ris_swiglu against
    their definitions, float32 and bf16."""
    ris = need_gpu()
    rng = np.random.default_rng(0)
    for dt, tol in [(torch.float32, 2e-6), (torch.bfloat16, 2e-2)]:
        x = torch.tensor(rng.standard_normal((37, 300)), dtype=dt, device="cuda")
        r = torch.tensor(rng.standard_normal((37, 300)), dtype=dt, device="cuda")
        w = torch.tensor(1 + 0.1 * rng.standard_normal(300), dtype=dt, device="cuda")
        xs, rs, ws = (t.double().cpu().numpy() for t in (x, r, w))
        out = torch.empty_like(x)
        ris.rmsnorm(x, w, out, 1e-6)
        np.testing.assert_allclose(out.double().cpu().numpy(), o_model.rmsnorm(xs, ws, 1e-6), atol=tol * 4)
        res = r.clone()
        ris.rmsnorm(x, w, out, 1e-6, residual=res)
        summed = (x.double() + r.double()).to(dt).double().cpu().numpy()
        assert np.array_equal(res.double().cpu().numpy(), summed)
        np.testing.assert_allclose(out.double().cpu().numpy(), o_model.rmsnorm(summed, ws, 1e-6), atol=tol * 4)
        gu = torch.tensor(rng.standard_normal((37, 2 * 300)), dtype=dt, device="cuda")
        m = torch.empty(37, 300, dtype=dt, device="cuda")
        ris.swiglu(gu, m)
        g = gu.double().cpu().numpy()
        np.testing.assert_allclose(m.double().cpu().numpy(), o_model.silu(g[:, :300]) * g[:, 300:], atol=tol * 4)


# Edges of the vector forms: one vector, a lane's last vector, one wave's
# registers full and one vector more (four waves), four waves' registers full
# and more (element-wise form), rows that are no whole vectors, and buffers off
# a 16-byte boundary; row counts off the workgroup's.
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols,off", [(1, 8, 0), (5, 1000, 0), (3, 1536, 0), (7, 2048, 0), (6, 2056, 0),
                                           (2, 4096, 0), (2, 4100, 0), (3, 8192, 0), (2, 8200, 0), (5, 301, 0),
                                           (4, 1536, 1)])
def test_host_layers_at_vector_edges(dtype, rows, cols, off):
    """ris_rmsnorm (residual kept bit-exact) and ris_swiglu in every form.

    Bars: one rounding at the store (bf16 has 8 significant bits, so half a unit
    in the last place is up to 2^-8 of the value; 2^-24 in float32)
    plus the float32 arithmetic, at most 32 roundings of 2^-24: a lane adds at
    most 32 squares and the root halves a sum's relative error, then six
    exchanges, the root, the division and two products; swiglu has an exp (2
    ulp), a sum, a quotient and a product."""
    ris = need_gpu()
    say(f"host layers {dtype} rows {rows} cols {cols} off {off}")
    gen = torch.Generator().manual_seed(rows * 10007 + cols)
    u = (2.0**-8 if dtype == torch.bfloat16 else 2.0**-24) + 32 * 2.0**-24

    def buf(n, scale=1.0, shift=0.0):
        b = torch.empty(n + off, dtype=dtype, device="cuda")[off:]
        return b.copy_(torch.randn(n, generator=gen) * scale + shift)

    x, r, w = buf(rows * cols).view(rows, cols), buf(rows * cols).view(rows, cols), buf(cols, 0.1, 1.0)
    out = buf(rows * cols).view(rows, cols)
    for res in (None, r.clone() if not off else r):
        summed = x if res is None else (x.float() + res.float()).to(dtype)
        ris.rmsnorm(x, w, out, 1e-6, residual=res)
        d = summed.double()
        want = d * torch.rsqrt(d.square().mean(-1, keepdim=True) + 1e-6) * w.double()
        assert (out.double() - want).abs().le(u * want.abs() + 1e-30).all()
        assert res is None or torch.equal(res, summed)
    gu, m = buf(rows * 2 * cols, 4.0).view(rows, 2 * cols), buf(rows * cols).view(rows, cols)
    gu[0, 0], gu[-1, cols - 1] = -200.0, 90.0                 # exp overflows; exp vanishes
    ris.swiglu(gu, m)
    g = gu.double()
    want = torch.nn.functional.silu(g[:, :cols]) * g[:, cols:]
    assert (m.double() - want).abs().le(u * want.abs() + 1e-30).all()


def test_swiglu_streamed():
    """Tensors of more than twice the last-level cache, read and written past
    the caches; a last workgroup of a few vectors.  Bar as above."""
    ris = need_gpu()
    rows, inter = 10001, 9000
    say("swiglu streamed")
    gen = torch.Generator(device="cuda").manual_seed(1)
    gu = torch.empty(rows, 2 * inter, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    m = torch.empty(rows, inter, dtype=torch.bfloat16, device="cuda")
    assert 2 * (gu.numel() + m.numel()) > 512 << 20
    ris.swiglu(gu, m)
    u = 2.0**-8 + 32 * 2.0**-24
    for r in range(0, rows, 1000):
        g = gu[r:r + 1000].double()
        want = torch.nn.functional.silu(g[:, :inter]) * g[:, inter:]
        assert (m[r:r + 1000].double() - want).abs().le(u * want.abs() + 1e-30).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(9, 8), (3, 256), (5, 1000), (33, 1536), (8, 2048), (7, 2056), (2, 4096), (3, 8192),
                                       (4097, 520), (4100, 1096), (4101, 1544), (4099, 2048)])
def test_host_layers_do_not_depend_on_alignment(dtype, rows, cols):
    """The forms that read 16-byte vectors, whole or off a 16-byte boundary,
    give the bits of the element-by-element form (buffers one element further
    on): the same sums in the same order, the same roundings, subnormal values
    and sums among them."""
    ris = need_gpu()
    say(f"alignment {dtype} rows {rows} cols {cols}")
    gen = torch.Generator().manual_seed(rows * 10007 + cols)

    def both(n, scale=1.0, shift=0.0):
        v = (torch.randn(n, generator=gen) * scale + shift).to(dtype).cuda()
        return v, torch.empty(n + 1, dtype=dtype, device="cuda")[1:].copy_(v)

    def same(pair):
        a, b = (t.view(torch.int16 if dtype == torch.bfloat16 else torch.int32) for t in pair)
        return torch.equal(a, b)

    x, r, w, gu = both(rows * cols), both(rows * cols), both(cols, 0.1, 1.0), both(rows * 2 * cols, 4.0)
    for t in x + r:
        t[:cols] *= 1e-39
    out, m = both(rows * cols), both(rows * cols)
    for i in (0, 1):
        ris.rmsnorm(x[i].view(rows, cols), w[i], out[i].view(rows, cols), 1e-6)
        ris.swiglu(gu[i].view(rows, 2 * cols), m[i].view(rows, cols))
    assert same(out), "rmsnorm"
    assert same(m), "swiglu"
    for i in (0, 1):
        ris.rmsnorm(x[i].view(rows, cols), w[i], out[i].view(rows, cols), 1e-6, residual=r[i].view(rows, cols))
    assert same(r) and same(out), "rmsnorm with a residual"
