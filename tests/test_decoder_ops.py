"""The decoder layer's elementwise kernels against float64.

Every result passes a few fp32 operations and one rounding to bf16 (8 significant bits, nearest even: at
most 2^-8 of the value), so the bar is 1.02 * 2^-8 |ref| plus 2^-20 of the operands' magnitude for the
fp32 rounding (cancellation in RoPE's two products).  The residual sum is one fp32
addition and compared exactly; rows that only move (v heads) bit for bit.
"""
import ctypes

import pytest
import torch

import paper_2609_39334_amd as tkv


def _close(got, ref, scale):
    assert torch.all((got.double() - ref).abs() <= 1.02 * 2.0 ** -8 * ref.abs() + 2.0 ** -20 * scale)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("rows,hidden", [(1, 8), (3, 1024), (5, 3584), (2, 8192), (2, 8200), (7, 1001), (4, 12), (2, 16384),
                                         (2, 16392), (3, 4095), (3, 4097), (1, 30001)])
@pytest.mark.parametrize("with_delta", [False, True])
def test_add_rmsnorm(rows, hidden, with_delta):
    # rows held in registers (multiples of 8 up to 8,192, and to 16,384) and read again (longer, odd)
    g = _gen(hidden)
    x, w = _randn(g, rows, hidden) * 3, torch.rand(hidden, generator=g, device="cuda") + 0.5
    delta = _randn(g, rows, hidden).bfloat16() if with_delta else None
    want = x + delta.float() if with_delta else x.clone()
    h = tkv.tkv_add_rmsnorm(x, delta, w, 1e-6)
    assert torch.equal(x, want)
    ref = want.double() * torch.rsqrt((want.double() ** 2).mean(-1, keepdim=True) + 1e-6) * w.double()
    _close(h, ref, ref.abs())


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (28, 4, 128), (1, 1, 128), (15, 5, 64)])
@pytest.mark.parametrize("n", [1, 33])
def test_rope_append(hq, hkv, d, n):
    g = _gen(hq * n)
    nb = n + 3
    qkv = _randn(g, n, (hq + 2 * hkv) * d).bfloat16()
    ang = torch.rand((n, d // 2), generator=g, device="cuda") * 1000
    cos, sin = torch.cos(ang), torch.sin(ang)
    dst = torch.randperm(nb * 16, generator=g, device="cuda")[:n].to(torch.int32)
    if n > 4:
        dst[1], dst[2], dst[3] = -1, nb * 16, -7          # no slot, outside the pool: not written
    k, v = (_randn(g, nb, hkv, 16, d).bfloat16() for _ in "kv")
    k0, v0 = k.clone(), v.clone()
    q = tkv.tkv_rope_append(qkv, cos, sin, dst, hq, k, v)
    heads = qkv.view(n, hq + 2 * hkv, d)
    a, b = heads[:, :hq + hkv, :d // 2].double(), heads[:, :hq + hkv, d // 2:].double()
    c, s = cos.double()[:, None], sin.double()[:, None]
    ref = torch.cat((a * c - b * s, b * c + a * s), -1)
    scale = torch.cat((a.abs() + b.abs(),) * 2, -1)
    _close(q, ref[:, :hq], scale[:, :hq])
    written = torch.zeros((nb, 16), dtype=torch.bool, device="cuda")
    for t, slot in enumerate(dst.tolist()):
        if 0 <= slot < nb * 16:
            written[slot // 16, slot % 16] = True
            _close(k[slot // 16, :, slot % 16], ref[t, hq:], scale[t, hq:])
            assert torch.equal(v[slot // 16, :, slot % 16], heads[t, hq + hkv:])
    keep = ~written[:, None, :, None].expand_as(k)
    assert torch.equal(k[keep], k0[keep]) and torch.equal(v[keep], v0[keep])


@pytest.mark.gpu
@pytest.mark.parametrize("rows,inter", [(1, 8), (3, 18944), (5, 1001), (257, 4), (2, 8 * 255)])
def test_swiglu(rows, inter):
    g = _gen(inter)
    gu = (_randn(g, rows, 2 * inter) * 6).bfloat16()
    gu[0, 0], gu[0, 1 % inter], gu[-1, inter - 1] = -300.0, 300.0, 0.0   # SiLU's ends: 0, the value, 0
    out = tkv.tkv_swiglu(gu)
    gate, up = gu[:, :inter].double(), gu[:, inter:].double()
    ref = gate / (1 + torch.exp(-gate)) * up
    _close(out, ref, ref.abs() + 2.0 ** -100)


@pytest.mark.gpu
@pytest.mark.parametrize("inter", [256, 255])
def test_swiglu_of_very_negative_gates(inter):
    # SiLU keeps its relative precision down to where exp(-gate) passes the fp32 range (88.7), here scaled up
    # by the other operand
    gate = torch.linspace(-88.5, -60.0, inter, device="cuda").bfloat16()
    up = torch.full((inter,), 2.0 ** 100, device="cuda").bfloat16()
    out = tkv.tkv_swiglu(torch.cat((gate, up))[None])
    g = gate.double()
    ref = g / (1 + torch.exp(-g)) * up.double()
    assert torch.all(ref < 0)
    _close(out[0], ref, ref.abs())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [512, 511])
def test_infinities_and_nan_as_the_tensor_operations_give_them(n):
    # a row each with +inf, -inf and NaN among its values, and one without; both forms of the row kernels
    inf, nan = float("inf"), float("nan")
    g = _gen(n)
    odd = [(0, inf), (1, -inf), (2, nan)]

    def same(got, ref):
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())
        ok = ref.isfinite()
        _close(got[ok], ref[ok].double(), ref[ok].double().abs() + 2.0 ** -100)
        assert torch.equal(got[ref.isinf()].sign(), ref[ref.isinf()].sign())

    gu = (_randn(g, 4, 2 * n) * 3).bfloat16()
    for r, x in odd:
        gu[r, 5], gu[r, n + 7], gu[r, 9], gu[r, n + 9] = x, x, x, 0.0
    gf = gu.float()
    same(tkv.tkv_swiglu(gu), (torch.nn.functional.silu(gf[:, :n]) * gf[:, n:]).bfloat16())

    w = torch.rand(n, generator=g, device="cuda") + 0.5
    for with_delta in (False, True):
        x = _randn(g, 4, n)
        delta = _randn(g, 4, n).bfloat16() if with_delta else None
        for r, bad in odd:
            (delta if with_delta else x)[r, 5] = bad
        want = x + delta.float() if with_delta else x.clone()
        h = tkv.tkv_add_rmsnorm(x, delta, w, 1e-6)
        assert torch.equal(x.isnan(), want.isnan()) and torch.equal(x.nan_to_num(), want.nan_to_num())
        same(h, (want * torch.rsqrt((want * want).mean(-1, keepdim=True) + 1e-6) * w).bfloat16())

    d, hq, hkv = 64, 2, 1
    qkv = _randn(g, 4, (hq + 2 * hkv) * d).bfloat16()
    for r, bad in odd:
        qkv[r, 3], qkv[r, 2 * d + 40], qkv[r, 3 * d + 1] = bad, bad, bad
    ang = torch.rand((4, d // 2), generator=g, device="cuda") * 100
    cos, sin = torch.cos(ang), torch.sin(ang)
    k, v = (torch.zeros((4, hkv, 16, d), device="cuda").bfloat16() for _ in "kv")
    dst = torch.arange(4, device="cuda", dtype=torch.int32) * 16
    q = tkv.tkv_rope_append(qkv, cos, sin, dst, hq, k, v)
    heads = qkv.view(4, -1, d).float()
    a, b = heads[:, :hq + hkv, :d // 2], heads[:, :hq + hkv, d // 2:]
    c, s = cos[:, None], sin[:, None]
    rot = torch.cat((a * c - b * s, b * c + a * s), -1).bfloat16()
    for got, ref in ((q, rot[:, :hq]), (k[:, :, 0], rot[:, hq:]), (v[:, :, 0], heads[:, hq + hkv:].bfloat16())):
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())


def test_bad_arguments_are_refused():
    # refused before any device access (no GPU needed)
    L = tkv.lib()
    one = 16
    assert L.tkv_add_rmsnorm(1, 0, 1e-6, one, None, one, one, None) == tkv.TKV_EINVAL
    assert L.tkv_add_rmsnorm(-1, 8, 1e-6, one, None, one, one, None) == tkv.TKV_EINVAL
    assert L.tkv_add_rmsnorm(1, 8, 1e-6, None, None, one, one, None) == tkv.TKV_EINVAL
    assert L.tkv_add_rmsnorm(0, 8, 1e-6, None, None, None, None, None) == tkv.TKV_OK
    assert L.tkv_swiglu(1, 0, one, one, None) == tkv.TKV_EINVAL and L.tkv_swiglu(1, 8, None, one, None) == tkv.TKV_EINVAL

    def rope(sh, n=1, q=one):
        return L.tkv_rope_append(ctypes.byref(tkv.tkv_shape(*sh)), n, one, one, one, one, q, one, one, None)

    for sh in ((8, 2, 96, 16, 4), (8, 2, 64, 32, 4), (0, 2, 64, 16, 4), (8, 0, 64, 16, 4), (8, 2, 64, 16, 1 << 28)):
        assert rope(sh) == tkv.TKV_EINVAL, sh
    assert rope((8, 2, 64, 16, 4), n=-1) == tkv.TKV_EINVAL and rope((8, 2, 64, 16, 4), q=None) == tkv.TKV_EINVAL
    assert rope((8, 2, 64, 16, 4), q=one + 8) == tkv.TKV_EINVAL and "aligned" in tkv.tkv_last_error()
    assert rope((8, 2, 64, 16, 4), n=0) == tkv.TKV_OK
