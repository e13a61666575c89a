"""The V codes of the E2M3 container come from a kernel of their own, one wave
per 32 tokens of every channel; those of the nibble container from the general
one.  Codes, scales and means of both are the same integers and the same bits,
and the oracle's, at token counts around its 32-, 64- and 128-token pieces, in
both input types, and for values that are not finite (compared with each other
there: the oracle is for finite values).
"""
import numpy as np
import pytest

from layouts import unpack_v, unpack_v_e2m3
from test_gpu_int4 import FORMATS, _cfg, _ra, _torch

pytestmark = pytest.mark.gpu


def _quantize(torch, ra, x, vg, smooth, fmt, fp16):
    BH, N = x.shape[:2]
    p = ra.make_params(1, BH, (1, 1, N), v_group=vg, kv_block=64, smooth=2 * smooth,
                       in_dtype=ra.FP16 if fp16 else ra.BF16, code_format=FORMATS[fmt])
    b = ra.alloc_int4(p)
    b["v_codes"].fill_(0xFF)
    ra.quantize_v(p, x, b["v_codes"], b["v_scale"], b["mu_v"] if smooth else None, ra.workspace(p, ra.PATH_INT4))
    torch.cuda.synchronize()
    npad = -(-N // 128) * 128
    codes = (unpack_v_e2m3 if fmt == "e2m3" else unpack_v)(b["v_codes"].cpu().numpy(), BH, npad, npad)
    return codes, b["v_scale"].cpu().numpy(), b["mu_v"].cpu().numpy()


@pytest.mark.parametrize("vg", [64, 128, 192, 1 << 21])
@pytest.mark.parametrize("n", [1, 31, 63, 64, 65, 127, 128, 129, 191, 193, 320])
def test_v_records(ora, n, vg):
    torch, ra = _torch(), _ra()
    for fp16 in (False, True):
        g = torch.Generator().manual_seed(100 * n + fp16)
        x = torch.randn((2, n, 128), generator=g) + 0.5
        x[0, :, 5] = 0.0
        x[0, :, 6] = 1e-40            # 7 / amax overflows
        xd = x.to(torch.float16 if fp16 else torch.bfloat16)
        bits = xd.view(torch.int16).numpy().view(np.uint16)
        for smooth in (0, 1):
            print(f"[v] n={n} group={vg} fp16={fp16} smooth={smooth}", flush=True)
            a = _quantize(torch, ra, xd.cuda(), vg, smooth, "e2m3", fp16)
            b = _quantize(torch, ra, xd.cuda(), vg, smooth, "int4", fp16)
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
            assert not np.delete(a[0][:, n:], 6, 2).any()
            if smooth:
                assert np.array_equal(a[2], b[2])
            if not fp16:
                cfg = _cfg(ora, 0, 128, 128, vg, 64, smooth=2 * smooth)
                for h in range(2):
                    ref = ora.quantize_v_head(cfg, bits[h])
                    assert np.array_equal(a[0][h, :n], ref["v_codes"])
                    assert np.array_equal(a[1].reshape(2, -1)[h], ref["v_scale"].ravel())
                    assert not smooth or np.array_equal(a[2].reshape(2, -1)[h], ref["mu_v"])


@pytest.mark.parametrize("vg", [64, 128, 256])
def test_v_records_of_values_not_finite(vg):
    torch, ra = _torch(), _ra()
    g = torch.Generator().manual_seed(7)
    x = torch.randn((1, 200, 128), generator=g)
    x[0, 3, 0], x[0, 70, 1], x[0, 199, 2], x[0, 130, 3] = np.inf, -np.inf, np.nan, 3e38
    x[0, :, 4] = np.nan
    xd = x.to(torch.bfloat16).cuda()
    a, b = (_quantize(torch, ra, xd, vg, 0, fmt, False) for fmt in ("e2m3", "int4"))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1], equal_nan=True)
