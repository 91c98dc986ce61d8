"""GPU parity of wq_pack where a code's quotient lies next to a half-integer:
weights a few fp32 steps to either side of (m + 1/2) s for every code
boundary m, scales from fp16 subnormals to large, and group counts that leave a
wave's last load partly empty.  Bit-exact against the CPU oracle."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import announce, gpu_pack, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1, 32), (7, 96), (33, 1056), (64, 4096)])
def test_pack_quotients_next_to_half_integers(n, k):
    announce(f"pack half-integers N={n} K={k}")
    rng = np.random.default_rng(n + k)
    groups = n * k // 32
    # Scales over the fp16 range, as exact multiples of 1/7 of the maximum.
    s = np.float16(np.exp2(rng.uniform(-24, 12, size=groups))).astype(np.float64)
    s = np.maximum(s, 2.0 ** -24)
    m = rng.integers(-8, 7, size=(groups, 32)) + 0.5
    w = (m * s[:, None]).astype(np.float32)
    steps = rng.integers(-6, 7, size=w.shape)
    for _ in range(6):
        w = np.where(steps > 0, np.nextafter(w, np.float32(np.inf)), np.where(steps < 0, np.nextafter(w, np.float32(-np.inf)), w))
        steps = steps - np.sign(steps)
    w = np.clip(w, (-7 * s[:, None]).astype(np.float32), (7 * s[:, None]).astype(np.float32))
    w[:, 5] = (7 * s).astype(np.float32)  # the group's maximum sets the scale
    w = np.ascontiguousarray(w.reshape(n, k), dtype=np.float32)
    packed, scales = gpu_pack(to_dev(w))
    rp, rs = oracle.quantize_pack(w)
    assert np.array_equal(to_host(scales, np.uint16), np.asarray(rs).view(np.uint16))
    assert np.array_equal(to_host(packed, np.uint32), rp)
