"""What paro_permute_quantize_qkv_keep refuses before it launches anything."""
import ctypes

import numpy as np


def test_refused_arguments():
    from paper_2506_16054_amd import binding as pb

    L = pb.lib()
    s = pb.make_shape(1, 2, 64, 2, 4, 8, 0, 32)
    ok, bad = np.array([0, 5], np.uint8), np.array([0, 6], np.uint8)

    def call(bits=(8, 8), perm=ok, dt=pb.PARO_F32, **at):
        p = dict(q=0x1000, k=0x2000, v=0x3000, qp=0x4000, kp=0x5000, vp=0x6000, qc=0x7000, sq=0x10, kc=0x8000, sk=0x20, vc=0x9000, sv=0x30)
        p.update(at)
        return L.paro_permute_quantize_qkv_keep(ctypes.byref(s), dt, *bits, None if perm is None else perm.ctypes.data, *p.values(), None)

    for bits in ((8, 16), (16, 8), (3, 8)):
        assert call(bits) == pb.PARO_EINVAL
    assert call(perm=None) == pb.PARO_EINVAL and call(perm=bad) == pb.PARO_EINVAL and call(dt=7) == pb.PARO_EINVAL
    for name in ("q", "k", "v", "qp", "kp", "vp", "qc", "sq", "kc", "sk", "vc", "sv"):
        assert call(**{name: None}) == pb.PARO_EINVAL, name
    for name in ("q", "vp", "kc"):
        assert call(**{name: 0xA004}) == pb.PARO_EINVAL, name  # alignment
    for name, other in (("qp", 0x1000), ("vp", 0x2000), ("kp", 0x4000), ("kp", 0x7000), ("vc", 0x6000), ("qc", 0x3000)):
        assert call(**{name: other}) == pb.PARO_EINVAL, name
        assert b"alias" in L.paro_last_error()
