"""Which calls with a time-invariant B and / or C are cut along the sequence, seen through the workspace they need: a buffer of the
uncut size off its alignment is refused for its alignment by a call that is not cut and for its size by one that is."""
import ctypes

import pytest

from paper_2312_00752_amd import binding as B

FAKE = 1 << 20


def _params(batch, seqlen, dim, io, flags, dstate=16):
    p = B.FwdParams()
    p.batch, p.dim, p.seqlen, p.dstate, p.io_dtype = batch, dim, seqlen, dstate, io
    for f in ("u", "delta", "Bmat", "Cmat", "A", "out"):
        setattr(p, f, FAKE)
    p.flags = flags | B.SS_SAVE_FOR_BWD
    p.workspace = FAKE + 128
    return p


def _refusal(p, nbytes):
    p.workspace_bytes = nbytes
    return B.lib().ss_scan_fwd(ctypes.byref(p), None)


def _bytes(p, nseg):
    """What a call cut into nseg segments needs (without a gate)."""
    up = lambda n: -(-n // 256) * 256
    rows, slots = p.batch * p.dim, p.dstate * (2 if p.flags & B.SS_COMPLEX_STATE else 1)
    fixed = bool(p.flags & B.SS_B_FIXED) + bool(p.flags & B.SS_C_FIXED)
    state, scalar = up(nseg * rows * 64), up(nseg * rows * 4)
    return up(-(-slots // 16) * -(-p.seqlen // B.SS_CHECKPOINT_STEPS) * rows * 64) + (1 + fixed) * state + 2 * scalar + (2 * state + scalar if nseg > 1 else 0)


def _is_cut(p):
    return {B.SS_ERR_ALIGN: False, B.SS_ERR_WORKSPACE: True}[_refusal(p, _bytes(p, 1))]


def segments(batch, seqlen, dim, io, flags, dstate=16):
    """Into how many segments a call with a time-invariant B or C that keeps what its backward pass needs is cut."""
    p = _params(batch, seqlen, dim, io, flags, dstate)
    for n in range(1, max(2, seqlen // 64 + 2)):
        if _refusal(p, _bytes(p, n)) == B.SS_ERR_ALIGN:
            assert _refusal(p, _bytes(p, n) - 256) == B.SS_ERR_WORKSPACE
            return n
    raise AssertionError("no number of segments fits")


BOTH, ZOH, CPLX = B.SS_B_FIXED | B.SS_C_FIXED, B.SS_EXACT_ZOH_B, B.SS_COMPLEX_STATE


# workgroups of 64 rows: 256 fill the chip once.  The backward kernels of the exact zero-order hold take a compute unit each, the float32
# ones with B and C in registers gain nothing from sharing one, and a grid of one to two per unit shares already
@pytest.mark.parametrize("batch,seqlen,dim,io,flags", [
    (4, 2048, 4096, B.SS_BF16, BOTH | ZOH), (4, 2048, 4096, B.SS_F32, B.SS_B_FIXED | ZOH), (4, 512, 4096, B.SS_BF16, B.SS_C_FIXED | ZOH),
    (4, 2048, 4096, B.SS_F32, BOTH), (3, 2048, 4096, B.SS_F32, BOTH), (4, 512, 4096, B.SS_F32, BOTH), (4, 256, 4096, B.SS_BF16, BOTH),
    (4, 256, 4096, B.SS_BF16, B.SS_B_FIXED), (5, 2048, 4096, B.SS_BF16, BOTH), (6, 2048, 4096, B.SS_F32, B.SS_C_FIXED), (1, 96, 64, B.SS_F32, BOTH), (1, 200, 4096, B.SS_F32, BOTH)])
def test_stays_whole(batch, seqlen, dim, io, flags):
    assert not _is_cut(_params(batch, seqlen, dim, io, flags))


@pytest.mark.parametrize("flags", [B.SS_B_FIXED, B.SS_C_FIXED, BOTH, B.SS_B_FIXED | ZOH, BOTH | ZOH])
@pytest.mark.parametrize("io", [B.SS_F32, B.SS_BF16])
@pytest.mark.parametrize("batch,seqlen,dim", [(1, 2048, 4096), (2, 2047, 4096), (1, 300, 64), (1, 1 << 16, 256)])
def test_few_rows_are_cut(batch, seqlen, dim, io, flags):
    assert _is_cut(_params(batch, seqlen, dim, io, flags))
    if not flags & ZOH:
        assert _is_cut(_params(batch, seqlen, dim, io, flags | CPLX, 8))


def test_the_size_that_is_asked_for_serves_every_call():
    """A query names neither the rule for B-bar nor, with its defaults, the io dtype."""
    for batch in (1, 2, 3, 4, 5, 6, 9, 10, 12):
        for seqlen in (96, 256, 511, 512, 2047, 2048, 8192):
            for flags in (B.SS_B_FIXED, B.SS_C_FIXED, BOTH):
                need = B.ss_workspace_bytes(batch, 4096, seqlen, 16, has_z=False, b_fixed=bool(flags & B.SS_B_FIXED), c_fixed=bool(flags & B.SS_C_FIXED))
                for io in (B.SS_F32, B.SS_BF16):
                    for zoh in (0, ZOH):
                        assert _refusal(_params(batch, seqlen, 4096, io, flags | zoh), need) == B.SS_ERR_ALIGN, (batch, seqlen, flags, io, zoh)
