"""Float32 rows of whole slices: a thread's slice is four steps from each half of a 32-step chunk, and the results of an odd
chunk (forward) or of an even block (backward) take the waiting ones of its neighbour along where tensors are large.  Lengths that end in the first and
in the second half of an even and of an odd chunk, in an even and in an odd block; whole and in segments; the patterns around
every output, NaN around every input (as for rows of any length).  Unsplit grids of at most 256 row groups and 16 states run the whole-row
forward kernel; larger ones and more states the four-wave kernel."""
import pytest

from tests import test_gpu_ragged

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    (1, 8, 64, 16, False), (2, 16, 65, 4, False), (1, 24, 3, 16, True), (1, 40, 70, 16, False), (2, 56, 66, 1, False), (1, 64, 130, 16, False),
    (1, 72, 64, 20, False), (1, 88, 40, 7, True), (3, 104, 33, 16, False),
    # split: the last segment ends in either half of an even and of an odd chunk
    (1, 520, 64, 16, False), (1, 536, 100, 16, True), (2, 560, 70, 5, False), (1, 2072, 64, 16, False), (1, 2096, 30, 18, False)])
def test_float_rows_of_whole_slices(batch, seqlen, dim, dstate, zoh):
    test_gpu_ragged.test_ragged_rows("f32", batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    (257, 8, 2, 16, False), (260, 16, 1, 3, False), (257, 24, 3, 16, True), (130, 40, 66, 7, False), (257, 56, 2, 1, False), (257, 64, 1, 8, True),
    (257, 72, 2, 4, False), (129, 88, 70, 16, False), (257, 104, 1, 6, True), (257, 120, 2, 12, False)])
def test_float_rows_of_whole_slices_beyond_whole_rows(batch, seqlen, dim, dstate, zoh):
    """More than 256 row groups, unsplit: the four-wave forward kernel with one, two and four slots per lane and the exact hold."""
    test_gpu_ragged.test_ragged_rows("f32", batch, seqlen, dim, dstate, zoh)


@pytest.mark.parametrize("batch,seqlen,dim,dstate,zoh", [
    # from 32 MB a tensor off whole lines: lengths off and on eight steps, an even and an odd last chunk; rows 4 MB apart
    (66, 529, 250, 16, False), (66, 545, 250, 3, False), (66, 531, 250, 7, True), (66, 536, 250, 4, False), (66, 552, 250, 16, False),
    (66, 552, 250, 5, True), (1, 1 << 20, 9, 2, False),
    # from 16 MB the backward pass alone
    (66, 320, 250, 7, False), (66, 288, 250, 16, True), (66, 299, 250, 12, False),
    # and in segments
    (1, 131083, 65, 4, False), (2, 65592, 70, 18, False)])
def test_float_results_that_wait(batch, seqlen, dim, dstate, zoh):
    """Tensors that leave the caches: results of neighbouring chunks and blocks are written together (those of smaller ones at once)."""
    test_gpu_ragged.test_ragged_rows("f32", batch, seqlen, dim, dstate, zoh)
