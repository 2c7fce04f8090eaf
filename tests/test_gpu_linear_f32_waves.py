"""The low-rank products of fp32 steps whose operands start at multiples of 16 bytes and whose contractions are long: rows, columns and
contractions that end inside a tile or a 32-wide piece, waves that share a contraction unevenly, both operand layouts, and what stays
with the kernels that take any alignment.  Bounds and references are those of the fp32 step's other tests."""
import pytest

torch = pytest.importorskip("torch")

from paper_2401_11504_amd import api  # noqa: E402
from test_gpu_linear_f32 import make, test_linear_step as linear_step  # noqa: E402

W16, W32, D16 = "waves-16x16", "waves-16x32", "direct-16x16"
#        T, d_in, d_out, r, name of the launch of H and dH
CASES = [(1, 2048, 2048, 4, W16), (17, 1100, 2052, 20, W16), (250, 1060, 2100, 36, W16), (64, 4096, 2036, 8, W16),
         (1024, 4096, 4096, 64, W32), (1009, 2052, 2076, 60, W32), (530, 4100, 4124, 56, W32),
         (1024, 4097, 4096, 64, D16), (1024, 4096, 4096, 62, D16), (512, 768, 768, 8, D16),
         # one 16x16 tile a CU and one more; rows that are no whole lines, ranks of 64 and 68
         (512, 1024, 1024, 64, W16), (513, 1024, 1024, 64, W32), (40, 1060, 1028, 64, W16), (40, 1060, 1028, 68, D16), (40, 1056, 1024, 68, W16),
         (1400, 1028, 1036, 64, W32), (2100, 1024, 1024, 16, W16), (2100, 1024, 1024, 20, W32)]


def test_sizes_reach_their_kernel():
    for *sizes, name in CASES:
        assert api.tl_k_linear_step_plan(*sizes)[0] == name, sizes


@pytest.mark.gpu
@pytest.mark.parametrize("T,din,dout,r,name", CASES)
def test_step(T, din, dout, r, name):
    linear_step(T, din, dout, r)


@pytest.mark.gpu
def test_operands_off_by_four_bytes():
    """The same values at addresses that are no multiples of 16 bytes: the direct kernel, the same results to within the order of the sums."""
    T, din, dout, r = 200, 2048, 2048, 16
    ins = [t.cuda() for t in make(T, din, dout, r)]

    def run(ops):
        outs = [torch.empty(s, device="cuda") for s in ((T, dout), (T, din), (r, din), (dout, r))]
        api.tl_linear_step(*ops, 1.5, 5e-5, 0.9, 0.999, 1e-8, 0.0, False, *outs, None, None)
        return outs
    odd = []
    for t in ins:
        flat = torch.empty(t.numel() + 1, device="cuda")
        flat[1:] = t.flatten()
        odd.append(flat[1:].view_as(t))
    for a, b in zip(run(ins), run(odd)):
        assert (a - b).norm() <= 1e-5 * a.norm()
