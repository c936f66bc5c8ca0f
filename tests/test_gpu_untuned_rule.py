"""Which transform an untuned plan takes for odd M = n + 1 on axes of at least one slab of
lines: the dense product, and chirp-z for M = 121 .. 129, for M = 241 .. 255 too along y of
grids less than 6 wide.  The result equals the path forced through the autotuner's cache
file bit for bit, and not the other one's."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M,default", [(255, 0), (241, 0), (239, 0), (201, 0), (131, 0), (129, 2), (127, 2), (121, 2),
                                       (119, 0), (97, 0)])
@pytest.mark.parametrize("axis,width", [(0, 4), (1, 6), (1, 5)])
def test_untuned_path_of_whole_slabs(tmp_path, axis, width, M, default):
    from paper_1212_1397_amd import helmholtz6 as h6
    arch = torch.cuda.get_device_properties(0).gcnArchName
    n = [width, width, 4]
    if width == 5 and M >= 241:
        default = 2
    n[axis] = M - 1
    plan = h6.Plan(n, 1.0 / M, 5.0 + 0.1j, "DDDDDD", precision="mixed")
    x = torch.randn(plan.shape, dtype=torch.complex128, device="cuda")
    got = [plan.apply_Pinv(x)]
    for code in (default, 2 - default):
        path = tmp_path / f"tune{code}.txt"
        xf, yf = (code, 0) if axis == 0 else (0, code)
        path.write_text(f"h6tune3 {arch} {plan.dims[0]} {plan.dims[1]} {plan.dims[2]} {h6.PRECISIONS['mixed']} tz=16 "
                        f"xfast={xf} yfast={yf} xlines=4 ylines=16\n")
        plan.autotune(str(path))
        got.append(plan.apply_Pinv(x))
    plan.close()
    assert torch.equal(got[0], got[1])
    assert not torch.equal(got[0], got[2])
