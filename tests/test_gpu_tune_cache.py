"""The autotuner's cache file where one line is not enough for a grid shape: 63 unknowns
an axis are M = 64 in the sine basis (FFT or dense) and M = 62 in the cosine basis (dense
only).  Each plan has its own line, whichever is tuned first, and reads it back; a
line that names no axes holds for both until one that does is found."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def plans(h6):
    kw = dict(precision="mixed")
    return (h6.Plan((63, 63, 20), 1.0 / 64, 3.0 + 0.2j, "DDDDDD", **kw),
            h6.Plan((61, 61, 20), 1.0 / 64, 3.0 + 0.2j, "NNNNDD", **kw))


def fields(line):
    return dict(f.split("=") for f in line.split() if "=" in f)


@pytest.mark.parametrize("first", [0, 1])
def test_bases_of_one_shape_keep_their_own_lines(tmp_path, first):
    from paper_1212_1397_amd import helmholtz6 as h6
    path = str(tmp_path / "tune.txt")
    pair = plans(h6)
    assert pair[0].dims == pair[1].dims
    for p in (pair[first], pair[1 - first]):
        p.autotune(path)
    lines = open(path).read().splitlines()
    assert len(lines) == 2 and all(ln.startswith("h6tune3 ") for ln in lines)
    by = {fields(ln)["axes"]: fields(ln) for ln in lines}
    assert set(by) == {"D64,D64", "N62,N62"}
    assert by["N62,N62"]["xfast"] == by["N62,N62"]["yfast"] == "0"
    x = torch.randn(pair[0].shape, dtype=torch.complex128, device="cuda")
    before = [p.apply_Pinv(x) for p in pair]
    for p, z in zip(plans(h6), before):
        p.autotune(path)                       # read back, nothing timed
        assert torch.equal(p.apply_Pinv(x), z)
        p.close()
    assert open(path).read().splitlines() == lines
    for p in pair:
        p.close()


def test_line_of_the_plans_axes_comes_before_one_without(tmp_path):
    from paper_1212_1397_amd import helmholtz6 as h6
    arch = torch.cuda.get_device_properties(0).gcnArchName
    d, n = plans(h6)
    x = torch.randn(d.shape, dtype=torch.complex128, device="cuda")
    key = f"h6tune3 {arch} {d.dims[0]} {d.dims[1]} {d.dims[2]} {h6.PRECISIONS['mixed']}"
    fft = d.apply_Pinv(x)                      # the untuned default
    path = tmp_path / "old.txt"
    path.write_text(f"{key} tz=8 xfast=0 yfast=0 xlines=4 ylines=16\n")
    d.autotune(str(path))
    dense = d.apply_Pinv(x)
    assert not torch.equal(dense, fft)
    path = tmp_path / "both.txt"
    path.write_text(f"{key} tz=8 xfast=0 yfast=0 xlines=4 ylines=16\n"
                    f"{key} tz=8 xfast=0 yfast=0 xlines=4 ylines=16 axes=N62,N62\n"
                    f"{key} tz=8 xfast=3 yfast=3 xlines=4 ylines=16 axes=D64,D64\n")
    text = path.read_text()
    d.autotune(str(path))
    assert torch.equal(d.apply_Pinv(x), fft)
    n.autotune(str(path))
    assert path.read_text() == text
    d.close()
    n.close()
