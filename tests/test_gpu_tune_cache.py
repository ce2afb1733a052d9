"""The autotuner's cache file names the variant that was timed: an entry stays
with its kernel whatever number the kernel has, and an entry of the form that
earlier builds wrote (a number) is timed anew, once, instead of selecting the
kernel that has the number now."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2107_03747_amd import gen, tgf          # noqa: E402

DIMS = (4, 4, 4, 8)


def tuned(nc, path):
    f = tgf.Flow([DIMS], "f64", nc=nc)
    f.load(0, gen.identity(DIMS, device="cuda") if nc is None else gen.identity_n(DIMS, nc, device="cuda"))
    return f.autotune(str(path))


def variants(path):
    """The variant lines of a cache file (not the work-group shapes)."""
    return [line.split() for line in path.read_text().splitlines() if "/blk/" not in line]


@pytest.mark.parametrize("nc", [None, 4, 5, 8])
def test_entries_name_the_variant(tmp_path, nc):
    p = tmp_path / "tune.txt"
    v = tuned(nc, p)
    (key, name), = variants(p)
    assert not name.lstrip("-").isdigit()
    if nc is None:
        assert tgf.variant_names()[v] == name
    assert tuned(nc, p) == v and len(variants(p)) == 1            # read back

    # every kernel can be named, and is then taken without a timing
    names = tgf.variant_names() if nc is None else (
        ["lds", "rows1"] + (["matrix"] if nc != 5 else []))
    for n in names:
        p.write_text(f"{key} {n}\n")
        got = tuned(nc, p)
        assert len(variants(p)) == 1
        if nc is None:
            assert tgf.variant_names()[got] == n
        else:
            lds = int(tgf.tgf_sun_variant_lds(nc, got))
            assert n == ("rows%d" % tgf.tgf_sun_rows_per_lane(nc, got), "lds", "matrix")[lds]


@pytest.mark.parametrize("nc", [None, 4, 7])
@pytest.mark.parametrize("old", ["1", "9", "no_such_kernel"])
def test_entries_of_another_form_are_timed_anew(tmp_path, nc, old):
    p = tmp_path / "tune.txt"
    tuned(nc, p)
    (key, _), = variants(p)
    p.write_text(f"{key} {old}\n")
    v = tuned(nc, p)
    lines = variants(p)
    print(f"  nc {nc} entry {old}: {lines}", flush=True)
    assert [x[0] for x in lines] == [key, key] and lines[0][1] == old
    assert tuned(nc, p) == v and len(variants(p)) == 2
