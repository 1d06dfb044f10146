"""The tuning cache: entries of this library's kernel set are taken as they
are, those of another set are not."""
import pytest

pytestmark = pytest.mark.gpu

KEYS = [f"{p}:32:fp64" for p in ("zinv", "yinv", "xpass", "yfwd")]


def tuned(path):
    import paper_2506_23712_amd as ens
    E = ens.Ensemble()
    E.add_member(ens.MemberSpec(n=32, nu=0.02, kf_hi=2.0, dt=0.01, seed=1))
    table = E.autotune(cache_path=str(path))
    E.close()
    return table


def entries(path):
    return dict(l.split() for l in path.read_text().splitlines() if l and not l.startswith("#"))


def test_entries_of_this_kernel_set_are_kept(tmp_path):
    path = tmp_path / "variants.txt"
    tuned(path)
    head = path.read_text().splitlines()[0]
    assert set(entries(path)) == set(KEYS)
    path.write_text(head + "\n# a comment\n" + "".join(f"{k} 1\n" for k in KEYS) + "yinv:64:fp32 3\n")
    assert all(tuned(path)[k] == 1 for k in KEYS)
    assert path.read_text().splitlines()[0] == head and entries(path)["yinv:64:fp32"] == "3"


@pytest.mark.parametrize("head", ["", "# libensdns kernel variants (pass:n:precision variant); 0 = 8, 1 = 16 values per thread\n",
                                  "# libensdns kernel set 1\n"])
def test_entries_of_another_kernel_set_are_timed_anew(tmp_path, head):
    """x-pass variant 1 (separate passes, 16 of 32 values per thread) takes nearly
    twice as long as the plane pass here: only an entry could choose it."""
    path = tmp_path / "variants.txt"
    path.write_text(head + "".join(f"{k} 1\n" for k in KEYS) + "xpass:64:fp32 2\n")
    assert tuned(path)["xpass:32:fp64"] != 1
    assert set(entries(path)) == set(KEYS) and entries(path)["xpass:32:fp64"] != "1"
