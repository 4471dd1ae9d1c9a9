"""The tiles a mesh's own stages are launched with: by size until some are chosen (tiles() gives (0, 0)
all the while), then those chosen; and the batched workload's record, which names the tiles that
ran."""
import pytest

from paper_2308_06605_amd import inputs as I

pytestmark = pytest.mark.gpu


def _fr():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    fr.load()
    return fr


def test_by_size_then_chosen():
    fr = _fr()
    small, large = (fr.FRMesh(I.box_mesh(n, q=1), 3, mu=1e-3) for n in (4, 14))
    assert small.tiles() == large.tiles() == (0, 0)
    assert small.tiles_in_force() == (1, 2) and large.tiles_in_force() == (0, 0)
    for t in [(0, 0), (0, 1), (1, 2)]:
        small.set_tiles(*t)
        assert small.tiles() == small.tiles_in_force() == t
    large.set_tiles(*small.tiles_in_force())
    assert large.tiles_in_force() == (1, 2)
    tuned, _ = small.autotune(2)
    assert small.tiles() == small.tiles_in_force() == tuned
    small.close()
    large.close()
    with pytest.raises(fr.FRError):
        fr._check(fr.load().fr_tiles_in_force(None, None, None))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_record_of_the_batched_workload(prec):
    fr = _fr()
    from paper_2308_06605_amd import batched

    res = batched.run(n_mesh=3, steps=1, warmup=1, seed=0, prec=prec, autotune=False, sizes=(3, 5))
    for m in res["meshes"]:
        g, _ = batched.build(fr, m, True, prec)
        assert tuple(m["tiles_alone"]) == g.tiles_in_force() != (0, 0)
        assert tuple(m["tiles"]) == ((0, 0) if prec == "fp32" else g.tiles_in_force())
        g.close()


@pytest.mark.parametrize("p,dims,prec,tiles", [
    # half blocks on at most one per CU, faces of one wave up to 32768 face points
    (3, (8, 8, 8), "fp64", (1, 2)), (3, (8, 8, 9), "fp64", (0, 2)), (3, (9, 9, 10), "fp64", (0, 0)),
    (2, (10, 10, 10), "fp32", (1, 2)),
    (2, (11, 11, 11), "fp32", (0, 0)), (5, (8, 8, 8), "fp32", (0, 0)),
    # p = 4: one element per block where the fullest CU has an odd number, in FP64 also up to four
    (4, (6, 6, 7), "fp32", (1, 2)), (4, (8, 8, 8), "fp32", (0, 0)), (4, (8, 8, 9), "fp32", (1, 0)),
    (4, (8, 8, 8), "fp64", (1, 0)), (4, (11, 11, 11), "fp64", (0, 0)), (4, (13, 13, 13), "fp64", (1, 0))])
def test_choice_by_size(p, dims, prec, tiles):
    fr = _fr()
    kw = dict(prec="fp32", ref_rho=1.0, ref_p=1.0) if prec == "fp32" else {}
    g = fr.FRMesh(I.box_mesh(dims, q=1), p, mu=1e-3, **kw)
    assert g.tiles_in_force() == tiles
    g.close()


@pytest.mark.parametrize("chosen", [None, (1, 1)])
def test_failed_autotune_chooses_nothing(chosen):
    """An error left by another HIP call of the thread (a device number out of range) is what the
    autotuner's first launch check reports: it fails, and the tiles stay by size, or those chosen."""
    import ctypes

    fr = _fr()
    g = fr.FRMesh(I.box_mesh(4, q=1), 3, mu=1e-3)
    if chosen:
        g.set_tiles(*chosen)
    before = g.tiles(), g.tiles_in_force(), g.fusion()
    hip = ctypes.CDLL("libamdhip64.so.7")  # the one the library is linked with
    assert hip.hipSetDevice(4096) != 0
    with pytest.raises(fr.FRError):
        g.autotune(1)
    hip.hipGetLastError()
    assert (g.tiles(), g.tiles_in_force(), g.fusion()) == before
    g.close()
