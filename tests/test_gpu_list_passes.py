"""The list passes at the sizes where they change form: one sort run, several runs in one
workgroup, runs merged by many workgroups (2^16 voxels and more, up to 32 instances), one and
several union-find batches with and without the sequential finish, one and several output
workgroups, the images' dual beside H0 or after it (more than 64 instances).  Bit for bit against
the oracle."""
import numpy as np
import pytest

import oracle
import synthetic as S
from gpu_util import diff_pairs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2606_04801_amd as fc  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
DEV = torch.device("cuda:0")


def staircase(n):
    """Every merge waits for the previous one: the rounds run out in every batch."""
    a = np.zeros(2 * n + 1, np.float32)
    a[0::2] = np.linspace(0.5, 0.1, n + 1).astype(np.float32)
    a[1::2] = np.linspace(1.0, 2.0, n).astype(np.float32)
    return a.reshape(1, -1)


# noise keeps about 0.31 edges, 0.2 minima a pixel; 0.33 edges, 0.2 squares a voxel
CASES = {
    "one_run_2k": lambda: S.uniform((81, 81), 1),                # 2,048 edges a run of two keys a thread
    "one_run_4k": lambda: S.uniform((114, 115), 2),              # about 4,096 edges
    "two_runs_in_place": lambda: S.uniform((117, 118), 3),
    "below_multi": lambda: S.uniform((255, 256), 4),             # 65,280 pixels: one workgroup a list
    "multi": lambda: S.uniform((256, 256), 5),
    "multi_ties": lambda: S.levels((256, 257), 7, 6),
    "multi_volume": lambda: S.uniform((40, 41, 41), 7),
    "strip": lambda: S.levels((1, 70000), 40, 8),
    "staircase_two_batches": lambda: staircase(9000),
    "seventeen_runs": lambda: S.uniform((340, 341), 9),          # 36k edges: five union-find batches
}


@pytest.mark.parametrize("filtration", ["V", "T"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_single(name, filtration):
    img = CASES[name]()
    print("case", name, img.shape, filtration, flush=True)
    got = fc.ph_diagram(torch.from_numpy(img).to(DEV), filtration=filtration).numpy()
    assert diff_pairs(got, oracle.diagram(img, filtration=filtration)) is None


@pytest.mark.parametrize("n", [32, 33, 64, 65])
def test_batches(n):
    """A multi-run image beside small instances, at both sides of the batch limits."""
    imgs = [S.uniform((256, 256), 20), S.uniform((24, 20, 22), 21)]
    imgs += [S.levels((17 + k % 5, 23), 9, 30 + k) for k in range(n - 2)]
    bt = fc.Batch([a.shape for a in imgs], device=DEV)
    bt.set_images([torch.from_numpy(a) for a in imgs])
    print("batch of", n, flush=True)
    bt.ph_diagram_batch()
    for a, got in zip(imgs, bt.results()):
        assert diff_pairs(got, oracle.diagram(a)) is None, a.shape


def test_multi_run_volume_with_h1():
    """Each vertex's first KEEP edge is found across runs (3D H1 looks its edges up by it)."""
    img = S.uniform((41, 40, 42), 40)
    fl = fc.PH_H0 | fc.PH_HTOP | fc.PH_H1
    print("h1", img.shape, flush=True)
    got = fc.ph_diagram(torch.from_numpy(img).to(DEV), flags=fl).numpy()
    want = oracle.diagram(img, dims=(0, 2))
    assert diff_pairs(got[got["dim"] != 1], want) is None
    small = S.levels((20, 60, 60), 6, 41)                        # 72,000 voxels, ties across runs
    got = fc.ph_diagram(torch.from_numpy(small).to(DEV), flags=fl).numpy()
    assert diff_pairs(got[got["dim"] != 1], oracle.diagram(small, dims=(0, 2))) is None
    assert (got["dim"] == 1).any()


def test_wide_rounds_past_a_clearing():
    """2^22 pixels of noise under PH_WIDE, against the call without the flag (one workgroup's union-find
    out of the workspace, runs merged in one pass): eight wide rounds, with the nodes' words cleared
    after seven, and merges in three passes."""
    img = torch.from_numpy(S.uniform((2100, 2050), 50)).to(DEV)
    print("wide", img.shape, flush=True)
    got = fc.ph_diagram(img, flags=fc.PH_H0 | fc.PH_HTOP | fc.PH_WIDE).numpy()
    assert len(got) > 10 ** 6 and diff_pairs(got, fc.ph_diagram(img).numpy()) is None


@pytest.mark.parametrize("n", [32, 33])
def test_wide_sort_in_batches(n):
    """Under PH_WIDE a large instance's lists are sorted by many workgroups beside any number of others:
    the three merge passes are launched, and the pairs are those of the call without the flag."""
    imgs = [S.uniform((1024, 1024), 60), S.uniform((24, 20, 22), 61)]
    imgs += [S.levels((17 + k % 5, 23), 9, 62 + k) for k in range(n - 2)]
    res = []
    for flags in (fc.PH_H0 | fc.PH_HTOP, fc.PH_H0 | fc.PH_HTOP | fc.PH_WIDE):
        bt = fc.Batch([a.shape for a in imgs], flags=flags, device=DEV)
        bt.set_images([torch.from_numpy(a) for a in imgs])
        print("batch of", n, "flags", flags, flush=True)
        fc.profile(True)
        bt.ph_diagram_batch()
        torch.cuda.synchronize()
        launches = fc.profile_read()
        fc.profile(False)
        res.append(bt.results())
        if flags & fc.PH_WIDE:
            assert launches["k_sort_merge"][0] == 3, launches
    for a, b in zip(*res):
        assert diff_pairs(a, b) is None


@pytest.mark.parametrize("filtration", ["V", "T"])
@pytest.mark.parametrize("kind", ["field", "ties"])
def test_h1_pairs_of_multi_run_volumes(kind, filtration):
    """The H1 pairs, too, where each vertex's first KEEP edge is found across runs: two runs and
    more of edges, against the oracle's reduction of every dimension."""
    img = S.grf((41, 40, 42), 0.7, 40) if kind == "field" else S.levels((41, 40, 42), 6, 41)
    bt = fc.Batch([img.shape], flags=fc.PH_H0 | fc.PH_HTOP | fc.PH_H1, filtration=filtration, device=DEV)
    bt.set_images([torch.from_numpy(img)])
    print("h1", kind, filtration, flush=True)
    bt.ph_diagram_batch()
    (got,) = bt.results()
    assert diff_pairs(got, oracle.diagram(img, dims=(0, 1, 2), filtration=filtration)) is None
    assert bt.work_counters()[0, 0] > 2048


@pytest.mark.parametrize("side, h0, top", [(440, False, False), (456, True, False), (610, True, True)])
def test_forests_at_the_lds_limit(side, h0, top):
    """The two union-finds of noise at both sides of 40,000 nodes, where they leave LDS for the workspace."""
    img = S.uniform((side, side + 1), 70)
    bt = fc.Batch([img.shape], device=DEV)
    bt.set_images([torch.from_numpy(img)])
    print("forests", img.shape, flush=True)
    bt.ph_diagram_batch()
    (got,) = bt.results()
    wc = bt.work_counters()
    assert (wc[0, 2] > 40000) == h0 and (wc[0, 3] > 40000) == top and 36000 < wc[0, 2 + top] < 44000, wc[0]
    assert diff_pairs(got, oracle.diagram(img)) is None


def ramp_noise(n, slope, seed):
    """Noise on a ramp: the lists' order follows the image, so sorted runs hold bands of it."""
    return S.uniform((n, n), seed) + slope * np.arange(n, dtype=np.float32)[:, None]


@pytest.mark.parametrize("filtration", ["V", "T"])
@pytest.mark.parametrize("kind", ["ramp", "checkerboard"])
def test_lists_ordered_like_the_image(kind, filtration):
    """Merges whose windows in the other runs are far larger than the keys placed, in one pass and
    (PH_WIDE) in three: the same pairs, the ramp's (V) as the oracle has them (the checkerboard takes it
    minutes; its pairs are counted)."""
    img = ramp_noise(1024, 0.05, 71) if kind == "ramp" else (np.indices((1024, 1024)).sum(axis=0) % 2).astype(np.float32)
    a = torch.from_numpy(img).to(DEV)
    got = []
    for flags in (fc.PH_H0 | fc.PH_HTOP, fc.PH_H0 | fc.PH_HTOP | fc.PH_WIDE):
        print("ordered", kind, filtration, flags, flush=True)
        got.append(fc.ph_diagram(a, flags=flags, filtration=filtration).numpy())
    assert diff_pairs(*got) is None
    if kind == "checkerboard":
        assert filtration == "T" or len(got[0]) == 1 << 19
    elif filtration == "V":
        assert diff_pairs(got[0], oracle.diagram(img)) is None
