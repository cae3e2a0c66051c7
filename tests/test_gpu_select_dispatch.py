"""Selection at the edges of its dispatch (one wave with one or two units per lane, or up to eight
where segments are many; a workgroup with one, two, four or eight per thread), with candidate
keys that agree in their high bits, are all equal, or span the whole key range, and budgets from
nothing to everything, against the oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_34653_amd import omnitide
    omnitide.lib()
    yield


def _scores(kind, rng, U):
    if kind == "clustered":                   # agree but for the low bits: first digit far down
        return (1 << 41) + rng.integers(0, 700, size=U)
    if kind == "equal":                       # ranked by unit id alone
        return np.full(U, 12345)
    return np.floor(2.0 ** rng.uniform(0, 49, size=U)).astype(np.int64)     # every key length


@pytest.mark.parametrize("U", [1, 63, 64, 65, 128, 129, 512, 1024, 1025, 2049, 4096, 8191,
                               8192])
@pytest.mark.parametrize("kind", ["clustered", "equal", "wide"])
def test_select_matches_oracle(U, kind):
    from paper_2609_34653_amd import omnitide as ot
    rng = np.random.default_rng(U + len(kind))
    lens = rng.integers(0, 60, size=U)
    lens[0] = 5
    end = np.cumsum(lens)
    first = np.where(lens > 0, end - lens, 10 ** 7)
    last = np.where(lens > 0, end - 1, -1)
    wsum = _scores(kind, rng, U) * lens + rng.integers(0, np.maximum(lens, 1))
    flags = (np.arange(U) == 0).astype(np.int64)
    total, sysn = int(lens.sum()), int(lens[0])
    up = lambda a, t=np.int32: torch.from_numpy(np.asarray(a, t)).cuda()   # noqa: E731
    dev = (up(wsum, np.int64), up(lens), up(first), up(last), up(flags))
    # nothing beyond the prefix, one candidate's worth, a part, all but one token, everything
    for budget, recent in ((sysn, 0), (sysn + 25, 0), (total // 3, 300), (total - 1, 0),
                           (total, total), (total, 100)):
        budget = max(budget, sysn)            # the prefix always fits
        sc = torch.full((U,), -7, dtype=torch.int64, device="cuda")
        keep = torch.full((U,), 9, dtype=torch.uint8, device="cuda")
        kept = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        stat = torch.zeros(1, dtype=torch.int32, device="cuda")
        ot.omnitide_select_units(*dev, 1, U, budget, recent, sc, keep, kept, stat)
        torch.cuda.synchronize()
        assert int(stat.item()) == 0
        score, want, n = oracle.select_units(wsum, lens, first, last, flags, budget, recent)
        assert np.array_equal(sc.cpu().numpy(), score)
        assert np.array_equal(keep.cpu().numpy(), want), (budget, recent)
        assert int(kept.item()) == n


@pytest.mark.parametrize("U,n_seg", [(129, 256), (129, 257), (256, 257), (257, 512), (257, 513),
                                     (512, 513), (513, 513)])
def test_select_many_segments(U, n_seg):
    """Both sides of the segment counts from which one wave plans more than 128 units: five
    patterns over all segments (one over budget, one malformed)."""
    from paper_2609_34653_amd import omnitide as ot
    rng = np.random.default_rng(U + n_seg)
    parts = []
    for i in range(5):
        lens = rng.integers(0, 60, size=U)
        lens[0] = 40
        end = np.cumsum(lens)
        first = np.where(lens > 0, end - lens, 10 ** 7)
        last = np.where(lens > 0, end - 1, -1)
        wsum = _scores(("clustered", "equal", "wide", "wide", "wide")[i], rng, U) * lens
        flags = np.zeros(U, np.int64)
        flags[:30 if i == 3 else 1] = 1                   # 3: the prefix alone exceeds the budget
        if i == 4:
            last[int(np.argmax(lens))] += 1               # 4: a unit's slots are not one run
        parts.append((wsum, lens, first, last, flags))
    budget, recent = 400, 150
    order = [(3 * i) % 5 for i in range(n_seg)]
    up = lambda k, t: torch.from_numpy(np.concatenate([parts[o][k] for o in order])  # noqa: E731
                                       .astype(t)).cuda()
    sc = torch.full((n_seg * U,), -7, dtype=torch.int64, device="cuda")
    keep = torch.full((n_seg * U,), 9, dtype=torch.uint8, device="cuda")
    kept = torch.full((n_seg,), -7, dtype=torch.int32, device="cuda")
    stat = torch.zeros(1, dtype=torch.int32, device="cuda")
    ot.omnitide_select_units(up(0, np.int64), up(1, np.int32), up(2, np.int32), up(3, np.int32),
                             up(4, np.int32), n_seg, U, budget, recent, sc, keep, kept, stat)
    torch.cuda.synchronize()
    assert int(stat.item()) in (ot.E_BUDGET, ot.E_TAGS)
    sc, keep = sc.cpu().numpy().reshape(n_seg, U), keep.cpu().numpy().reshape(n_seg, U)
    kept = kept.cpu().numpy()
    for o in range(5):
        at = [i for i in range(n_seg) if order[i] == o]
        if o < 3:
            score, want, n = oracle.select_units(*parts[o], budget, recent)
            assert np.array_equal(sc[at], np.tile(score, (len(at), 1)))
        else:
            want, n = np.zeros(U), 0
        assert np.array_equal(keep[at], np.tile(want, (len(at), 1))), o
        assert np.all(kept[at] == n)
