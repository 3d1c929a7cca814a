"""The symmetry check of an incoming H over the forms of storage it accepts: sorted and shuffled rows, duplicate
entries, entries stored on one side only.  No GPU."""
import numpy as np
import pytest

import synth
import paper_1702_05167_amd as pkg
import paper_1702_05167_amd.hsc as H

FAULTS = (None, "value", "imaginary", "one_sided_zero", "missing", "moved")


@pytest.mark.parametrize("fault", FAULTS)
@pytest.mark.parametrize("form", ["sorted", "shuffled", "duplicates", "shuffled_duplicates"])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_symmetry_check(form, fault, seed):
    rng = np.random.default_rng(seed)
    dev = synth.cuboid(5, 4, 3)
    rows = [[] for _ in range(dev.n)]
    for r in range(dev.n):
        for q in range(dev.indptr[r], dev.indptr[r + 1]):
            rows[r].append((int(dev.indices[q]), complex(dev.values[q])))
    r = int(rng.integers(dev.n))
    k = next(i for i, (c, _) in enumerate(rows[r]) if c != r)
    c, v = rows[r][k]
    if fault == "value":
        rows[r][k] = (c, v + 0.25)
    elif fault == "imaginary":
        rows[r][k] = (c, v + 0.25j)
    elif fault == "one_sided_zero":
        far = next(x for x in rng.permutation(dev.n).tolist() if x != r and all(x != y for y, _ in rows[r]))
        rows[r].append((far, 0.0))
        rows[r].sort()
    elif fault == "missing":
        del rows[r][k]
    elif fault == "moved":      # the same number of entries, one in a column that has no mirror
        far = next(x for x in rng.permutation(dev.n).tolist() if x != r and all(x != y for y, _ in rows[r]))
        rows[r][k] = (far, v)
        rows[r].sort()
    indptr, indices, values = [0], [], []
    for entries in rows:
        if "duplicates" in form:    # in exact halves and quarters
            entries = [e for c_, v_ in entries for e in ([(c_, v_ / 2), (c_, v_ / 4), (c_, v_ / 4)] if rng.random() < 0.5
                                                         else [(c_, v_)])]
        if "shuffled" in form:
            entries = [entries[i] for i in rng.permutation(len(entries))]
        indices += [e[0] for e in entries]
        values += [e[1] for e in entries]
        indptr.append(len(indices))
    contacts = [(x.sites, x.lead_onsite, x.lead_hopping, x.coupling) for x in dev.contacts]
    args = (dev.n, np.array(indptr), np.array(indices), np.array(values), dev.coords, contacts, 7, 2)
    if fault is None:
        pkg.Tree.build(*args)
    else:
        with pytest.raises(H.HscError) as e:
            pkg.Tree.build(*args)
        assert e.value.code == -2
