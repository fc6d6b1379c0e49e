"""What choose_layout allocates: any candidate's own workspace fits, all of them side by side only where they share one
pass, and not where the memory is not there. Host arithmetic; no GPU."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture
def sizes(monkeypatch):
    import paper_2412_14973_amd as tl
    asked, limit = [], [1 << 60]

    def empty(n, dtype, device):   # sizes only
        assert dtype == torch.uint8 and device == "cuda"
        asked.append(n)
        if n > limit[0]:
            raise torch.OutOfMemoryError()
        return n
    monkeypatch.setattr(tl.torch, "empty", empty)

    def ask(nr, cand, memory=1 << 60):
        limit[0] = memory
        return tl._layout_workspace(nr, np.array(cand, dtype=np.int32), "cuda"), [tl._ranks_workspace_bytes(nr, d)
                                                                                    for d in cand if 1 <= d <= 1024]
    return ask


# a candidate that does not share the pass (up to 32 rows, above 256), and one alone
@pytest.mark.parametrize("nr,cand", [(1024, [256, 512]), (4000, [256, 512, 1024]), (1024, [16, 32, 64]), (1024, [128]),
                                     (300, [512, 16])])
def test_no_room_that_no_pass_uses(sizes, nr, cand):
    total, alone = sizes(nr, cand)
    assert total == max(alone)


SHARED = [(1024, [64, 128, 256]), (97, [33, 97]), (410, [200, 64, 256, 200]), (300, [256, 256]), (64, [64, 128, 256]),
          (9000, [200, 256])]


@pytest.mark.parametrize("nr,cand", SHARED)
def test_room_for_all_in_one_pass(sizes, nr, cand):
    total, alone = sizes(nr, cand)
    assert max(alone) < total <= sum(alone) + 2 ** 16


@pytest.mark.parametrize("nr,cand", SHARED)
def test_one_by_one_where_the_memory_is_short(sizes, nr, cand):
    alone = max(sizes(nr, cand)[1])
    assert sizes(nr, cand, memory=alone)[0] == alone


def test_sizes_out_of_range_are_the_librarys_to_report(sizes):
    import paper_2412_14973_amd as tl
    assert sizes(1024, [-3, 64])[0] == tl._ranks_workspace_bytes(1024, 64)
    for cand in ([2000], [64, 2000], [0]):
        with pytest.raises(tl._lib.TLRMDDError):
            sizes(1024, cand)
