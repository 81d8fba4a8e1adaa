"""The hand-over of generation's one launch, as the library states it for every work item: no GPU."""
import numpy as np
import pytest

import paper_2410_13229_amd as Q

WRITTEN, AWAITED, WATCHED = 0, 1, 2


def _items(*shape):
    """Rows (buffer, word, tag minus number of the block, how) of every item, roles one after the other."""
    items = []
    for role in range(4):
        item = 0
        while (words := Q.quamba_debug_decode_stack_words(*shape, role, item)) is not None:
            items.append(np.frombuffer(words, np.int32).reshape(-1, 4))
            item += 1
    return items


@pytest.mark.parametrize("shape", [(768, 1536, 48, 1), (768, 1536, 48, 2), (1024, 2048, 64, 1), (1280, 2560, 256, 2), (3072, 1536, 16, 1),
                                   (2560, 5120, 160, 1), (2560, 5120, 160, 2)])
def test_a_word_keeps_its_tag_until_every_item_that_needs_this_very_tag_has_read_it(shape):
    """The item that writes a word for the next block has to depend, through the words it awaits itself, on every item that accepts
    the present tag alone; otherwise an item that is held up misses the tag and waits for ever."""
    items = _items(*shape)
    n = len(items)
    items = [rows.tolist() for rows in items]
    writer = {(b, w): (i, t) for i, rows in enumerate(items) for b, w, t, how in rows if how == WRITTEN}
    same, before = np.zeros((n, n), bool), np.zeros((n, n), bool)  # direct: [i, j] item i awaits a word of j, of its own block or of the one before
    needs = []                                                     # item, writer, is the writer's next word one of the item's own block
    for i, rows in enumerate(items):
        for b, w, t, how in rows:
            if how == AWAITED:
                j, written = writer[b, w]
                own = t == written
                assert own or t == written - 1
                (same if own else before)[i, j] = True
                needs.append((i, j, not own))
    closed = same | np.eye(n, dtype=bool)
    for _ in range(2):  # four roles in a row
        closed = (closed.astype(np.float32) @ closed.astype(np.float32)) > 0
    through = (closed.astype(np.float32) @ before.astype(np.float32) @ closed.astype(np.float32)) > 0
    for i, j, in_this_block in set(needs):
        assert (closed if in_this_block else through)[j, i], f"item {i} may miss the tag of a word of item {j}"


@pytest.mark.parametrize("Di", [1536, 5120])
@pytest.mark.parametrize("Bt", [1, 2])
def test_every_word_that_is_waited_for_is_one_that_some_item_writes(Di, Bt):
    """At every rank and the widths of the model around and below it, where there are more columns of x_proj than of out_proj to wait at
    (d_model 64 with rank 16: 12 items of x_proj, 7 of out_proj)."""
    for Dm in [*range(16, 200, 16), 336, 496, 624, 640, 688, 704, 720, 2560]:
        for R in range(16, 257, 16) if Bt == 1 else (16, 160, 256):
            rows = np.concatenate(_items(Dm, Di, R, Bt))
            words = np.unique(rows[:, 0] * 2 ** 24 + rows[:, 1] + (rows[:, 3] == WRITTEN) * 2 ** 30)
            written = words[words >= 2 ** 30] - 2 ** 30
            lost = np.setdiff1d(words[words < 2 ** 30], written)
            assert lost.size == 0, f"d_model {Dm} rank {R}: nobody writes words {[(int(k) >> 24, int(k) % 2 ** 24) for k in lost[:4]]}"
