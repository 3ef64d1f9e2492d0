"""What the binding takes of the card for the 12-bit copies, against a library and an allocator that only count."""
import pytest

from paper_2311_13581_amd import binding

GB = 1 << 30


class OutOfMemory(RuntimeError):
    pass


class Tensor:
    def __init__(self, card, nbytes):
        self.card, self.nbytes = card, nbytes
        card.used += nbytes

    def data_ptr(self):
        return 4096

    def numel(self):
        return self.nbytes

    def __del__(self):
        self.card.used -= self.nbytes


class Card:
    """torch, as far as the binding uses it for memory, on a card (number 3, not the current one) of a given size."""
    uint8, OutOfMemoryError = None, OutOfMemory

    def __init__(self, total):
        self.total, self.used, self.cuda = total, 0, self

    def empty(self, nbytes, dtype, device):
        assert device == 3
        if self.used + nbytes > self.total:
            raise OutOfMemory
        return Tensor(self, nbytes)

    def mem_get_info(self, dev):
        assert dev == 3
        return self.total - self.used, self.total

    def synchronize(self, dev):
        assert dev == 3

    def memory_reserved(self, dev):
        return 0

    memory_allocated = memory_reserved


class Library:
    def __init__(self, coded, train, unfit=0):
        self.coded, self.train, self.unfit, self.on, self.begun = coded, train, unfit, 0, []

    def pass_coded_bytes(self, h):
        return self.coded

    def pass_coded_begin(self, h, base, nbytes):
        assert nbytes == self.coded
        self.on, self.coded, self.unfit = nbytes, self.coded - self.unfit, 0
        return 0

    def pass_coded_end(self, h):
        self.on = 0
        return 0

    def pass_set_option(self, h, name, value):
        return 0

    def pass_train_bytes(self, h):
        return self.train

    def pass_train_begin(self, h, base, nbytes, token):
        self.begun.append(nbytes)
        return 0

    def pass_destroy(self, h):
        self.on = 0


def context(card, lib, arena, mode=None):
    g = binding.Pass.__new__(binding.Pass)
    g._torch, g.lib, g.h, g.coded, g._coded_mode, g._logits = card, lib, 1, None, None, binding._Results((1, 1), 0)
    g.arena = Tensor(card, arena)
    g.arena.device = 3
    if mode is not None:
        g.set_option("tune.coded", mode)
    return g


@pytest.mark.parametrize("arena,copies,mode,taken", [(14, 10, None, True), (180, 27, None, True), (180, 28, None, False), (180, 28, 1, True), (14, 10, 0, False),
                                                     (270, 28, 1, False)])
def test_copies_leave_the_card_to_the_program(arena, copies, mode, taken):
    """No more than a quarter of what is free of 288 GB unless they are asked for, and none where they are declined."""
    card, lib = Card(288 * GB), Library(copies * GB, 0)
    g = context(card, lib, arena * GB, mode)
    g._code_weights()
    assert (g.coded is not None) == taken == (lib.on > 0)
    assert card.used == arena * GB + (copies * GB + 256 if taken else 0)
    g.set_option("tune.coded", 0)  # declined later: given back
    assert g.coded is None and lib.on == 0 and card.used == arena * GB
    g.close()


def test_matrices_without_a_copy_give_their_share_back():
    card = Card(288 * GB)
    for unfit, left in ((4, 6), (10, 0)):
        lib = Library(10 * GB, 0, unfit * GB)
        g = context(card, lib, 14 * GB)
        g._code_weights()
        assert lib.on == left * GB and card.used == 14 * GB + (left * GB + 256 if left else 0)
        g.close()
        del g


def test_training_takes_the_room_of_the_copies():
    """Training that fits beside a model must fit when the model has copies."""
    card, lib = Card(288 * GB), Library(30 * GB, 100 * GB)
    g = context(card, lib, 60 * GB)
    g._code_weights()
    assert g.coded is not None
    other = card.empty(90 * GB, None, 3)
    g.train_begin()  # 60 + 30 + 90 + 100 would be 280: fits, its own copies do not
    assert lib.begun == [100 * GB] and lib.on
    g.train_ws = None
    more = card.empty(20 * GB, None, 3)
    g.train_begin()
    assert lib.begun == [100 * GB] * 2 and not lib.on and g.coded is None
    g.train_ws = None
    last = card.empty(60 * GB, None, 3)
    with pytest.raises(OutOfMemory):
        g.train_begin()
    g.close()
    del other, more, last
