"""The order in which a decode launch walks the groups of a sequence, from a host build of the header that the kernel includes."""
import pytest

from tests.decode_model import build_model

WAVES = 4


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    return build_model(tmp_path_factory)


def walk(model, count, n, bits):
    """(groups of every wave in its order, by (split, wave); rounds that split 0 sits out)."""
    skip = model.rounds_left_out(count, n, bits)
    waves = {}
    for split in range(n):
        for wave in range(WAVES):
            r, mine = skip if split == 0 else 0, []
            while True:
                g = model.group_of_round(n, split, wave, skip, r)
                if g >= count:
                    break
                mine.append(g)
                r += 1
            waves[split, wave] = mine
    return waves, skip


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 16, 31, 32])
def test_every_group_once_and_in_as_few_rounds_as_one_skipped_round_takes(model, n, bits):
    for count in list(range(0, 40 * n if n < 8 else 10 * n)) + [1023, 1024, 1025]:
        waves, skip = walk(model, count, n, bits)
        assert sorted(g for mine in waves.values() for g in mine) == list(range(count)), (count, n)
        assert skip in (1, 2) and (bits == 2 or skip == 1)
        if n > 1 and count > 0:
            rounds = max(len(mine) + (skip if split == 0 and mine else 0) for (split, _), mine in waves.items())
            assert rounds <= -(-(count + WAVES) // (WAVES * n)), (count, n, skip)


def test_the_first_group_of_the_other_splits_does_not_depend_on_the_length(model):
    """Their waves request it before the length of the sequence is known."""
    for n in (2, 3, 8, 32):
        for split in range(1, n):
            for wave in range(WAVES):
                assert model.group_of_round(n, split, wave, 1, 0) == model.group_of_round(n, split, wave, 2, 0)
