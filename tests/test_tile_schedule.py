"""The order in which the tile backward hands out its items (tile_schedule and next_item of lp_mfma_bwd_tile.h), modelled on the CPU: every
item is marched exactly once, over whole rounds, a move of the workgroups from round to round, and a partial round."""
import pytest

WAVES = 8


def _items(items, blocks, spread):
    """How often each item is handed out.  `spread`: a group is one item of each eighth of the list, else eight neighbours."""
    waves = blocks * WAVES
    rounds, tail = divmod(items, waves)
    busy = -(-tail // blocks)
    if rounds and busy > WAVES // 2:
        busy = WAVES
    tail_per_xcd = -(-(-(-tail // busy)) // 8) if busy else 0
    n_groups = rounds * blocks
    mul = next((p for p in (7919, 7907, 7901, 7883) if n_groups % p), 1)
    shift = blocks * 5 // 8 | 1
    step = [(shift + blocks) * mul % n_groups, shift * mul % n_groups] if n_groups else [0, 0]
    count = [0] * items
    for block in range(blocks):
        place, group = block, block * mul % n_groups if rounds else 0
        for _ in range(rounds):
            for wave in range(WAVES):
                count[wave * n_groups + group if spread else group * WAVES + wave] += 1
            place += shift
            wraps = place >= blocks
            place -= blocks * wraps
            group += step[wraps]
            group -= n_groups * (group >= n_groups)
        for wave in range(WAVES):
            item = n_groups * WAVES + (tail_per_xcd * (block % 8) + block // 8) * busy + wave
            if wave < busy and block // 8 < tail_per_xcd and item < items:
                count[item] += 1
    return count


@pytest.mark.parametrize("spread", [False, True])
@pytest.mark.parametrize("blocks", [8, 24, 80, 256, 304])
def test_every_item_once(blocks, spread):
    waves = blocks * WAVES
    for items in (1, 7, blocks - 1, blocks, blocks + 1, 3 * blocks + 5, waves - 1, waves, waves + 1, waves + blocks, waves + 5 * blocks, 2 * waves,
                  3 * waves + 517, 4 * waves + 1, 7 * waves - 1, 19 * waves + 4 * blocks + 3):
        assert set(_items(items, blocks, spread)) == {1}, items


@pytest.mark.parametrize("blocks,rounds", [(8, 7919), (8, 7907), (16, 7919)])
def test_rounds_that_the_first_prime_divides(blocks, rounds):
    for tail in (0, 3, 5 * blocks):
        assert set(_items(rounds * blocks * WAVES + tail, blocks, tail == 0)) == {1}
