"""The seats that teams of workgroups reserve and the time they are waited for
(host code, no GPU needed)."""
import itertools
import threading

import paper_2409_15468_amd as cb

XCDS, CUS = 8, 256


def test_teams_that_are_seated_together_fit_every_xcd():
    """Workgroup w of a launch runs on XCD w % 8, so a team of G takes
    ceil(G / 8) of the 32 CUs of the first ones: teams whose seats sum to at
    most 256 must not ask any XCD for more than it has."""
    seats = cb.lib().cb_internal_team_seats
    sizes = [1, 7, 8, 9, 41, 63, 65, 120, 121, 128]
    for n in (1, 2, 3, 4):
        for teams in itertools.combinations_with_replacement(sizes, n):
            if sum(seats(g, CUS) for g in teams) <= CUS:
                assert sum(-(-g // XCDS) for g in teams) <= CUS // XCDS, teams
    for g in (1, 8, 9, 200, 249, 256):
        assert g <= seats(g, CUS) <= CUS
    assert seats(30, 30) == 30  # a device of fewer CUs seats the largest team it takes


def test_wait_shrinks_while_teams_do_not_form():
    """A quarter of half a second for each team in a row that does not form, 2 ms
    at least, and all of it again after one that does; per host thread."""
    waited = cb.lib().cb_internal_team_waited
    assert waited(1) == 500000
    assert [waited(0) for _ in range(12)] == [125000, 31250, 7812, 2000] + [2000] * 8
    other = []
    t = threading.Thread(target=lambda: other.append(waited(1)))
    t.start()
    t.join()
    assert other == [500000] and waited(0) == 2000
    assert waited(1) == 500000
