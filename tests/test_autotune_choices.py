"""The tile search on the CPU, with a solver that only keeps its tiles: choices that launch the same
kernel are timed once, and passes that are not launched are not searched."""

import pytest

from paper_2602_14016_amd import autotune as at


class Tiles:
    def __init__(self, N):
        self.N, self.B = N, 1
        self.t = dict(row_variant=2, row_teams=4, adj_variant=2, adj_teams=4, col_variant=1, col_block=2, col_split=0)

    def set_tiles(self, **t):
        self.t.update(t)

    def get_tiles(self):
        return dict(self.t)


def search(monkeypatch, N, cost):
    """The search's result, the tiles of every timing and the final tiles, where the i-th timing reads cost(i)."""
    s, seen = Tiles(N), []

    def timing(solver, omega0, n_steps, classes, reps):
        seen.append((classes, solver.get_tiles()))
        return cost(len(seen))

    monkeypatch.setattr(at, "_class_cost", timing)
    monkeypatch.setattr(at, "_time_solve", lambda *a: 1.0)
    return at.autotune(s, omega0=0), seen, s.get_tiles()


@pytest.mark.parametrize("N", [8, 32, 64])
def test_grids_without_these_passes_are_not_searched(monkeypatch, N):
    out, seen, tiles = search(monkeypatch, N, lambda i: 0.0)
    assert len(seen) == 3 and tiles == Tiles(N).t
    assert {r["pass"] for r in out["trials"]} == {"row", "adj", "col"} and all(r["ms"] == 0.0 for r in out["trials"])


# rows: plans 0, 1, 2 and the pipelined one with 1, 2, 4 and 8 rows, less what the 256 threads or four
# wavefronts of a workgroup cap; columns: three plans, four widths, three forms
@pytest.mark.parametrize("N,rows,cols", [(128, 15, 36), (256, 14, 36), (512, 3, 12), (1024, 1, 24)])
def test_equal_launches_are_timed_once(monkeypatch, N, rows, cols):
    """Every timing reads less than the one before: a copy timed again would be taken for its noise."""
    out, seen, tiles = search(monkeypatch, N, lambda i: 100.0 - 0.1 * i)
    per_pass = [sum(1 for c, _ in seen if c == k) for k in ((0,), (2,), (1, 3))]
    assert per_pass == [rows, rows, cols]
    assert len(out["trials"]) == 16 + 16 + 48   # every choice is listed with its launch's time
    assert tiles["col_split"] != 4
    if N == 1024:
        assert (tiles["row_variant"], tiles["row_teams"]) == (0, 1)
    if N == 512:
        assert tiles["row_variant"] == tiles["adj_variant"] == 0 and tiles["row_teams"] == 4
