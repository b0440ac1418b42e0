"""Autotuner for the FFT tile shapes of a Solver.

Knobs (pa_set_tiles), one set per pass: the register plan of the 1D
transforms (variant 0: more elements per thread; 1: more threads per
transform; 2: four elements per thread where the length allows; 3, row
passes only: variant 2's plan in persistent wavefronts that prefetch their
next rows into LDS), the workgroup shape (rows per workgroup for the forward
and the adjoint row passes, kx columns per workgroup for the column pass) and
for the column pass whether a column's two signals run on one team or on twin
teams (0: chosen per launch from the wavefronts it has; 1: one; 2 or 4:
twins).  The three passes are separate kernels reading and writing fixed
layouts, so each is tuned on its own: every candidate runs a short batched
forward + adjoint solve of the solver's own shape while the library times that
pass's launches with HIP events on the solver's stream (pa_profile_start).
Forward rows are scored by the right-hand-side row kernel, adjoint rows by the
adjoint-product row kernel, and the column pass by its forward plus adjoint
stage launches; for the column pass every (variant, block) pair is tried with
each col_split, since the best form depends on the block.  The best of each is
applied and returned.  Results depend on the choice only through the rounding
of the transforms (not at all on the column form).

Choices that run the same kernel with the same launch (same_launch) are timed
once, so that no noise decides between them, and the first of them is taken.
Grids up to 64^2 run their time loop in one kernel without these passes: a
pass whose first candidate launched nothing is not timed again, and its tiles
are left as they are.
"""

import time

import torch

ROW_VARIANTS = (0, 1, 2, 3)
COL_VARIANTS = (0, 1, 2)
BLOCKS = (1, 2, 4, 8)
COL_SPLITS = (0, 1, 2, 4)
ROW_NL, COL_FWD, ROW_ADJ, COL_ADJ = 0, 1, 2, 3

# threads per transform of the row plans 0, 1 and 2 (512 points have one plan, 1024 a plan of their own)
ROW_THREADS = {128: (8, 16, 32), 256: (16, 32, 64), 512: (64, 64, 64)}


def same_launch(N, name, variant, block, split):
    """A key that is equal for choices of one pass which launch the same kernel in the same shape."""
    if name != "col":
        if N == 1024:
            return ()   # four rows of plan 3 whatever the tiles
        if N == 512:
            variant = 2
        if N not in ROW_THREADS:
            return variant, block
        # variant 3: up to four wavefronts per workgroup; else up to 256 threads
        return variant, min(block, 4 if variant == 3 else 256 // ROW_THREADS[N][variant])
    if N == 512:
        variant = 1
    if N == 1024 and variant == 2:
        variant = 1
    return variant, block, 2 if split == 4 else split


def _class_cost(solver, omega0, n_steps, classes, reps):
    """Total device time (ms) of the launches of `classes` in one solve (min over reps)."""
    n = solver.N
    best = None
    for _ in range(reps):
        total = 0.0
        for cls in classes:
            solver.profile_start(cls, 1)
            solver.adjoint_impulse(omega0, n_steps, n // 2, n // 2, 1, ckpt_every=n_steps)
            p = solver.profile_stop()
            total += p["total_ms"] / max(p["timed_launches"], 1) * p["launches"]
        best = total if best is None else min(best, total)
    return best


def _time_solve(solver, omega0, n_steps, reps):
    stream = torch.cuda.current_stream(solver.device)
    n = solver.N
    solver.adjoint_impulse(omega0, n_steps, n // 2, n // 2, 1, ckpt_every=n_steps)   # warm
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(reps):
        solver.adjoint_impulse(omega0, n_steps, n // 2, n // 2, 1, ckpt_every=n_steps)
    e1.record(stream)
    e1.synchronize()
    return e0.elapsed_time(e1) / reps


def autotune(solver, omega0=None, n_steps=8, reps=2, verbose=False):
    """Pick the tiles of every pass for `solver`, apply them; returns a dict."""
    if omega0 is None:
        omega0 = solver.init_field(list(range(solver.B)), kind=0, k0=max(2.0, solver.N / 25), target=0.5)
    t_start = time.perf_counter()
    trials = []
    chosen = {}
    searches = (
        ("row", ROW_VARIANTS, "row_variant", "row_teams", (ROW_NL,)),
        ("adj", ROW_VARIANTS, "adj_variant", "adj_teams", (ROW_ADJ,)),
        ("col", COL_VARIANTS, "col_variant", "col_block", (COL_FWD, COL_ADJ)),
    )
    solver.set_tiles(col_split=0)
    for name, variants, vkey, bkey, classes in searches:
        splits = COL_SPLITS if name == "col" else (None,)
        best = None
        timed = {}
        kept = solver.get_tiles()
        for v in variants:
            for blk in BLOCKS:
                try:
                    solver.set_tiles(**{vkey: v, bkey: blk})
                except Exception:
                    continue
                for sp in splits:
                    key = same_launch(solver.N, name, v, blk, sp)
                    ms = timed.get(key)
                    if best is not None and best[0] == 0.0:
                        ms = 0.0
                    if ms is None:
                        if sp is not None:
                            solver.set_tiles(col_split=sp)
                        ms = timed[key] = _class_cost(solver, omega0, n_steps, classes, reps)
                    trials.append({"pass": name, "variant": v, "block": blk, "ms": ms}
                                  | ({} if sp is None else {"split": sp}))
                    if best is None or ms < best[0]:
                        best = (ms, v, blk, sp)
        if best[0] == 0.0:   # the solve launches no such pass (grids up to 64^2): keep its tiles
            best = (0.0, kept[vkey], kept[bkey], kept["col_split"] if splits != (None,) else None)
        chosen[vkey], chosen[bkey] = best[1], best[2]
        solver.set_tiles(**{vkey: best[1], bkey: best[2]})
        if best[3] is not None:
            chosen["col_split"] = best[3]
            solver.set_tiles(col_split=best[3])
    out = dict(solver.get_tiles())
    out["ms"] = _time_solve(solver, omega0, n_steps, reps)
    out["trials"] = trials
    out["seconds"] = time.perf_counter() - t_start
    out["probe"] = f"{solver.B} x {solver.N}^2, {n_steps} forward + {n_steps} adjoint steps"
    if verbose:
        for r in trials:
            print("autotune", r)
        print("autotune best", {k: out[k] for k in chosen} | {"ms": out["ms"]})
    return out
