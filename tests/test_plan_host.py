"""The plan of a tiled contraction launch (rows of a tile, pieces of a contraction) against its own estimate of every form that it
weighs.  The planner is host code and works on 256 compute units here; no GPU needed."""
import ctypes
import random

import pytest

CUS = 256
ANY = 2 ** 64 - 1


class SplitJob(ctypes.Structure):
    _fields_ = [("tiles_c", ctypes.c_int), ("KC", ctypes.c_int), ("out_bytes", ctypes.c_size_t), ("split", ctypes.c_int)]


class Planner:
    def __init__(self, lib):
        i, b, d, z, p = ctypes.c_int, ctypes.c_bool, ctypes.c_double, ctypes.c_size_t, ctypes.POINTER(SplitJob)
        self.plan_fn = lib._ZN4peqa9gemm_planEiPNS_8SplitJobEibbbdmi           # peqa::gemm_plan
        self.plan_fn.argtypes, self.plan_fn.restype = [i, p, i, b, b, b, d, z, i], i
        self.us_fn = lib._ZN4peqa12gemm_form_usEiPKNS_8SplitJobEiibbdi         # peqa::gemm_form_us
        self.us_fn.argtypes, self.us_fn.restype = [i, p, i, i, b, b, d, i], d
        self.chains_fn = lib._ZN4peqa13bwd_dx_chainsEiPKNS_8SplitJobEii        # peqa::bwd_dx_chains
        self.chains_fn.argtypes, self.chains_fn.restype = [i, p, i, i], b
        self.rows_fn = lib._ZN4peqa14gemm_row_tilesEi                          # peqa::gemm_row_tiles

    def rows(self, T):
        return self.rows_fn(T)

    def plan(self, jobs, T, grouped, single, dds=False, other=0.0, most=ANY):
        """(row tiles per tile, pieces of every job); jobs: (columns, contraction length, bytes of a piece's results)."""
        a = self._jobs(jobs, [1] * len(jobs))
        return self.plan_fn(len(jobs), a, T, grouped, single, dds, other, most, CUS), [j.split for j in a]

    def us(self, jobs, splits, T, rt, grouped, single, other=0.0):
        return self.us_fn(len(jobs), self._jobs(jobs, splits), T, rt, grouped, single, other, CUS)

    def chains(self, jobs, splits, T):
        return self.chains_fn(len(jobs), self._jobs(jobs, splits), T, CUS)

    @staticmethod
    def _jobs(jobs, splits):
        return (SplitJob * len(jobs))(*[SplitJob((c + 255) // 256, kc, nb, s) for (c, kc, nb), s in zip(jobs, splits)])


@pytest.fixture(scope="module")
def planner():
    from paper_2305_14152_amd import peqa
    return Planner(peqa.lib())


def _forward(layers, T):
    return [(n, k, 4 * T * n) for n, k in layers]


def _forms(planner, jobs, T, grouped, single, other):
    """Every form that may be taken, with its estimate: (whole?, rows, pieces, us); the one of gemm_row_tiles rows, whole, first."""
    longest, by_rows = max(kc for _, kc, _ in jobs), planner.rows(T)
    for rt in [by_rows] + [r for r in (4, 6, 7) if r < by_rows]:
        tiles_t = (T + 16 * rt - 1) // (16 * rt)
        for d in (1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48):
            if d > 1 and (longest + d - 1) // d < 512:
                break
            target = (longest + d - 1) // d
            splits = [min((kc + target - 1) // target, max(1, kc // 512)) for _, kc, _ in jobs]
            if rt != by_rows and sum((c + 255) // 256 * tiles_t * s for (c, _, _), s in zip(jobs, splits)) > 3 * CUS:
                break
            yield d == 1, rt, splits, planner.us(jobs, splits, T, rt, grouped, single, other)


def test_no_form_over_one_with_a_lesser_estimate(planner):
    """Of the forms that meet their bound (5 % below the whole contractions in their own rows; 17 % for pieces where those are more
    than a round of workgroups), the one with the least estimate, in whatever order they are looked at."""
    rng = random.Random(7)
    shapes = [([(13184, 1536)], 571, False, True), ([(3456, 4096)], 1169, False, True), ([(14336, 512)], 530, False, True),
              ([(384, 384)] * 4 + [(1024, 384)] * 2 + [(384, 1024)], 1092, False, False)]
    for _ in range(1500):
        d = 128 * max(1, round(2 ** rng.uniform(0, 6)))
        f = 128 * round(d * rng.uniform(2.5, 3.5) / 128)
        block = [(d, d)] * 4 + [(f, d)] * 2 + [(d, f)]
        one = [(128 * rng.randint(1, 150), 128 * rng.randint(1, 100))]
        shapes.append((rng.choice([block, [(3 * d, d), (d, d), (2 * f, d), (d, f)], one]), int(2 ** rng.uniform(4.1, 12)),
                       rng.random() < 0.5, None))
    taken = {"plain": 0, "rows": 0, "pieces": 0}
    for layers, T, grouped, single in shapes:
        single = single if single is not None else len(layers) == 1
        jobs, other = _forward(layers, T), 0.0 if single else rng.choice([0.0, 500.0, 20000.0])
        forms = list(_forms(planner, jobs, T, grouped, single, other))
        unsplit = forms[0][3]
        round_1 = sum((c + 255) // 256 * ((T + 16 * forms[0][1] - 1) // (16 * forms[0][1])) for c, _, _ in jobs) <= 2 * CUS
        rows = [f for f in forms[1:] if f[0] and f[3] < 0.95 * unsplit]
        pieces = [f for f in forms[1:] if not f[0] and f[3] < (0.95 if round_1 else 0.83) * unsplit]
        want = min(rows + pieces, key=lambda f: f[3], default=forms[0])
        rt, splits = planner.plan(jobs, T, grouped, single, other=other)
        got = planner.us(jobs, splits, T, rt, grouped, single, other)
        assert got <= want[3], (layers, T, grouped, other, (rt, splits, got), want)
        assert any((rt, splits) == (f[1], f[2]) for f in rows + pieces + forms[:1]), (layers, T, grouped, rt, splits)
        taken["plain" if (rt, splits) == (forms[0][1], forms[0][2]) else "rows" if max(splits) == 1 else "pieces"] += 1
    assert min(taken.values()) > 50, taken


def _block(d, f):
    return [(d, d)] * 4 + [(f, d)] * 2 + [(d, f)]


# layers, T, group-wise, us of token tiles beside, measured: {(row tiles per tile, pieces of the longest contraction): us per call}
MEASURED = [
    (_block(3072, 7936), 458, False, 0, {(8, 1): 114.1, (8, 2): 117.8, (4, 1): 107.8, (4, 2): 110.7, (6, 1): 101.4, (6, 2): 106.2,
                                         (7, 1): 111.3, (7, 2): 116.3}),
    (_block(896, 2816), 607, True, 0, {(8, 1): 51.9, (8, 2): 35.6, (8, 4): 34.4, (8, 5): 33.2, (4, 1): 41.9, (4, 2): 31.0,
                                       (4, 3): 29.7, (4, 4): 37.8, (6, 2): 34.7, (6, 3): 33.4, (6, 4): 33.4, (7, 3): 34.8}),
    (_block(384, 1024), 1092, False, 0, {(8, 1): 26.9, (8, 2): 24.8, (7, 1): 25.3, (7, 2): 23.4, (6, 1): 23.2, (6, 2): 22.8, (4, 1): 20.0,
                                           (4, 2): 21.6}),
    (_block(1920, 6656), 566, False, 0, {(8, 1): 94.2, (8, 2): 74.5, (8, 3): 85.8, (4, 1): 70.1, (4, 3): 68.9, (6, 1): 80.6,
                                         (6, 2): 73.3, (6, 3): 73.2, (7, 2): 79.7}),
    # dX beside token contractions: 11008 x 4096, T = 500 (groups of 64) and 922 (128)
    ([(4096, 11008)], 500, True, 32 * 43 * 16.8, {(8, 1): 186.4, (8, 2): 114.7, (8, 3): 102.6, (8, 4): 106.4, (4, 1): 151.7, (4, 2): 112.2}),
    ([(4096, 11008)], 922, True, 32 * 43 * 24.5, {(8, 1): 203.3, (8, 2): 166.3, (8, 3): 171.5, (8, 4): 174.3, (6, 2): 170.9, (7, 2): 169.6}),
]


@pytest.mark.parametrize("layers,T,grouped,other,measured", MEASURED)
def test_forms_that_were_measured(planner, layers, T, grouped, other, measured):
    """Launches in which the longest workgroup shares its unit for part of its time only, in which one workgroup more than there
    are places starts a second round, or which token tiles fill: the plan is within an
    eighth of the best form measured."""
    jobs = _forward(layers, T)
    rt, splits = planner.plan(jobs, T, grouped, False, other=float(other))
    longest = max(range(len(jobs)), key=lambda j: jobs[j][1])
    assert (rt, splits[longest]) in measured, (rt, splits)
    assert measured[rt, splits[longest]] <= 1.125 * min(measured.values()), (rt, splits)


def test_block_workspace_holds_the_plan_of_dx_alone(planner):
    """A group-wise block backward that asks for dX only launches dX by itself, in the pieces of such a launch, not in those (fewer)
    that it takes beside the token contractions: the workspace holds either."""
    from paper_2305_14152_amd import peqa
    N, K, T = 3072, 6912, 260
    jobs = [(K, N, 4 * T * K)]
    alone = planner.plan(jobs, T, True, False)[1]
    beside = planner.plan(jobs, T, True, False, other=(K // 128) * (N // 256) * (0.55 * 10 + 8))[1]
    assert beside < alone
    L = peqa.layout(N, K, 4, 128)
    items = peqa.block_items([dict(L=L, packed=16, s0=16, z0=16, dY=16, dX=16)])
    need = peqa.block_workspace_bytes(items, T, peqa.PEQA_OP_BWD)
    peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 4)                   # forced forms are whole contractions
    try:
        whole = peqa.block_workspace_bytes(items, T, peqa.PEQA_OP_BWD)
    finally:
        peqa.set_option(peqa.PEQA_OPT_GEMM_WAVES, 0)
    assert need - whole >= alone[0] * 4 * T * K


def test_workgroups_that_scale_dY():
    """Multiples of 8, no more than there are row blocks, 64 to 512: many beside tiles that last no longer than the scaling, few in
    launches of many rounds.  By measurement (backward, us): d = 256, f = 640, T = 3727 130 with 64 workgroups and 51 with 512, d = 3072,
    f = 8192, T = 1024 399 and 388 with 192, d = 4096, f = 11008, T = 2048 1222 and 1231 with 192."""
    from paper_2305_14152_amd import peqa
    i, d = ctypes.c_int, ctypes.c_double
    fn = peqa.lib()._ZN4peqa11scaling_wgsEididi                    # peqa::scaling_wgs
    fn.argtypes, fn.restype = [i, d, i, d, i], i
    assert fn(1864, 6340.0, 304, 19.0, 2 * CUS) == 512
    assert fn(512, 4150.0, 992, 150.0, 2 * CUS) == 192
    assert fn(1024, 9574.0, 2656, 466.0, 2 * CUS) == 64
    assert fn(0, 0.0, 8, 20.0, 2 * CUS) == 0 and fn(3, 11.0, 8, 20.0, 2 * CUS) == 8 and fn(81, 300.0, 24, 20.0, 2 * CUS) == 88
    rng = random.Random(0)
    for _ in range(500):
        blocks, tiles, launch = rng.randint(1, 5000), rng.randint(8, 8000), rng.uniform(10, 3000)
        n = fn(blocks, rng.uniform(3, 30) * blocks, tiles, launch, 2 * CUS)
        assert n % 8 == 0 and min(64, blocks) <= n <= min(512, blocks + 7)
        assert tiles >= 8 * CUS or n >= min(192, blocks)
