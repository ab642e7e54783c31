"""The flop counts the benchmark's rooflines divide by, checked against an operation-counting
run of the arithmetic they describe (CPU only).

pair_dft_flops(L): an L-point complex DFT with the terms r, L - r and the outputs om, L - om
taken in conjugate pairs.  The counting version below performs exactly that arithmetic on
Python complex numbers, tallies its real adds and FMAs (an FMA counts 2), and must also
reproduce the plain DFT sum_r b[r] w^(om r)."""
import json

import numpy as np
import pytest

import bench


class Tally:
    def __init__(self):
        self.flops = 0

    def add(self, a, b):          # complex add: 2 real adds
        self.flops += 2
        return a + b

    def sub(self, a, b):
        self.flops += 2
        return a - b

    def fma_real(self, a, s, c):  # complex a times real s plus complex c: 2 real FMAs
        self.flops += 4
        return a * s + c


def paired_dft(b, w, L, t):
    M, ev = (L - 1) // 2, L % 2 == 0
    u = {r: t.add(b[r], b[L - r]) for r in range(1, M + 1)}
    d = {r: t.sub(b[r], b[L - r]) for r in range(1, M + 1)}
    f0 = b[0]
    for r in range(1, M + 1):
        f0 = t.add(f0, u[r])
    if ev:
        f0 = t.add(f0, b[L // 2])
    F = [0j] * L
    F[0] = f0
    for om in range(1, M + 1):
        P, Q = b[0], 0j
        for r in range(1, M + 1):
            k = (om * r) % L
            P = t.fma_real(u[r], w[k].real, P)
            Q = t.fma_real(d[r], w[k].imag, Q)
        if ev:
            P = t.fma_real(b[L // 2], -1.0 if om & 1 else 1.0, P)
        F[om] = t.add(P, 1j * Q)       # (P.x - Q.y, P.y + Q.x): 2 real adds
        F[L - om] = t.sub(P, 1j * Q)
    if ev:
        fh = b[0]
        for r in range(1, M + 1):
            fh = t.fma_real(u[r], -1.0 if r & 1 else 1.0, fh)
        F[L // 2] = t.fma_real(b[L // 2], -1.0 if (L // 2) & 1 else 1.0, fh)
    return np.array(F)


@pytest.mark.parametrize("L", range(2, 8))
@pytest.mark.parametrize("sign", [-1, 1])
def test_pair_dft_count_and_value(L, sign):
    rng = np.random.default_rng(L)
    b = rng.standard_normal(L) + 1j * rng.standard_normal(L)
    w = np.exp(sign * 2j * np.pi * np.arange(L) / L)
    t = Tally()
    got = paired_dft(list(b), w, L, t)
    ref = np.array([sum(b[r] * w[(om * r) % L] for r in range(L)) for om in range(L)])
    assert np.abs(got - ref).max() <= 1e-12
    assert t.flops == bench.pair_dft_flops(L)


def test_flop_counts_per_voxel():
    # paper's cube: 4hL + h x-DFTs of 52 flops + 13 y rows (rows 3, 4 of mu = 0 skipped), each
    # a DFT (52), 5 magnitudes (20), 2 pair sums, 3 weight groups (18) and the row factor (6)
    assert bench.gen_flops_per_voxel(5) == 4 * 3 * 5 + 3 * 52 + 13 * (52 + 20 + 2 + 18 + 6) == 1490
    assert bench.dft_flops_per_voxel(5) == 3660
    assert bench.slide_flops_per_voxel(16) == 53760 and bench.slide_flops_per_voxel(8) == 6784
    assert bench.dft_flops_per_voxel(16) == 313920 and bench.dft_flops_per_voxel(8) == 23200


def slide_products(p, L, R, q, t):
    """p w^(kt v) for every kt, v = 4q + R, as the sliding kernel forms them: a few products of the
    plane bin p, then quarter turns (swaps and signs, no flops)."""
    w = [np.exp(-2j * np.pi * k / L) for k in range(L)]
    i8 = np.exp(-2j * np.pi / 8)
    Q = {0: p}

    def mul(c, flops):
        t.flops += flops
        return p * c

    if L == 16:
        if R == 0:
            Q.update({b: p for b in (1, 2, 3)})
        elif R == 2:
            p2 = mul(i8, 5)               # one product shared by two FMAs
            Q.update({1: p2, 2: -1j * p, 3: -1j * p2})
        else:
            p2 = mul(i8, 5)
            z1, z3 = mul(w[1], 5), mul(w[3], 5)   # two products shared by four FMAs
            Q.update({1: z1, 2: p2, 3: z3} if R == 1 else {1: z3, 2: -1j * p2, 3: -z1})
        NB = 4
    else:
        p2 = mul(i8, 5) if R % 2 else p
        Q[1] = (p2 if R == 1 else -1j * p2) if R % 2 else (-1j) ** (R // 2) * p
        NB = 2
    turn = {0: 1, 1: (-1j) ** q, 2: (-1) ** q, 3: (-1) ** q * (-1j) ** q} if L == 16 else {0: 1, 1: (-1) ** q}
    return [(-1j) ** ((kt // NB) * R) * turn[kt % NB] * Q[kt % NB] for kt in range(L)]


@pytest.mark.parametrize("L", [8, 16])
def test_slide_products_count_and_value(L):
    want = {16: (0, 15, 5, 15), 8: (0, 5, 0, 5)}[L]
    for v in range(L):
        t, p = Tally(), complex(0.3 + v, -1.7)
        got = slide_products(p, L, v % 4, v // 4, t)
        assert np.abs(np.array(got) - p * np.exp(-2j * np.pi * (np.arange(L) * v % L) / L)).max() <= 1e-14
        assert t.flops == want[v % 4]


@pytest.mark.parametrize("L", [8, 16])
def test_slide_kernel_flops(L):
    """The count, from the slots a lane holds: M tiles mt of 8 ky, two ky a lane and tile (q), L kt."""
    h, MT, lanes = L // 2 + 1, L // 8, 4 * (L // 2)     # lanes of one window: groups x columns
    seen, sums = set(), 0
    for p in range(h):
        kts = (p,) if p in (0, L // 2) else (p, L - p)
        for q in range(2):                              # first tile: a weight set per ky
            seen |= {(0, q, kt) for kt in kts}
            sums += len(kts) - 1 + 3 * 2
        for mt in range(1, MT):                         # others: ky and -ky share theirs
            seen |= {(mt, q, kt) for q in range(2) for kt in kts}
            sums += 2 * len(kts) - 1 + 3 * 2
    assert len(seen) == 2 * MT * L                      # every slot once
    bins, plane = L ** 3 // 2, L * L // 2
    assert lanes * len(seen) == bins
    t = Tally()
    for v in range(4):
        slide_products(1.0 + 0j, L, v, 0, t)
    products = t.flops * plane // 4
    dfts = 2 * L * L + 8 * L * L * (L // 2)
    # a stored bin: two additions, four for the magnitude (the square root as one)
    assert bench.slide_kernel_flops_per_voxel(L) == dfts + products + 2 * bins + 4 * bins + lanes * sums
    assert bench.slide_kernel_flops_per_voxel(L) == {16: 36672, 8: 4848}[L]


def test_printed_line_is_short():
    """The printed line keeps the contract's keys and stays short enough to be kept whole, however
    long the record is."""
    roof = {"bound": "alu", "achieved": 60.123456789, "peak": 78.6, "unit": "TFLOP/s", "frac": 0.76543210987, "traffic": None,
            "kernel": "k", "flops_convention": "x" * 600}
    form = {"voxels_per_s": 1.23456789e9, "ms_per_step": 3.3, "roofline": roof, "max_rel_err_vs_oracle": {"E": 1.23456789e-7}}
    contract = {"metric": bench.METRIC, "value": 1616551363.8330588, "unit": "voxels/s", "n_gpus": 1, "steps": 20, "warmup": 5,
                "ms_per_step": 332.10878665000007, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
                "dtype": "f32", "data": "synthetic", "config": {"workload": "w", "L": 16}}
    table = {"maps": {"L8_fp32": {m: {"max": 2e-7 + i * 1e-7, "mean": 1e-8} for i, m in enumerate(
        ("E_t", "E_x", "E_y", "S_t", "S_x", "S_y", "S"))}}}
    rec = dict(contract, max_rel_err_vs_oracle={"E": 2.123456e-7}, roofline=roof, forms={"a": form}, legs={}, streamed=None,
               precision_table=table, cpu_baseline={"value": 48560.123456, "sample": "text"})
    out = bench.compact(rec)
    assert {k: out[k] for k in contract} == contract
    assert out["roofline"] == {"bound": "alu", "achieved": 60.12, "peak": 78.6, "unit": "TFLOP/s", "frac": 0.7654,
                               "traffic": None, "kernel": "k"}
    assert out["forms"]["a"]["voxels_per_s"] == 1.235e9 and out["forms"]["a"]["roofline"]["frac"] == 0.7654
    assert out["precision_table"] == {"L8_fp32": [4e-7, 7e-7, 8e-7]}
    for n in (30, 300):
        rec["forms"] = {"f%d" % i: form for i in range(n)}
        rec["legs"] = {"l%d" % i: dict(form, forms=rec["forms"]) for i in range(3)}
        out = bench.compact(rec)
        assert len(json.dumps(out)) <= bench.LINE_LIMIT and {k: out[k] for k in contract} == contract


def test_counter_records_cover_the_kernel():
    """A committed counter record counts as long as nothing the kernel is made of changes: helpers,
    structs and constants in its file and the shared headers, not comments, launchers or others'."""
    used = bench.kernel_definitions("k_energy_slide")
    assert {"k_energy_slide", "products", "take", "quarter", "group_sums", "SlideGeo", "box_tile", "refl_idx", "mfma4"} <= set(used)
    assert {"TileCfg", "Geo", "box_tile"} <= set(bench.kernel_definitions("k_energy_f32"))
    assert {"gelu_f", "FPW", "conv_fu"} <= set(bench.kernel_definitions("k_conv3"))
    assert not {"k_dcs_axis", "launch_slide_L", "batch_per_box", "launch_energy_slide"} & set(used)
    before = bench.kernel_source_hash("k_energy_slide")

    def edited(name, old, new):
        def read(f):
            src = bench._read_source(f)
            if f == name:
                assert old in src
                src = src.replace(old, new)
            return src
        return bench.kernel_source_hash("k_energy_slide", read)

    f = "sal_energy_slide.hip"
    assert edited(f, "const float a = p.y * H;", "const float a = p.y * H + 0.f;") != before
    assert edited("sal_device.h", "u = u < 0 ? -u : u;", "u = u < 0 ? 0 : u;") != before
    assert edited(f, "constexpr int STY = 16", "constexpr int STY = 32") != before
    assert edited(f, "// (x, y) as a complex number times (-i)^K", "// another comment") == before
    assert edited(f, "while (np < 8 &&", "while (np < 4 &&") == before
    assert edited("sal_device.h", "int opaque(int v)", "int opaque(int u)") == before

