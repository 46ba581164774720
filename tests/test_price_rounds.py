"""The start of the exact solver at M = 8 and 16 (smoothed price rounds), emulated in numpy with the constants of the device
code: how many pruned entries its choice leaves in the wrong row, on blocks of several kinds.  Each of them is a search to
come, so a schedule that stops working on a kind of blocks shows here and not in the masks, which stay optimal."""
import os
import re

import numpy as np
import pytest

SOURCE = open(os.path.join(os.path.dirname(__file__), "..", "paper_2102_08124_amd", "csrc", "tmask_solvers.hpp")).read()


def _schedule(M):
    body = re.search(r"struct PriceSchedule<%d> \{(.*?)\n\};" % M, SOURCE, re.S).group(1)
    return {k: float(v) for k, v in re.findall(r"(\w+) = ([\d.]+)f?[,;]", body)}


def _constant(pattern):
    return np.float32(re.search(pattern, SOURCE).group(1))


def _costs(a, M):
    bits = 26 if M == 16 else 27
    exponent = np.frexp(np.maximum(a.max(axis=(1, 2), keepdims=True), np.float32(1e-30)))[1]
    return np.floor(np.ldexp(a.astype(np.float64), bits - exponent)).astype(np.int64), bits


def _choose(cost, price, K, M, bits):
    i = np.arange(M)
    key = ((cost + price[:, :, None] + (1 << (bits - 1))) << 4) | ((i[:, None] - i[None, :]) & (M - 1))
    return key < np.partition(key, K, axis=1)[:, K, None, :]


def _excess(x, K):
    return np.maximum(x.sum(axis=2) - K, 0).sum(axis=1)


def left_over(a, K):
    """Excess that the start leaves in each block; a: (blocks, M, M) magnitudes, fp32."""
    f32 = np.float32
    M = a.shape[1]
    s = _schedule(M)
    cost, bits = _costs(a, M)
    c = cost.astype(f32)                                             # exact: 24 significant bits
    mean = c.mean(axis=(1, 2), dtype=f32)[:, None]
    dev = mean - c.mean(axis=2, dtype=f32)
    level = c + dev[:, :, None]
    spread = np.abs(level[:, :M // 2] - level[:, M // 2:]).mean(axis=(1, 2), dtype=f32)[:, None]
    with np.errstate(divide="ignore", invalid="ignore"):
        chance = _constant(r"chance = ([\d.]+)f \* spread") * spread * f32(np.sqrt(M / 2)) / np.abs(dev).sum(axis=1)[:, None]
    part = f32(1) - _constant(r"part = 1\.f - ([\d.]+)f") * np.where(chance < 1, chance, f32(1))
    unit = np.maximum(np.minimum(_constant(r"unit = ([\d.]+)f \* spread") * spread, mean), f32(1))
    offset = f32(1 << bits)
    price, velocity = offset + part * dev, np.zeros_like(dev)
    slope, step = -(1 / f32(s["window"])) / unit, f32(s["step"]) * unit
    drift, drift_velocity = np.zeros_like(unit), np.zeros_like(unit)
    for _ in range(int(s["rounds"])):
        key = price[:, :, None] + c
        sel = np.partition(key, (K - 1, K), axis=1)
        middle = sel[:, K - 1] + sel[:, K]
        f = np.clip(key * slope[:, :, None] + (f32(0.5) - f32(0.5) * slope * middle)[:, None, :], 0, 1).sum(axis=2, dtype=f32)
        velocity = f32(s["momentum"]) * velocity + step * f
        price = price + velocity
        drift_velocity = f32(s["momentum"]) * drift_velocity + step * f32(K)
        drift = drift + drift_velocity
        slope, step = slope * f32(1 / s["window_next"]), step * f32(s["step_next"])
    top = 1 << (bits - 1)
    final = np.clip(price - drift - (offset - f32(top)), 1, (1 << bits) - 1 - 64).astype(np.int64) - top
    e = _excess(_choose(cost, final, K, M, bits), K)
    plain = _excess(_choose(cost, np.zeros_like(final), K, M, bits), K)
    return np.where(e > 2, np.minimum(e, plain), e)                  # the choice without prices, where many are left


def _blocks(kind, M, n):
    rng = np.random.default_rng(910 + M)
    x = rng.standard_normal((n, M, M))
    row, col = rng.standard_normal((n, M, 1)), rng.standard_normal((n, 1, M))
    i = np.arange(M)
    x = {"normal": lambda: x, "laplace": lambda: rng.laplace(size=x.shape), "t2": lambda: rng.standard_t(2, size=x.shape),
         "uniform": lambda: rng.random(x.shape), "rows scaled": lambda: x * np.exp(row), "columns scaled": lambda: x * np.exp(col),
         "columns alike": lambda: np.abs(row) + 0.01 * np.abs(x), "rows alike": lambda: np.abs(col) + 0.01 * np.abs(x),
         "columns alike 0.1": lambda: np.abs(row) + 0.1 * np.abs(x), "rows alike 0.1": lambda: np.abs(col) + 0.1 * np.abs(x),
         "ramp": lambda: np.broadcast_to(i[:, None] * M + i[None, :] + 1.0, x.shape), "equal": lambda: np.ones_like(x),
         "distance": lambda: np.abs(i[:, None] - i[None, :]) + 1 + 0.01 * x,
         "zeros 0.3": lambda: np.where(rng.random(x.shape) < 0.3, 0, x), "zeros 0.9": lambda: np.where(rng.random(x.shape) < 0.9, 0, x),
         "zero": lambda: np.zeros_like(x)}[kind]()
    return np.abs(x).astype(np.float32)


# mean excess per block; 1.2 to 2 times what the present schedule leaves.  In brackets: with windows and steps in multiples
# of the mean alone, from prices of three quarters of the row means
@pytest.mark.parametrize("kind,at8,at16", [
    ("normal", 0.04, 0.10), ("laplace", 0.05, 0.11), ("t2", 0.15, 0.20), ("uniform", 0.05, 0.09), ("rows scaled", 0.20, 0.40),
    ("columns scaled", 0.11, 0.22),
    ("columns alike", 0.9, 3.3),                     # (12.8, 47)
    ("columns alike 0.1", 0.4, 1.3),                 # (2.0, 3.8)
    ("rows alike", 0.05, 0.12),                      # (4.3, 12.4)
    ("rows alike 0.1", 0.05, 0.12),                  # (1.5, 2.6)
    ("ramp", 0.0, 0.0),                              # (16, 64)
    ("distance", 0.0, 0.0), ("equal", 0.0, 0.0), ("zero", 0.0, 0.0), ("zeros 0.3", 0.24, 0.5), ("zeros 0.9", 2.5, 7.5)])
def test_excess_left_by_the_start(kind, at8, at16):
    for M, n, most in ((8, 2000, at8), (16, 500, at16)):
        e = left_over(_blocks(kind, M, n), M // 2)
        assert e.mean() <= most, (M, e.mean())
        assert e.max() <= M * M // 4                                 # what one column pattern for all leaves


@pytest.mark.parametrize("M,K", [(8, 1), (8, 2), (8, 7), (16, 1), (16, 4), (16, 15)])
def test_any_number_of_pruned_entries(M, K):
    for kind, most in (("normal", 0.42 if K == 15 else 0.14), ("rows alike", 0.3), ("equal", 0.0)):
        e = left_over(_blocks(kind, M, 400), K)
        assert e.mean() <= most, (kind, e.mean())
