"""Which launches the time loops of three layers and more run in: chosen on the device by alive pieces and timesteps, above some rows.  A launch
of several layers multiplies the rows between the layers in other kernels than a launch per layer, so that some bit of its results
differs: that tells the forms apart."""
import numpy as np
import pytest

from oracle import pack as opack
from paper_2210_05064_amd import workloads as wl
from tests.gpu_util import LstmRun
from tests.test_gpu_lstm import case

pytestmark = pytest.mark.gpu


def shape(pieces, steps, layers, compute, hidden):
    w = wl.scaled(wl.WORKLOADS["manip"], budget=pieces * steps, n_envs=pieces, speed_sigma=0.0, hidden=hidden, input_dim=36, n_layers=layers, p_done=0.0,
                  minibatches=1)
    return w, dict(seed=pieces + layers, compute=compute)


def layer_by_layer(ver, w, seed, compute):
    """Whether every layer ran alone: the same bits as with the switch that asks for that."""
    ro = wl.make_rollout(w, seed=seed, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    x, M = opack.gather_rows(ro["obs"], meta["gather_idx"]), meta["M"]
    rng = np.random.default_rng(seed)
    d_u, d_v = (rng.standard_normal((M, w.act_dim)) / M).astype(np.float32), (rng.standard_normal(M) / M).astype(np.float32)
    out = []
    for switch in (False, True):
        run = LstmRun(ver, w, ro["weights"], x, meta, compute=compute, layer_by_layer=switch)
        u, v = run.forward()
        out.append([u, v, run.backward(d_u, d_v)[1]])
    return all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("pieces,steps,layers,compute,hidden,alone", [
    # four layers and five, bf16: 45 + T / 4 pieces, more than 768 rows
    (49, 17, 4, 1, 64, False), (50, 17, 4, 1, 64, True), (256, 3, 4, 1, 64, False), (257, 3, 4, 1, 64, True), (49, 17, 5, 1, 64, False), (257, 3, 5, 1, 64, True),
    # fp32: the same up to 320 units, beyond 12 + T / 2
    (50, 20, 4, 0, 256, False), (51, 20, 4, 0, 256, True), (32, 40, 4, 0, 384, False), (33, 40, 4, 0, 384, True)])
def test_lines_of_pairs(ver, pieces, steps, layers, compute, hidden, alone):
    w, how = shape(pieces, steps, layers, compute, hidden)
    assert layer_by_layer(ver, w, **how) == alone
    if compute == 0 or layers == 4:
        case(ver, w, **how)


@pytest.mark.parametrize("pieces,steps,compute,hidden,alone", [
    # up to 256 units, bf16: three in a launch up to 64 pieces, else as pairs
    (64, 13, 1, 64, False), (65, 13, 1, 64, True), (65, 11, 1, 64, False), (128, 4, 1, 128, False), (171, 3, 1, 128, False), (257, 3, 1, 128, True),
    # above: up to 32, else the two lower layers up to 45 + T / 4
    (32, 25, 1, 384, False), (33, 25, 1, 384, False), (51, 25, 1, 384, False), (52, 25, 1, 384, True),
    # 320 units: from 17 pieces on from 24 timesteps on, 128 rows
    (17, 7, 1, 320, False), (18, 23, 1, 320, False), (18, 24, 1, 320, False), (58, 50, 1, 320, True),
    # fp32 up to 256 units: 16 pieces, 40 from 20 timesteps on, 64 from 20 (up to 128 units) or 40 on
    (16, 9, 0, 128, False), (17, 19, 0, 128, False), (40, 20, 0, 256, False), (41, 20, 0, 256, False), (64, 20, 0, 64, False), (65, 20, 0, 64, True),
    # above: 2 T >= 16 + 3 pieces, 64 rows; else the two lower layers up to 45 + T / 4 (320 units) or 12 + T / 2
    (8, 8, 0, 384, False), (8, 20, 0, 384, False), (8, 19, 0, 384, False), (33, 42, 0, 384, False), (34, 42, 0, 384, True), (33, 42, 0, 320, False)])
def test_lines_of_three_layers(ver, pieces, steps, compute, hidden, alone):
    w, how = shape(pieces, steps, 3, compute, hidden)
    assert layer_by_layer(ver, w, **how) == alone
    case(ver, w, **how)
