"""ver_lstm_fwd / ver_lstm_bwd against the CPU oracle (unpacked, per piece,
fp64).  fp32 path: every element within 1e-4 of max(|ref|, rms(ref)).
bf16-operand path: every element within 2e-2 in the same metric, except the
tensors that come out of back-propagation through time, which have a bar of
their own (tests/util.py: assert_close_bf16_bptt)."""
import numpy as np
import pytest
import torch

from oracle import lstm as olstm, pack as opack
from paper_2210_05064_amd import workloads as wl
from tests.gpu_util import LstmRun, grads_to_list, GRAD_NAMES
from tests.util import closer, l2_rel_err, rel_err

pytestmark = pytest.mark.gpu


def oracle_run(ro, w, meta, h0, c0, d_u, d_v):
    W = olstm.weights_f64(ro["weights"])
    fwd = olstm.minibatch_forward(ro["obs"], meta["seq_first"], meta["seq_len"], W, h0, c0)
    u = olstm.to_packed([f[0] for f in fwd], meta["t_off"])
    v = olstm.to_packed([f[1] for f in fwd], meta["t_off"])
    grads = olstm.zero_grads(W)
    du_p = olstm.from_packed(d_u, meta["t_off"], meta["seq_len"])
    dv_p = olstm.from_packed(d_v, meta["t_off"], meta["seq_len"])
    dx = [olstm.piece_backward(du_p[j], dv_p[j], W, fwd[j][2], grads) for j in range(meta["n_seq"])]
    return u, v, grads, olstm.to_packed(dx, meta["t_off"])


def case(ver, w, seed, b=0, compute=0, x_bf16=False, states=True, bias_scale=0.2, layer_by_layer=False):
    ro = wl.make_rollout(w, seed=seed, bias_scale=bias_scale)
    B = w.minibatches
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], B, b, ro["env_started_episode"])
    h0 = c0 = None
    if states:
        h0 = opack.initial_states(ro["rnn_h"], meta["seq_first"], meta["seq_is_ep_start"])
        c0 = opack.initial_states(ro["rnn_c"], meta["seq_first"], meta["seq_is_ep_start"])
    rng = np.random.default_rng(seed + 1)
    M = meta["M"]
    d_u = (rng.standard_normal((M, w.act_dim)) / M).astype(np.float32)
    d_v = (rng.standard_normal(M) / M).astype(np.float32)
    x_packed = opack.gather_rows(ro["obs"], meta["gather_idx"])
    run = LstmRun(ver, w, ro["weights"], x_packed, meta, h0, c0, compute, x_bf16, layer_by_layer)
    u, v = run.forward()
    grads, d_x = run.backward(d_u, d_v)
    r_u, r_v, r_grads, r_dx = oracle_run(ro, w, meta, h0, c0, d_u, d_v)
    close = closer(compute)
    close(u, r_u, "head_out")
    close(v, r_v, "value")
    close(d_x, r_dx, "d_x")
    names = [f"layer{l}.{n}" for l in range(w.n_layers) for n in GRAD_NAMES] + ["W_a", "b_a", "w_v", "b_v"]
    for name, g, r in zip(names, grads, grads_to_list(r_grads)):
        close(g, r, name)
    return run, meta


SMALL = dict(budget=640, n_envs=12, hidden=128, input_dim=36, p_done=0.02, minibatches=2)


@pytest.mark.parametrize("compute", [0, 1])
@pytest.mark.parametrize("b", [0, 1])
def test_two_layers_ragged(ver, compute, b):
    """Several MFMA tiles in every dimension, ragged tail of single pieces,
    initial states, both minibatches (the second opens with a split piece)."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], **SMALL), seed=21, b=b, compute=compute)


@pytest.mark.parametrize("compute", [0, 1])
def test_two_layers_one_launch_per_layer(ver, compute):
    """Two-layer networks normally run both time loops in one launch; the layer-by-layer path (one layer, and the
    top layer of an odd number) is checked against the oracle on the same case through the library's diagnostic switch."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], **SMALL), seed=21, b=1, compute=compute, layer_by_layer=True)


@pytest.mark.parametrize("compute", [0, 1])
def test_two_layer_launch_matches_layer_by_layer(ver, compute):
    """Same inputs through both paths: they differ only in the order of fp32 additions in the projection
    between the layers."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=1500, n_envs=70, hidden=128, input_dim=36, p_done=0.03, minibatches=1)
    ro = wl.make_rollout(w, seed=31, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    h0 = opack.initial_states(ro["rnn_h"], meta["seq_first"], meta["seq_is_ep_start"])
    c0 = opack.initial_states(ro["rnn_c"], meta["seq_first"], meta["seq_is_ep_start"])
    rng = np.random.default_rng(2)
    d_u = (rng.standard_normal((meta["M"], w.act_dim)) / meta["M"]).astype(np.float32)
    d_v = (rng.standard_normal(meta["M"]) / meta["M"]).astype(np.float32)
    res = []
    for layer_by_layer in (False, True):
        run = LstmRun(ver, w, ro["weights"], opack.gather_rows(ro["obs"], meta["gather_idx"]), meta, h0, c0, compute,
                      layer_by_layer=layer_by_layer)
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        res.append([u, v, dx] + grads)
    for a, b in zip(*res):
        # bf16 operands: a last-bit difference in fp32 can flip the rounding of an operand (2^-9 relative)
        assert rel_err(a, b) < (1e-5 if compute == 0 else 1e-2)


@pytest.mark.parametrize("compute", [0, 1])
def test_tiny_workload(ver, compute):
    case(ver, wl.WORKLOADS["tiny"], seed=3, compute=compute)


def test_categorical_no_initial_state_bf16_input(ver):
    case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=512, n_envs=8, hidden=64, input_dim=20, p_done=0.05),
         seed=5, compute=1, x_bf16=True, states=False)


@pytest.mark.parametrize("compute", [0, 1])
def test_many_short_pieces(ver, compute):
    """More pieces than one MFMA tile holds (n_seq > 16) and T_max small."""
    case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=600, n_envs=40, hidden=64, input_dim=12, p_done=0.2,
                        minibatches=1, speed_sigma=0.3), seed=6, compute=compute)


def test_single_long_piece(ver):
    """One environment owns the minibatch: batch size 1 at every timestep."""
    case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=300, n_envs=1, hidden=64, input_dim=8, p_done=0.0,
                        minibatches=1), seed=7)


@pytest.mark.parametrize("compute", [0, 1])
def test_two_pieces_leave_a_group_empty(ver, compute):
    """Two-layer launch with fewer pieces than groups: the third group has no piece and no timestep."""
    case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=200, n_envs=2, hidden=64, input_dim=8, p_done=0.0,
                        minibatches=1, speed_sigma=1.0), seed=11, compute=compute)


@pytest.mark.parametrize("n_envs", [3000, 5000])
def test_thousands_of_pieces(ver, n_envs):
    """Two-layer launch over thousands of pieces of 2 timesteps: the plan's prefix sums run over several blocks of
    pieces (held in LDS up to 4096 pieces, in global memory beyond), a group holds more than 64 tiles of 16 pieces,
    a timestep of a group more rows than a GEMM tile."""
    _, meta = case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=2 * n_envs, n_envs=n_envs, hidden=64, input_dim=8, p_done=0.0,
                                  minibatches=1, speed_sigma=0.0), seed=12, compute=1)
    assert meta["n_seq"] >= n_envs


def test_long_and_short_pieces(ver):
    """Two-layer launch with more than 1024 timesteps (the plan's row prefix runs over several blocks of
    timesteps) and pieces of very different lengths."""
    _, meta = case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=3000, n_envs=6, hidden=64, input_dim=8, p_done=0.001,
                                  minibatches=1, speed_sigma=1.5), seed=13, compute=0)
    assert meta["T_max"] > 1024


@pytest.mark.parametrize("compute", [0, 1])
def test_more_timesteps_than_the_workers_keep_offsets_of(ver, compute):
    """Two-layer launch with more than 2048 timesteps: the workers keep the row offsets of the first 2048 in LDS and read
    the others from memory; one chunk of 8 timesteps has offsets of both."""
    _, meta = case(ver, wl.scaled(wl.WORKLOADS["nav"], budget=4500, n_envs=2, hidden=64, input_dim=8, p_done=0.0,
                                  minibatches=1, speed_sigma=0.05), seed=14, compute=compute)
    assert meta["T_max"] > 2060 and meta["batch_sizes"][2060] == 2


def test_wide_hidden_not_a_multiple_of_128(ver):
    """hidden = 576 (bf16 operands; fp32 keeps its share of W_hh in registers only up to hidden = 512): more than 32
    tiles of 16 units (workgroups of 32 units) and a contraction that does not split into whole operand blocks four
    ways: the general (not width-specialised) forms of both time loops."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=200, n_envs=5, hidden=576, input_dim=20, p_done=0.02,
                        minibatches=1), seed=17, compute=1)


@pytest.mark.parametrize("seed", range(12))
def test_two_layer_launch_random_packings(ver, seed):
    """The plan of the two-layer launch (which pieces a group runs, its chunks, the gathered rows of the workers'
    tiles) over packings of very different shape: 1 to 60 environments, 40 to 900 rows, few to many episode ends."""
    rng = np.random.default_rng(1000 + seed)
    n_envs = int(rng.integers(1, 61))
    budget = int(rng.integers(max(40, 2 * n_envs), 901))
    w = wl.scaled(wl.WORKLOADS["nav"], budget=budget, n_envs=n_envs, hidden=64, input_dim=8,
                  p_done=float(rng.choice([0.0, 0.01, 0.05, 0.3])), minibatches=1, speed_sigma=float(rng.choice([0.0, 0.5, 1.5])))
    case(ver, w, seed=50 + seed, compute=int(seed % 2))


def test_three_layers_wide_input(ver):
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=256, n_envs=6, hidden=192, input_dim=260, n_layers=3,
                        p_done=0.03, minibatches=1), seed=8)


@pytest.mark.parametrize("layer_by_layer", [False, True])
@pytest.mark.parametrize("n_layers,compute", [(3, 1), (4, 0), (5, 0)])
def test_pairs_of_layers(ver, n_layers, compute, layer_by_layer):
    """Deeper networks run two layers per launch, an odd top layer alone: one pair and a top layer, two pairs, two pairs
    and a top layer; the launch per layer on the same case."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=700, n_envs=9, hidden=128, input_dim=36, n_layers=n_layers, p_done=0.03,
                        minibatches=1), seed=9, compute=compute, layer_by_layer=layer_by_layer)


@pytest.mark.parametrize("rows,hidden,input_dim", [(32, 64, 4), (33, 64, 32), (63, 128, 68), (127, 64, 132), (129, 320, 36), (1000, 512, 516), (130, 512, 1028), (700, 512, 388)])
def test_fp32_contractions(ver, rows, hidden, input_dim):
    """Edges of the 32 x 32 and 64 x 64 tiles of the fp32 contractions (64 x 64: K-major at 1000 rows, K-minor at 388 and 1028 inputs): one to 32 K-tiles, rows and
    columns one short of and one beyond a tile, K-tiles with 4 valid k."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=rows, n_envs=max(2, rows // 25), hidden=hidden, input_dim=input_dim, p_done=0.05,
                        minibatches=1), seed=rows)


@pytest.mark.parametrize("rows,hidden,input_dim,layers,x_bf16", [
    (63, 64, 4, 1, False), (65, 64, 36, 1, True), (128, 128, 68, 2, False), (129, 192, 132, 3, True),   # 64 x 64 tiles and their edges
    (1100, 1024, 260, 1, True),    # projection in 128 x 256 tiles
    (4100, 512, 132, 1, True),     # projection in 256 x 256 tiles, last rows of tiles partly filled
    (200, 320, 644, 2, False),     # 128-row tiles in list order
    (150, 960, 932, 2, True)])     # 256-row tiles in list order
def test_bf16_contractions(ver, rows, hidden, input_dim, layers, x_bf16):
    """Tiles of the bf16 contractions at their edges; input widths that are not a multiple of 8 (the 16-byte chunk that
    straddles the end of a row); fp32 input rows, converted on the way."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=rows, n_envs=max(2, rows // 25), hidden=hidden, input_dim=input_dim, n_layers=layers,
                        p_done=0.05, minibatches=1), seed=rows, compute=1, x_bf16=x_bf16)


@pytest.mark.parametrize("rows,hidden,input_dim,layers", [(1023, 64, 36, 1), (1024, 64, 4, 1), (1025, 64, 36, 2), (1600, 128, 132, 1), (2100, 64, 260, 3)])
def test_bf16_weight_gradients_in_parts(ver, rows, hidden, input_dim, layers):
    """Weight gradients of few tiles are split over the rows from 1024 rows on: one part, two and more, the last one shorter."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=rows, n_envs=rows // 20, hidden=hidden, input_dim=input_dim, n_layers=layers,
                        p_done=0.05, minibatches=1), seed=rows, compute=1, x_bf16=True)


@pytest.mark.parametrize("rows,hidden,input_dim,layers", [(59, 64, 4092, 1), (59, 64, 4096, 1), (31, 64, 4100, 2), (33, 128, 6148, 1), (70, 320, 8196, 1), (450, 512, 8200, 1)])
def test_wide_inputs(ver, rows, hidden, input_dim, layers):
    """fp32 projections of few rows are split over the inputs from 4096 on: one part, two and more, the last one shorter; the last
    case in tiles of 64."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=rows, n_envs=max(2, rows // 20), hidden=hidden, input_dim=input_dim, n_layers=layers,
                        p_done=0.05, minibatches=1), seed=rows + input_dim)


@pytest.mark.parametrize("rows,hidden,act_dim", [(31, 64, 1), (32, 64, 15), (33, 128, 16), (65, 320, 47), (130, 64, 63)])
def test_head_gradients(ver, rows, hidden, act_dim):
    """Row blocks of the heads' weight gradients at their edges; head counts at the edges of the 16-row products."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=rows, n_envs=3, hidden=hidden, input_dim=8, act_dim=act_dim, n_layers=1, p_done=0.05,
                        minibatches=1), seed=rows)


@pytest.mark.parametrize("compute", [0, 1])
def test_fp32_rows_at_any_word(ver, compute):
    """Input rows and the input gradient that begin 4, 8 and 12 bytes behind a 16-byte boundary: bit for bit the result of
    aligned ones."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=150, n_envs=5, hidden=64, input_dim=36, n_layers=2, p_done=0.05, minibatches=1)
    ro = wl.make_rollout(w, seed=4, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    x = opack.gather_rows(ro["obs"], meta["gather_idx"])
    d_u = np.full((meta["M"], w.act_dim), 1.0 / meta["M"], np.float32)
    d_v = np.full(meta["M"], 1.0 / meta["M"], np.float32)
    res = []
    for words in range(4):
        run = LstmRun(ver, w, ro["weights"], x, meta, compute=compute)
        at = torch.zeros(x.size + words, device="cuda")[words:].view(x.shape)
        at.copy_(run.x)
        run.x = at
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        res.append([u, v, dx] + grads)
    for other in res[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(res[0], other))


def test_packing_order_invariance_on_device(ver):
    """Another random order of the same sequences (B = 1): identical weight gradients up to rounding."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=400, n_envs=10, hidden=64, input_dim=16, p_done=0.03,
                  minibatches=1, epochs=2)
    ro = wl.make_rollout(w, seed=9, bias_scale=0.2)
    rng = np.random.default_rng(1)
    du_flat = (rng.standard_normal((ro["S"], w.act_dim)) / ro["S"]).astype(np.float32)
    dv_flat = (rng.standard_normal(ro["S"]) / ro["S"]).astype(np.float32)
    outs = []
    for e in range(2):
        meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][e], 1, 0)
        g = meta["gather_idx"]
        run = LstmRun(ver, w, ro["weights"], ro["obs"][g], meta)
        u, v = run.forward()
        grads, _ = run.backward(du_flat[g], dv_flat[g])
        flat_u = np.zeros_like(u)
        flat_u[g] = u
        outs.append((flat_u, grads))
    assert rel_err(outs[0][0], outs[1][0]) < 1e-5
    for a, b in zip(outs[0][1], outs[1][1]):
        assert rel_err(a, b) < 1e-4


def test_bitwise_reproducible(ver):
    w = wl.scaled(wl.WORKLOADS["manip"], **SMALL)
    ro = wl.make_rollout(w, seed=4)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 2, 0)
    rng = np.random.default_rng(0)
    d_u = rng.standard_normal((meta["M"], w.act_dim)).astype(np.float32)
    d_v = rng.standard_normal(meta["M"]).astype(np.float32)
    res = []
    for _ in range(2):
        run = LstmRun(ver, w, ro["weights"], ro["obs"][meta["gather_idx"]], meta, compute=1)
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        res.append([u, v, dx] + grads)
    assert all(np.array_equal(a, b) for a, b in zip(*res))


def test_unsupported_shapes(ver):
    for kw in (dict(hidden=96), dict(hidden=1024), dict(input_dim=6), dict(n_layers=9)):
        c = dict(n_layers=1, input_dim=8, hidden=64, act_dim=4)
        c.update(kw)
        cfg = ver.lstm_cfg(c["n_layers"], c["input_dim"], c["hidden"], c["act_dim"], 0, 0)
        assert ver.ver_lstm_workspace_bytes(cfg, 16) == 0


@pytest.mark.parametrize("input_dim", [4, 60, 64, 68, 124, 128, 196])
def test_bf16_input_projection_any_width(ver, input_dim):
    """bf16 rows into the first layer: the projection walks the input width in tiles of 64, so widths just below,
    at and just above a multiple of 64 (and narrower than one tile), over three row tiles with a ragged last one."""
    case(ver, wl.scaled(wl.WORKLOADS["large"], budget=300, n_envs=5, hidden=64, input_dim=input_dim, p_done=0.02,
                        minibatches=1), seed=40 + input_dim, compute=1, x_bf16=True)


@pytest.mark.parametrize("input_dim,layer_by_layer", [(516, False), (1044, False), (544, False), (548, False), (1056, True),
                                                      (512, False), (640, True)])
def test_grouped_weight_gradients(ver, input_dim, layer_by_layer):
    """bf16 operands at a hidden size whose weight gradients leave in one grouped launch (4H a multiple of 1024),
    over input widths on both sides of its rules: a few columns beyond the last whole 128-column tile ride along
    with the whole tiles (4 or 20 columns beyond four whole tiles: two 16-row slices per tile; 20 or 32 beyond
    eight: one), more than 32 columns or no remainder take column tiles of their own."""
    case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=420, n_envs=9, hidden=256, input_dim=input_dim, p_done=0.02,
                        minibatches=1), seed=41, compute=1, x_bf16=True, layer_by_layer=layer_by_layer)


@pytest.mark.parametrize("compute,hidden", [(0, 64), (0, 320), (0, 512), (1, 64), (1, 320), (1, 512), (1, 704), (1, 1024)])
@pytest.mark.parametrize("n_layers,n_envs", [(1, 150), (2, 60)])
def test_forms_of_the_time_loops(ver, compute, hidden, n_layers, n_envs):
    """A group's timesteps change form with its alive pieces (forward: more than 16, 16 .. 5, 4 .. 1; backward: up to 1 or 2,
    up to 4, up to 16, more): groups that start with about 20 pieces and end with one pass through all of them, at
    widths with whole, partly filled and empty shares of the contraction."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=6 * n_envs, n_envs=n_envs, n_layers=n_layers, hidden=hidden, input_dim=20,
                  p_done=0.01, minibatches=1, speed_sigma=0.8)
    _, meta = case(ver, w, seed=17 + hidden, compute=compute, x_bf16=bool(compute))
    assert meta["n_seq"] > 16 * (8 if n_layers == 1 else 3) and meta["batch_sizes"][-1] <= 8


@pytest.mark.parametrize("compute", [0, 1])
@pytest.mark.parametrize("hidden", [64, 128, 192, 256, 320, 576])
def test_workers_hold_the_weights_several_times(ver, compute, hidden):
    """Two-layer launch at widths whose W_ih1 fits the workers 16, 8, 5, 4 and 3 times: groups of about 40 pieces, whose
    chunks several teams share (an even number of teams) or take in turn (5 and 3)."""
    if compute == 0 and hidden > 512:
        pytest.skip("fp32 holds its weights up to 512 units")
    w = wl.scaled(wl.WORKLOADS["manip"], budget=1500, n_envs=100, n_layers=2, hidden=hidden, input_dim=12, p_done=0.01,
                  minibatches=1, speed_sigma=0.6)
    _, meta = case(ver, w, seed=60 + hidden, compute=compute, x_bf16=bool(compute))
    assert meta["n_seq"] > 3 * 32


@pytest.mark.parametrize("compute,hidden", [(0, 192), (0, 384), (0, 448), (1, 192), (1, 384), (1, 448), (1, 960)])
def test_general_widths_with_many_pieces(ver, compute, hidden):
    """One layer at widths without a loop of their own, up to the most operand blocks that the general form of each
    arithmetic holds (14 of 16 in fp32, 7 of 8 and 30 of 32 in bf16), groups of 20 pieces throughout."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=640, n_envs=160, n_layers=1, hidden=hidden, input_dim=12, p_done=0.0,
                  minibatches=1, speed_sigma=0.0)
    _, meta = case(ver, w, seed=80 + hidden, compute=compute, x_bf16=bool(compute))
    assert meta["batch_sizes"][-1] > 8 * 16


@pytest.mark.parametrize("hidden,n_envs,steps", [(384, 120, 10), (512, 60, 13), (384, 900, 2)])
def test_fp32_chunks_of_many_pieces(ver, hidden, n_envs, steps):
    """Two-layer launch in fp32 whose weights two teams of workers hold: chunks of about 256 rows (6 and 8 timesteps of 40
    and 20 pieces per group), and chunks of more rows than a worker numbers at once (2 timesteps of 300 pieces)."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=steps * n_envs, n_envs=n_envs, n_layers=2, hidden=hidden, input_dim=12, p_done=0.0,
                  minibatches=1, speed_sigma=0.0)
    _, meta = case(ver, w, seed=70 + hidden, compute=0)
    assert meta["M"] >= 48 * meta["T_max"] and meta["n_seq"] > 3 * 16


@pytest.mark.parametrize("n_envs,steps", [(112, 13), (150, 9)])
def test_bf16_chunks_of_many_pieces(ver, n_envs, steps):
    """Two-layer launch in bf16 at 512 units with 90 alive pieces per timestep or more: chunks of about 192 rows (5 and 3
    timesteps of 37 and 50 pieces per group, the last chunk shorter)."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=steps * n_envs, n_envs=n_envs, n_layers=2, hidden=512, input_dim=12, p_done=0.0,
                  minibatches=1, speed_sigma=0.0)
    _, meta = case(ver, w, seed=90 + n_envs, compute=1, x_bf16=True)
    assert meta["M"] >= 90 * meta["T_max"] and meta["n_seq"] > 3 * 16


def poisoned(ver, w, seed, compute, poison):
    """Forward (and backward) runs with clean initial states and with `poison` applied to them; poison(h0, n_seq) changes
    the states in place."""
    ro = wl.make_rollout(w, seed=seed, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    clean = opack.initial_states(ro["rnn_h"], meta["seq_first"], meta["seq_is_ep_start"])
    c0 = opack.initial_states(ro["rnn_c"], meta["seq_first"], meta["seq_is_ep_start"])
    h0 = np.array(clean, np.float32)
    poison(h0, meta["n_seq"])
    x = opack.gather_rows(ro["obs"], meta["gather_idx"])
    runs = [LstmRun(ver, w, ro["weights"], x, meta, h, c0, compute) for h in (clean, h0)]
    return ro, meta, h0, c0, runs


@pytest.mark.parametrize("n_envs", [16, 72, 160])
@pytest.mark.parametrize("compute,hidden", [(0, 320), (1, 320), (1, 576), (1, 704), (1, 832), (1, 960), (1, 1024)])
def test_infinite_initial_state(ver, compute, hidden, n_envs):
    """An infinite hidden state saturates the gates and leaves finite results, in the last 64 units above all: above 512
    units they are a share of the contraction that is only partly filled at odd multiples of 64 (groups of 2, 9 and 20
    pieces: both small forms and the form for many)."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=3 * n_envs, n_envs=n_envs, n_layers=1, hidden=hidden, input_dim=8, p_done=0.0,
                  minibatches=1, speed_sigma=0.0)

    def poison(h0, n):
        for j in range(n):
            h0[0, j, hidden - 1 - (7 * j) % 64 if j % 4 else (31 * j) % hidden] = np.inf if j % 2 else -np.inf
    ro, meta, h0, c0, (_, run) = poisoned(ver, w, 5, compute, poison)
    u, v = run.forward()
    with np.errstate(over="ignore"):
        fwd = olstm.minibatch_forward(ro["obs"], meta["seq_first"], meta["seq_len"], olstm.weights_f64(ro["weights"]), h0, c0)
    close = closer(compute)
    close(u, olstm.to_packed([f[0] for f in fwd], meta["t_off"]), "head_out")
    close(v, olstm.to_packed([f[1] for f in fwd], meta["t_off"]), "value")


@pytest.mark.parametrize("n_layers,n_envs", [(1, 16), (1, 72), (1, 160), (2, 9), (2, 40), (2, 70)])
@pytest.mark.parametrize("compute,hidden", [(0, 64), (0, 320), (1, 64), (1, 576), (1, 1024)])
def test_nan_stays_in_its_piece(ver, compute, hidden, n_layers, n_envs):
    """A piece whose state is NaN (in fp32 the one whose bits mark an empty word of the exchange ring) stays NaN to its end,
    ends no wait and leaves every other piece as it was, bit by bit; the gradients it contributes to are NaN."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=5 * n_envs, n_envs=n_envs, n_layers=n_layers, hidden=hidden, input_dim=8,
                  p_done=0.0, minibatches=1, speed_sigma=0.4)
    bits = np.array([0xffffffff if compute == 0 else 0x7fc00000], np.uint32).view(np.float32)[0]
    bad = []

    def poison(h0, n):
        for j in range(0, n, 5):
            bad.append(j)
            h0[0, j, :] = bits
    _, meta, _, _, runs = poisoned(ver, w, 6, compute, poison)
    (u, v), (u_bad, v_bad) = [r.forward() for r in runs]
    rows = np.concatenate([meta["t_off"][t] + np.array([j for j in bad if j < n], int) for t, n in enumerate(meta["batch_sizes"])])
    hit = np.zeros(meta["M"], bool)
    hit[rows] = True
    assert np.isnan(u_bad[hit]).all() and np.isnan(v_bad[hit]).all()
    assert np.array_equal(u_bad[~hit], u[~hit]) and np.array_equal(v_bad[~hit], v[~hit])
    rng = np.random.default_rng(7)
    d_u, d_v = rng.standard_normal(u.shape).astype(np.float32) / meta["M"], rng.standard_normal(v.shape).astype(np.float32) / meta["M"]
    (_, dx), (grads_bad, dx_bad) = [r.backward(d_u, d_v) for r in runs]
    assert np.isnan(dx_bad[hit]).all() and np.array_equal(dx_bad[~hit], dx[~hit])
    assert np.isnan(grads_bad[1]).any()


def one_timestep(ver, rows, input_dim, compute, H=64):
    """One timestep of `rows` pieces, with plain torch in 64 bits as the reference.  fp32: a sum of n terms as P partial sums of chains of
    n / (4 P) additions is off by about 2^-24 sqrt(n / (8 P)) of its size; P = 8, and half as much again.  bf16: gate gradients
    rounded to 8 bits."""
    A = 4
    M, D, g = rows, input_dim, torch.Generator(device="cuda").manual_seed(rows)
    normal = lambda *shape, scale=1.0: torch.randn(*shape, generator=g, device="cuda").mul_(scale)
    x = normal(M, D)
    x = x.bfloat16() if compute else x
    w = [normal(4 * H, D, scale=D ** -0.5), normal(4 * H, H, scale=H ** -0.5), normal(4 * H, scale=0.1), normal(4 * H, scale=0.1),
         normal(A, H, scale=H ** -0.5), normal(A, scale=0.1), normal(H, scale=H ** -0.5), normal(1, scale=0.1)]
    if compute:
        w[0] = w[0].bfloat16().float()   # (exact in the operand type: the rounding of the weights is not what is tested)
    d_u, d_v = normal(M, A, scale=1.0 / M), normal(M, scale=1.0 / M)
    i32 = dict(dtype=torch.int32, device="cuda")
    info, bs, t_off = torch.tensor([M, 1, M, 0], **i32), torch.zeros(M, **i32), torch.full((M + 1,), M, **i32)
    bs[0], t_off[0] = M, 0
    cfg = ver.lstm_cfg(1, D, H, A, compute, compute)
    ws = ver.workspace(ver.ver_lstm_workspace_bytes(cfg, M))
    nan = lambda t: torch.full_like(t, float("nan"))
    u, v, grads, dx = nan(d_u), nan(d_v), [nan(t) for t in w], torch.full((M, D), float("nan"), device="cuda")
    ver.ver_lstm_fwd(cfg, x, M, info, bs, t_off, None, None, 0, w, u, v, ws)
    ver.ver_lstm_bwd(cfg, x, M, info, bs, t_off, None, None, 0, w, d_u, d_v, grads, dx, ws)
    torch.cuda.synchronize()
    assert ws[0].item() == 0
    W = [t.double().requires_grad_() for t in w]
    x64 = x.double().requires_grad_()
    gate_i, _, gate_g, gate_o = (x64 @ W[0].t() + (W[2] + W[3])).chunk(4, 1)
    h = torch.sigmoid(gate_o) * torch.tanh(torch.sigmoid(gate_i) * torch.tanh(gate_g))
    u64, v64 = h @ W[4].t() + W[5], h @ W[6] + W[7]
    ((u64 * d_u.double()).sum() + (v64 * d_v.double()).sum()).backward()
    off = lambda got, ref: ((got.double() - ref).norm() / ref.norm()).item()
    chain = lambda n: 1.5 * 2.0 ** -24 * (n / 64) ** 0.5
    tight, rounded = max(chain(D), 2e-6), 2.0 ** -8
    assert off(u, u64.detach()) <= tight and off(v, v64.detach()) <= tight
    assert off(grads[0], W[0].grad) <= (rounded if compute else max(chain(M), tight))
    assert off(dx, x64.grad) <= (rounded if compute else tight)
    assert off(grads[2], W[2].grad) <= (rounded if compute else 1e-5) and not grads[1].any()


@pytest.mark.parametrize("rows,input_dim,compute", [(520000, 1044, 0), (2000, 270000, 0), (1040000, 1044, 1), (4000, 270000, 1)])
def test_arrays_beyond_2_gigabytes(ver, rows, input_dim, compute):
    """Input rows and their gradient of 2 GB and more (the general contraction kernel): few tiles and a long contraction in the
    weight gradient (many rows) or in the projection (wide rows)."""
    one_timestep(ver, rows, input_dim, compute)


@pytest.mark.parametrize("rows,input_dim,hidden", [(53184, 60, 64), (53249, 60, 64), (14000, 252, 128), (3000, 252, 1024), (3000, 260, 1024), (3000, 36, 1024)])
def test_bf16_tiles_of_contractions(ver, rows, input_dim, hidden):
    """Narrow input gradients on either side of 832 tiles of 64 x 64; projections of many tiles whose contraction is shorter than
    256 and not."""
    one_timestep(ver, rows, input_dim, 1, hidden)


def even(ver, pieces, steps, layers, compute, hidden, **kw):
    """`pieces` pieces of `steps` timesteps each."""
    return case(ver, wl.scaled(wl.WORKLOADS["manip"], budget=pieces * steps, n_envs=pieces, speed_sigma=0.0, hidden=hidden, input_dim=36,
                               n_layers=layers, p_done=0.0, minibatches=1), seed=pieces + layers, compute=compute, **kw)


@pytest.mark.parametrize("pieces,steps,layers,compute,hidden", [
    (49, 17, 3, 1, 64), (50, 17, 3, 1, 64), (256, 3, 3, 1, 64), (257, 3, 3, 1, 64), (300, 3, 4, 1, 320), (900, 1, 5, 1, 128),
    (20, 30, 4, 1, 320), (16, 50, 4, 1, 1024),   # pairs above pairs
    (50, 20, 3, 0, 256), (51, 20, 3, 0, 256), (32, 40, 3, 0, 384), (33, 40, 3, 0, 384), (400, 2, 4, 0, 64), (300, 3, 5, 0, 128)])
def test_many_pieces_and_layers(ver, pieces, steps, layers, compute, hidden):
    """Three layers and more share launches in pairs up to 45 + T / 4 alive pieces per timestep (fp32 beyond 320 units: 12 + T / 2) and
    up to 768 rows; beyond, every layer runs alone: both sides of the lines, a single timestep, pairs above pairs in either form."""
    run, meta = even(ver, pieces, steps, layers, compute, hidden)
    assert meta["n_seq"] == pieces and meta["T_max"] == steps


@pytest.mark.parametrize("pieces,steps,layers,hidden", [(40, 20, 5, 128), (12, 60, 7, 64), (10, 70, 8, 192)])
def test_pairs_above_pairs_bf16(ver, pieces, steps, layers, hidden):
    """Two and more pairs, in launches of pairs and layer by layer.  Either form is up to 7e-3 from the exact gradients in the 2-norm
    (five layers 5.4e-3, seven 7.1e-3, the same in both), so that they are up to twice that from each other; from five layers on the
    largest element is beyond the oracle tests' 7e-2 in both (8.6e-2)."""
    w = wl.scaled(wl.WORKLOADS["manip"], budget=pieces * steps, n_envs=pieces, speed_sigma=0.0, hidden=hidden, input_dim=36, n_layers=layers,
                  p_done=0.0, minibatches=1)
    ro = wl.make_rollout(w, seed=layers, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    d_u, d_v = np.full((meta["M"], w.act_dim), 1.0 / meta["M"], np.float32), np.full(meta["M"], 1.0 / meta["M"], np.float32)
    res = []
    for layer_by_layer in (False, True):
        run = LstmRun(ver, w, ro["weights"], opack.gather_rows(ro["obs"], meta["gather_idx"]), meta, compute=1, layer_by_layer=layer_by_layer)
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        res.append([u, v, dx] + grads)
    for a, b in zip(*res):
        assert l2_rel_err(a, b) <= 1.4e-2


@pytest.mark.parametrize("compute", [0, 1])
def test_pairs_and_single_layers_in_one_workspace(ver, compute):
    """Minibatches of few and of many pieces in turn, in the same workspace: what either form leaves there is not taken for the
    other's.  Each as in a workspace of its own, bit for bit."""
    runs = []
    for pieces, steps in ((10, 80), (400, 2)):
        w = wl.scaled(wl.WORKLOADS["manip"], budget=800, n_envs=pieces, speed_sigma=0.0, hidden=64, input_dim=36, n_layers=3, p_done=0.0, minibatches=1)
        ro = wl.make_rollout(w, seed=5, bias_scale=0.2)
        meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
        runs.append(LstmRun(ver, w, ro["weights"], opack.gather_rows(ro["obs"], meta["gather_idx"]), meta, compute=compute))
    d_u, d_v = np.full((800, w.act_dim), 1.0 / 800, np.float32), np.full(800, 1.0 / 800, np.float32)

    def step(run):
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        return [u, v, dx] + grads
    alone = [step(run) for run in runs]
    runs[1].ws = runs[0].ws
    for _ in range(2):
        for run, ref in zip(runs, alone):
            assert all(np.array_equal(a, b) for a, b in zip(step(run), ref))


def test_conversion_of_16_giga_elements(ver):
    """fp32 input rows of a bf16 call, 2^34 elements and a few more: every row converted (equal rows, equal outputs)."""
    M, D, H, A = 2000000, 8592, 64, 2
    assert M * D > 2 ** 34
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB")
    row, w = torch.linspace(-1, 1, D, device="cuda"), [torch.full((4 * H, D), 2.0 ** -13, device="cuda"), torch.zeros(4 * H, H, device="cuda")]
    w[0][:, D // 2:] = 2.0 ** -10
    w += [torch.zeros(4 * H, device="cuda"), torch.zeros(4 * H, device="cuda"), torch.full((A, H), 0.5, device="cuda"),
          torch.zeros(A, device="cuda"), torch.full((H,), 0.25, device="cuda"), torch.zeros(1, device="cuda")]
    cfg = ver.lstm_cfg(1, D, H, A, 1, 0)
    i32 = dict(dtype=torch.int32, device="cuda")
    outs = []
    for rows in (16, M):
        x = row.expand(rows, D).contiguous()
        info, bs, t_off = torch.tensor([rows, 1, rows, 0], **i32), torch.zeros(rows, **i32), torch.full((rows + 1,), rows, **i32)
        bs[0], t_off[0] = rows, 0
        ws = ver.workspace(ver.ver_lstm_workspace_bytes(cfg, rows))
        ws.fill_(-1)
        u, v = torch.full((rows, A), float("nan"), device="cuda"), torch.full((rows,), float("nan"), device="cuda")
        ver.ver_lstm_fwd(cfg, x, rows, info, bs, t_off, None, None, 0, w, u, v, ws)
        torch.cuda.synchronize()
        assert ws[0].item() == 0
        outs.append((u, v))
        del x, ws
    torch.cuda.empty_cache()
    (u16, v16), (u, v) = outs
    assert u16.abs().min() > 1e-3
    # (another contraction kernel: sums in another order)
    assert ((u - u16[0]).abs() <= 1e-5 * u16[0].abs()).all() and ((v - v16[0]).abs() <= 1e-5 * v16[0].abs()).all()


@pytest.mark.parametrize("n_envs,layers", [(1, 1), (2, 2), (5, 2), (9, 2), (14, 2), (40, 1)])
@pytest.mark.parametrize("compute,hidden", [(0, 64), (0, 512), (1, 64), (1, 320), (1, 576)])
def test_one_to_five_pieces_per_group(ver, compute, hidden, n_envs, layers):
    """Groups that come from and go to one, two, four and five alive pieces: four lanes own a (piece, unit) up to four.
    576 units: the last slice of the contraction has half of its operand blocks (1024 units: test_forms_of_the_time_loops; over so few
    rows the largest of 4 million elements is at 7e-2 in any form)."""
    w = wl.Workload("quad", n_envs, 24 * n_envs, 0, 0, 0.9, 20, layers, hidden, 1, 3, 0.01, 1, 1, bool(compute))
    case(ver, w, seed=70 + n_envs, compute=compute, x_bf16=bool(compute))


@pytest.mark.parametrize("n_envs,steps,hidden,compute", [
    (1, 30, 64, 1), (3, 40, 320, 0), (9, 60, 64, 0), (9, 60, 512, 0), (24, 50, 320, 1), (40, 30, 128, 1)])
def test_three_layers_in_a_launch(ver, n_envs, steps, hidden, compute):
    """Ragged pieces, with and without the choice of a launch per layer, workers that hold the weights one to eight times, groups without pieces."""
    w = wl.Workload("three", n_envs, steps * n_envs, 0, 0, 0.9, 36, 3, hidden, 1, 3, 0.01, 1, 1, bool(compute))
    case(ver, w, seed=90 + n_envs, compute=compute, x_bf16=bool(compute))


@pytest.mark.parametrize("pieces,steps,compute,hidden", [(46, 12, 1, 64), (47, 12, 1, 64), (35, 10, 0, 128), (36, 10, 0, 128), (10, 20, 0, 384), (11, 20, 0, 384)])
def test_three_layers_lines(ver, pieces, steps, compute, hidden):
    """Three layers share a launch up to 46 alive pieces per timestep, fp32 30 + T / 2, from 384 units on T / 2: both sides."""
    even(ver, pieces, steps, 3, compute, hidden)


@pytest.mark.parametrize("n_envs,steps,hidden", [(5, 40, 576), (24, 50, 1024)])
def test_three_wide_layers(ver, n_envs, steps, hidden):
    """In a launch and layer by layer: either is up to 7e-3 from the exact gradients in the 2-norm (tests/util.py), so up to twice that from the other."""
    w = wl.Workload("three", n_envs, steps * n_envs, 0, 0, 0.9, 36, 3, hidden, 1, 3, 0.01, 1, 1, True)
    ro = wl.make_rollout(w, seed=n_envs, bias_scale=0.2)
    meta = opack.pack_minibatch(ro["dones"], ro["env_off"], ro["seq_key"][0], 1, 0, ro["env_started_episode"])
    rng = np.random.default_rng(n_envs)
    M = meta["M"]
    d_u, d_v = (rng.standard_normal((M, w.act_dim)) / M).astype(np.float32), (rng.standard_normal(M) / M).astype(np.float32)
    res = []
    for layer_by_layer in (False, True):
        run = LstmRun(ver, w, ro["weights"], opack.gather_rows(ro["obs"], meta["gather_idx"]), meta, compute=1, layer_by_layer=layer_by_layer)
        u, v = run.forward()
        grads, dx = run.backward(d_u, d_v)
        res.append([u, v, dx] + grads)
    for a, b in zip(*res):
        assert l2_rel_err(a, b) <= 1.4e-2


@pytest.mark.parametrize("pieces,steps,layers", [(136, 5, 1), (267, 4, 1), (53, 12, 2), (100, 2, 2)])
@pytest.mark.parametrize("compute,hidden", [(0, 192), (0, 512), (1, 64), (1, 576)])
def test_tiles_of_16_pieces(ver, pieces, steps, layers, compute, hidden):
    """17, 33, 34 alive pieces in a group until its last timestep: two tiles and three, the last with one or two pieces."""
    even(ver, pieces, steps, layers, compute, hidden)


@pytest.mark.parametrize("pieces,steps,layers", [(136, 24, 1), (267, 25, 1), (76, 26, 2), (150, 24, 2)])
@pytest.mark.parametrize("compute,hidden", [(0, 320), (0, 512), (1, 64), (1, 192), (1, 512), (1, 576)])
def test_tiles_of_16_pieces_backward(ver, pieces, steps, layers, compute, hidden):
    """The same from the 24 timesteps on that the backward loop asks for: 17, 25, 33, 34, 50 alive pieces in a group."""
    even(ver, pieces, steps, layers, compute, hidden)


def test_tiles_of_16_pieces_of_256(ver):
    """257 pieces in four of the groups and 256 in the others, the most that the backward loop takes 16 at a time."""
    even(ver, 2052, 24, 1, 1, 192)


@pytest.mark.parametrize("layers", [1, 2])
@pytest.mark.parametrize("compute,hidden", [(0, 512), (1, 64), (1, 320), (1, 576)])
def test_tiles_of_16_pieces_ragged(ver, layers, compute, hidden):
    """Groups with more than 16 pieces in their first timesteps and few in their last, pieces that end in between."""
    n_envs = 260 // (layers * layers)
    w = wl.Workload("tiles", n_envs, 40 * n_envs, 0, 0, 0.9, 60, layers, hidden, 1, 3, 0.02, 1, 1, bool(compute))
    case(ver, w, seed=120 + layers, compute=compute, x_bf16=bool(compute))
