"""The work a user of this package has it do, as measurable cases.

A learner calls the package once per rollout (bucketing of the collection buffer, advantages and importance
weights, the index arrays of all minibatches) and once per minibatch (gathers, LSTM forward, PPO loss, LSTM
backward, optimiser step).  The cases are those calls, each through its entry point, over the sizes from the
smallest configuration (59 steps, one layer of 64 units) to rollouts far above the largest one, and one whole
update.  Sizes are those of the package's own configurations or generic; `draw` gives others of the same ranges.

Inputs follow the package's recipe for synthetic rollouts: log-normal environment speeds, Bernoulli episode
ends, normal observations and recurrent states, Xavier-uniform weights.
"""
import math

import numpy as np
import torch

from paper_2210_05064_amd import binding as ver
from paper_2210_05064_amd import workloads
from paper_2210_05064_amd.learner import Learner

GAMMA, LAM, CLIP, VALUE_COEF, ENTROPY_COEF, MAX_IS = 0.99, 0.95, 0.2, 0.5, 1e-4, 1.0
LR0, BETA1, BETA2, EPS, SCHEDULE, MAX_NORM = 2.5e-4, 0.9, 0.999, 1e-8, 100000, 0.5


def listed():
    return [
        # Advantages and importance weights of one rollout at the paper's size (16 environments x 128 steps):
        # the smallest call of an update, all latency.
        dict(name="targets_nav", op="targets", S=2048, N=16, sigma=0.5, p_done=0.002),
        # The same for a rollout of a massively parallel simulator; neither count is a round number.
        dict(name="targets_huge", op="targets", S=13421773, N=104857, sigma=1.0, p_done=0.005),
        # Bucketing of the collection buffer at the largest configuration: ids sorted, every per-step field moved.
        dict(name="ingest_max", op="ingest", S=32768, N=256, sigma=1.0, D=1044, H=1024, layers=2, act=11, epochs=4),
        # Index arrays and gathers of one epoch of the 64-environment configuration (four minibatches, bf16 rows).
        dict(name="pack_large", op="pack", S=8192, N=64, sigma=0.75, p_done=0.002, B=4, D=516, H=512, layers=2, act=0, x_bf16=True),
        # PPO loss and gradient, 11 Gaussian actions, over a large odd number of rows.
        dict(name="loss_gauss_big", op="loss", M=1000003, act=11, dist=1),
        # Optimiser step over the 2 x 1024 policy's 17 million parameters with gradient clipping.
        dict(name="adam_max", op="adam", D=1044, H=1024, layers=2, act=11),
        # Forward and backward of the smallest policy (one layer of 64 units, 59 rows, fp32): all launches and steps.
        dict(name="lstm_tiny", op="lstm", layers=1, H=64, D=32, act=4, M=59, N=4, sigma=0.3, p_done=0.05,
             compute=0, x_bf16=False, backward=True, dx=False),
        # A minibatch of the navigation configuration, fp32, with the input gradient a visual encoder needs.
        dict(name="lstm_nav", op="lstm", layers=2, H=512, D=516, act=4, M=1024, N=8, sigma=0.5, p_done=0.002,
             compute=0, x_bf16=False, backward=True, dx=True),
        # A deeper policy of uncommon width on an odd number of rows; observations stay fp32, contractions in bf16.
        dict(name="lstm_deep", op="lstm", layers=3, H=320, D=132, act=11, M=3001, N=24, sigma=0.75, p_done=0.005,
             compute=1, x_bf16=False, backward=True, dx=True),
        # A minibatch of the largest configuration: the call that dominates training.
        dict(name="lstm_max", op="lstm", layers=2, H=1024, D=1044, act=11, M=8192, N=64, sigma=1.0, p_done=0.005,
             compute=1, x_bf16=True, backward=True, dx=False),
        # Evaluation of a whole rollout of the largest configuration (collection log-probabilities): forward only.
        dict(name="lstm_eval_max", op="lstm", layers=2, H=1024, D=1044, act=11, M=32768, N=256, sigma=1.0, p_done=0.005,
             compute=1, x_bf16=True, backward=False, dx=False),
        # One whole update of the 64-environment configuration, from the collection buffer to the new weights.
        dict(name="update_large", op="update", S=8192, N=64, sigma=0.75, D=516, layers=2, H=512, dist=0, act=4,
             p_done=0.002, epochs=2, B=4, bf16=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    top = max(work(c)["flops"] for c in listed())
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= top:
            return c


def _draw(rng):
    op = rng.choice(["targets", "ingest", "pack", "loss", "adam", "lstm", "lstm", "lstm", "lstm", "update"])
    sigma, p_done = rng.choice([0.5, 0.75, 1.0]), rng.choice([0.002, 0.005, 0.05])
    if op == "targets":
        S = _log_int(rng, 500, 13000000)
        return dict(op=op, S=S, N=max(1, S // _log_int(rng, 16, 512)), sigma=sigma, p_done=p_done)
    if op == "ingest":
        S = _log_int(rng, 500, 32768)
        return dict(op=op, S=S, N=max(1, S // _log_int(rng, 16, 512)), sigma=sigma, D=4 * rng.randint(8, 261),
                    H=64 * rng.randint(1, 16), layers=rng.randint(1, 2), act=rng.choice([0, 7, 11]), epochs=rng.randint(1, 4))
    if op == "pack":
        B = rng.randint(1, 4)
        S = B * _log_int(rng, 100, 4096)
        return dict(op=op, S=S, N=max(1, S // _log_int(rng, 16, 512)), sigma=sigma, p_done=p_done, B=B, D=4 * rng.randint(8, 261),
                    H=64 * rng.randint(1, 16), layers=rng.randint(1, 2), act=rng.choice([0, 7, 11]), x_bf16=rng.random() < 0.5)
    if op == "loss":
        return dict(op=op, M=_log_int(rng, 59, 1000000), act=rng.choice([2, 4, 6, 7, 11, 18]), dist=rng.randint(0, 1))
    if op == "adam":
        return dict(op=op, D=4 * rng.randint(8, 261), H=64 * rng.randint(1, 16), layers=rng.randint(1, 3), act=rng.choice([4, 7, 11]))
    if op == "update":
        B = rng.randint(1, 4)
        bf16 = rng.random() < 0.5
        S = B * _log_int(rng, 64, 2048 if bf16 else 1024)
        return dict(op=op, S=S, N=max(1, S // rng.randint(64, 160)), sigma=sigma, D=4 * rng.randint(8, 133), layers=rng.randint(1, 2),
                    H=64 * rng.randint(1, 8), dist=rng.randint(0, 1), act=rng.choice([4, 7, 11]), p_done=p_done,
                    epochs=rng.randint(1, 2), B=B, bf16=bf16)
    compute = rng.randint(0, 1)
    M = _log_int(rng, 59, 8192 if compute else 2048)
    return dict(op=op, layers=rng.choice([1, 2, 2, 2, 3]), H=64 * rng.randint(1, 16 if compute else 8), D=4 * rng.randint(8, 261),
                act=rng.choice([4, 7, 11]), M=M, N=max(1, M // rng.randint(64, 160)), sigma=sigma, p_done=p_done, compute=compute,
                x_bf16=bool(compute) and rng.random() < 0.7, backward=rng.random() < 0.75, dx=rng.random() < 0.5)


# ---- inputs (plain torch and numpy) ---------------------------------------------------------------------------

class _Rand:
    def __init__(self, seed):
        self.np = np.random.default_rng(seed)
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda").mul_(scale)

    def uniform(self, *shape, bound=1.0):
        return torch.rand(*shape, generator=self.g, device="cuda").mul_(2.0).sub_(1.0).mul_(bound)

    def bits(self, *shape):
        return torch.randint(-2 ** 31, 2 ** 31, shape, generator=self.g, device="cuda", dtype=torch.int64).to(torch.int32)

    def actions(self, rows, act):
        """act > 0: that many Gaussian actions; 0: categorical over four (int32)."""
        if act > 0:
            return self.normal(rows, act)
        return torch.randint(0, 4, (rows,), generator=self.g, device="cuda", dtype=torch.int64).to(torch.int32)

    def dones(self, n, p):
        return (torch.rand(n, generator=self.g, device="cuda") < p).to(torch.uint8)


def _offsets(rnd, S, N, sigma):
    """Exclusive prefix sums of N ragged stretches that add up to S (a very slow environment may have none)."""
    speed = rnd.np.lognormal(0.0, sigma, size=N)
    off = np.zeros(N + 1, np.int64)
    off[1:] = np.floor(np.cumsum(speed) / speed.sum() * S + 0.5)
    off[N] = S
    return np.minimum(off, S)


def _weights(rnd, D, H, layers, act):
    """Flat list in the order of the C ABI: per layer W_ih, W_hh, b_ih, b_hh, then W_a, b_a, w_v, b_v."""
    out = []
    for l in range(layers):
        d = D if l == 0 else H
        out += [rnd.uniform(4 * H, d, bound=math.sqrt(6.0 / (4 * H + d))), rnd.uniform(4 * H, H, bound=math.sqrt(6.0 / (5 * H))),
                rnd.normal(4 * H, scale=0.1), rnd.normal(4 * H, scale=0.1)]
    return out + [rnd.uniform(act, H, bound=math.sqrt(6.0 / (act + H))), rnd.normal(act, scale=0.1),
                  rnd.uniform(H, bound=math.sqrt(6.0 / (1 + H))), rnd.normal(1, scale=0.1)]


def _targets_inputs(c, seed):
    rnd = _Rand(seed)
    S, N = c["S"], c["N"]
    off = _offsets(rnd, S, N, c["sigma"])
    return dict(env_off=torch.from_numpy(off.astype(np.int32)).cuda(), rewards=rnd.normal(S, scale=0.1), values=rnd.normal(S),
                last_values=rnd.normal(N), dones=rnd.dones(S, c["p_done"]))


def _ingest_inputs(c, seed):
    rnd = _Rand(seed)
    S, N = c["S"], c["N"]
    off = _offsets(rnd, S, N, c["sigma"])
    when, env, t = np.empty(S), np.empty(S, np.int32), np.empty(S, np.int32)
    for i in range(N):   # an environment's steps arrive in time order, the environments interleave
        a, b = int(off[i]), int(off[i + 1])
        when[a:b] = np.cumsum(rnd.np.exponential(1.0 / max(b - a, 1), size=b - a))
        env[a:b] = i
        t[a:b] = np.arange(b - a)
    arrival = np.argsort(when, kind="stable")
    H, layers = c["H"], c["layers"]
    fields = [rnd.normal(S, scale=0.1), rnd.normal(S), rnd.dones(S, 0.005), rnd.normal(S, c["D"]), rnd.actions(S, c["act"]), rnd.normal(S)]
    fields += [rnd.bits(S) for _ in range(c["epochs"])]
    fields += [rnd.normal(S, H, scale=0.1) for _ in range(2 * layers)]
    return dict(env=torch.from_numpy(env[arrival]).cuda(), t=torch.from_numpy(t[arrival]).cuda(), fields=fields)


def _pack_inputs(c, seed):
    rnd = _Rand(seed)
    S, N, H, layers = c["S"], c["N"], c["H"], c["layers"]
    off = _offsets(rnd, S, N, c["sigma"])
    return dict(env_off=torch.from_numpy(off.astype(np.int32)).cuda(), dones=rnd.dones(S, c["p_done"]), started=rnd.dones(N, 0.25),
                seq_key=rnd.bits(S), obs=rnd.normal(S, c["D"]), actions=rnd.actions(S, c["act"]), logp_old=rnd.normal(S), adv=rnd.normal(S),
                ret=rnd.normal(S), is_weight=torch.rand(S, generator=rnd.g, device="cuda"), rnn_h=rnd.normal(layers, S, H, scale=0.1),
                rnn_c=rnd.normal(layers, S, H, scale=0.1))


def _loss_inputs(c, seed):
    rnd = _Rand(seed)
    M, A = c["M"], c["act"]
    u, value = rnd.normal(M, A, scale=0.5), rnd.normal(M)
    if c["dist"] == 1:
        actions, log_std = rnd.normal(M, A), rnd.normal(A, scale=0.1)
    else:
        actions = torch.randint(0, A, (M,), generator=rnd.g, device="cuda", dtype=torch.int64).to(torch.int32)
        log_std = None
    logp = _logp(u.double(), actions, None if log_std is None else log_std.double())
    gap = rnd.normal(M, scale=0.1).double()
    # the gradient jumps where the ratio crosses the clip range: rows within rounding of it are moved away, so that
    # two correct evaluations take the same side
    near = ((torch.exp(gap) - 1.0).abs() - CLIP).abs() < 1e-3
    gap = torch.where(near, gap * 0.9, gap)
    return dict(u=u, value=value, log_std=log_std, actions=actions, logp_old=(logp - gap).float(), adv=rnd.normal(M), ret=rnd.normal(M),
                weight=torch.rand(M, generator=rnd.g, device="cuda"))


def _adam_inputs(c, seed):
    rnd = _Rand(seed)
    p = _weights(rnd, c["D"], c["H"], c["layers"], c["act"]) + [rnd.normal(c["act"], scale=0.1)]
    return dict(params=p, grads=[rnd.normal(*t.shape, scale=1e-3) for t in p], m=[rnd.normal(*t.shape, scale=1e-3) for t in p],
                v=[rnd.normal(*t.shape, scale=1e-3).square_() for t in p])


def _layout(lengths):
    """Time-major packing of pieces given longest first: alive pieces per timestep and where a timestep's rows begin."""
    T = int(lengths[0])
    bs = np.searchsorted(-lengths, -np.arange(T), side="left")   # pieces longer than t
    return bs.astype(np.int32), np.concatenate([[0], np.cumsum(bs)]).astype(np.int32)


def _lstm_inputs(c, seed):
    rnd = _Rand(seed)
    M, H, layers, D, A = c["M"], c["H"], c["layers"], c["D"], c["act"]
    off = _offsets(rnd, M, c["N"], c["sigma"])
    ends = np.nonzero(rnd.np.random(M) < c["p_done"])[0] + 1
    cuts = np.unique(np.concatenate([off, ends]))                 # pieces: stretches cut after every episode's end
    fresh = np.isin(cuts[:-1], ends) | (rnd.np.random(len(cuts) - 1) < 0.25)
    lengths = np.diff(cuts)
    order = np.argsort(-lengths, kind="stable")
    lengths, fresh = lengths[order], fresh[order]
    bs, t_off = _layout(lengths)
    x = rnd.normal(M, D)
    keep = torch.from_numpy((~fresh).astype(np.float32)).cuda().view(1, -1, 1)
    n = len(lengths)
    return dict(bs=bs, t_off=t_off, n_seq=n, x=x.bfloat16() if c["x_bf16"] else x, h0=rnd.normal(layers, n, H, scale=0.1).mul_(keep),
                c0=rnd.normal(layers, n, H, scale=0.1).mul_(keep), weights=_weights(rnd, D, H, layers, A),
                d_u=rnd.normal(M, A, scale=1.0 / M), d_v=rnd.normal(M, scale=1.0 / M))


def _update_inputs(c, seed):
    w = workloads.Workload("update", c["N"], c["S"], 0, 0, c["sigma"], c["D"], c["layers"], c["H"], c["dist"], c["act"],
                           c["p_done"], c["epochs"], c["B"], c["bf16"])
    ro = workloads.make_rollout(w, seed, bias_scale=0.1)
    arrival = workloads.arrival_order(ro["env_off"], seed + 1)
    # a fresh policy is close to the uniform one (categorical) or to a unit normal at zero (Gaussian)
    if c["dist"] == 0:
        base = np.full(c["S"], -math.log(c["act"]), np.float32)
    else:
        ls = ro["weights"]["log_std"]
        base = (-0.5 * np.square(ro["actions"] * np.exp(-ls)) - ls - 0.5 * math.log(2 * math.pi)).sum(1).astype(np.float32)
    return w, ro, arrival, base + ro["logp_noise"]


# ---- what a program keeps between calls -----------------------------------------------------------------------

def _zeros(*shape, dtype=torch.float32):
    return torch.zeros(*shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    return {"targets": _prepare_targets, "ingest": _prepare_ingest, "pack": _prepare_pack, "loss": _prepare_loss, "adam": _prepare_adam,
            "lstm": _prepare_lstm, "update": _prepare_update}[case["op"]](case, seed)


def run(state):
    return state["run"](state)


def _prepare_targets(c, seed):
    S = c["S"]
    return dict(c, run=_run_targets, i=_targets_inputs(c, seed), adv=_zeros(S), ret=_zeros(S), weight=_zeros(S),
                ws=ver.workspace(ver.ver_gae_workspace_bytes(S)))


def _run_targets(s):
    i = s["i"]
    ver.ver_gae(i["rewards"], i["values"], i["dones"], i["last_values"], i["env_off"], s["N"], s["S"], GAMMA, LAM, s["adv"], s["ret"], s["ws"])
    ver.ver_is_weight(i["env_off"], s["N"], s["S"], MAX_IS, s["weight"])
    return s["adv"], s["ret"], s["weight"]


def _prepare_ingest(c, seed):
    i = _ingest_inputs(c, seed)
    return dict(c, run=_run_ingest, i=i, env_off=_zeros(c["N"] + 1, dtype=torch.int32), order=_zeros(c["S"], dtype=torch.int32),
                info=_zeros(4, dtype=torch.int32), pairs=[(f, torch.zeros_like(f)) for f in i["fields"]],
                ws=ver.workspace(ver.ver_ingest_workspace_bytes(c["N"], c["S"])))


def _run_ingest(s):
    ver.ver_ingest(s["i"]["env"], s["i"]["t"], s["N"], s["S"], s["env_off"], s["order"], s["info"], s["ws"])
    ver.ver_ingest_gather_batch(s["order"], s["S"], s["pairs"])
    return [s["env_off"], s["order"], s["info"]] + [dst for _, dst in s["pairs"]]


def _prepare_pack(c, seed):
    i = _pack_inputs(c, seed)
    S, N, B, H, layers = c["S"], c["N"], c["B"], c["H"], c["layers"]
    M = S // B
    i32 = torch.int32
    sets = []
    for _ in range(B):
        sets.append(dict(info=_zeros(4, dtype=i32), seq_first=_zeros(M, dtype=i32), seq_len=_zeros(M, dtype=i32),
                         seq_is_ep_start=_zeros(M, dtype=torch.uint8), batch_sizes=_zeros(M, dtype=i32), t_off=_zeros(M + 1, dtype=i32),
                         gather_idx=_zeros(M, dtype=i32),
                         obs_packed=_zeros(M, c["D"], dtype=torch.bfloat16 if c["x_bf16"] else torch.float32),
                         actions_packed=torch.zeros_like(i["actions"][:M]), logp_old_packed=_zeros(M), adv_packed=_zeros(M),
                         ret_packed=_zeros(M), is_weight_packed=_zeros(M), h0=_zeros(layers, M, H), c0=_zeros(layers, M, H)))
    return dict(c, run=_run_pack, i=i, M=M, sets=sets, ws=[ver.workspace(ver.ver_pack_workspace_bytes(N, S, B)) for _ in range(B)])


def _pack_block(s, b, index_ready):
    i = s["i"]
    return ver.pack_args(dones=i["dones"], env_off=i["env_off"], env_started_episode=i["started"], seq_key=i["seq_key"], N=s["N"], S=s["S"],
                         B=s["B"], b=b, obs=i["obs"], D=s["D"], obs_packed_bf16=int(s["x_bf16"]), actions=i["actions"],
                         act_bytes=i["actions"][0].numel() * 4, logp_old=i["logp_old"], adv=i["adv"], ret=i["ret"], is_weight=i["is_weight"],
                         rnn_h=i["rnn_h"], rnn_c=i["rnn_c"], n_layers=s["layers"], H=s["H"], seq_cap=s["M"], workspace=s["ws"][b],
                         index_ready=index_ready, **s["sets"][b])


def _run_pack(s):
    ver.ver_pack_index_batch([_pack_block(s, b, 0) for b in range(s["B"])])
    for b in range(s["B"]):
        ver._check(ver.lib.ver_pack_minibatch(_pack_block(s, b, 1), ver._stream()))
    return [t for o in s["sets"] for t in o.values()]


def _prepare_loss(c, seed):
    M, A = c["M"], c["act"]
    return dict(c, run=_run_loss, i=_loss_inputs(c, seed), cfg=ver.ppo_cfg(CLIP, VALUE_COEF, ENTROPY_COEF, c["dist"], A), scalars=_zeros(6),
                d_u=_zeros(M, A), d_v=_zeros(M), d_ls=_zeros(A) if c["dist"] == 1 else None,
                ws=ver.workspace(ver.ver_ppo_loss_workspace_bytes(M, A)))


def _run_loss(s):
    i = s["i"]
    ver.ver_ppo_loss(s["cfg"], s["M"], i["u"], i["value"], i["log_std"], i["actions"], i["logp_old"], i["adv"], i["ret"], i["weight"],
                     s["scalars"], s["d_u"], s["d_v"], s["d_ls"], s["ws"])
    return [s["scalars"], s["d_u"], s["d_v"]] + ([s["d_ls"]] if s["d_ls"] is not None else [])


def _prepare_adam(c, seed):
    return dict(c, run=_run_adam, i=_adam_inputs(c, seed), k=0, norm=_zeros(1),
                cfg=ver.adam_cfg(lr0=LR0, total_steps=SCHEDULE, beta1=BETA1, beta2=BETA2, eps=EPS, max_grad_norm=MAX_NORM),
                ws=ver.workspace(ver.ver_adam_workspace_bytes()))


def _run_adam(s):
    i = s["i"]
    ver.ver_adam_step(s["cfg"], i["params"], i["grads"], i["m"], i["v"], s["k"], s["norm"], s["ws"])
    s["k"] += 1
    return i["params"] + i["m"] + i["v"] + [s["norm"]]


def _prepare_lstm(c, seed):
    i = _lstm_inputs(c, seed)
    M, T = c["M"], len(i["bs"])
    bs, t_off = np.zeros(M, np.int32), np.full(M + 1, M, np.int32)
    bs[:T], t_off[:T + 1] = i["bs"], i["t_off"]
    cfg = ver.lstm_cfg(c["layers"], c["D"], c["H"], c["act"], c["compute"], int(c["x_bf16"]))
    return dict(c, run=_run_lstm, i=i, cfg=cfg, info=torch.tensor([i["n_seq"], T, i["n_seq"], 0], dtype=torch.int32, device="cuda"),
                bs=torch.from_numpy(bs).cuda(), t_off=torch.from_numpy(t_off).cuda(), u=_zeros(M, c["act"]), v=_zeros(M),
                grads=[torch.zeros_like(t) for t in i["weights"]] if c["backward"] else [],
                d_x=_zeros(M, c["D"]) if c["backward"] and c["dx"] else None, ws=ver.workspace(ver.ver_lstm_workspace_bytes(cfg, M)))


def _run_lstm(s):
    i = s["i"]
    ver.ver_lstm_fwd(s["cfg"], i["x"], s["M"], s["info"], s["bs"], s["t_off"], i["h0"], i["c0"], i["n_seq"], i["weights"], s["u"], s["v"], s["ws"])
    if s["backward"]:
        ver.ver_lstm_bwd(s["cfg"], i["x"], s["M"], s["info"], s["bs"], s["t_off"], i["h0"], i["c0"], i["n_seq"], i["weights"], i["d_u"], i["d_v"],
                         s["grads"], s["d_x"], s["ws"])
    return [s["u"], s["v"]] + s["grads"] + ([s["d_x"]] if s["d_x"] is not None else [])


def _prepare_update(c, seed):
    _, ro, arrival, logp_old = _update_inputs(c, seed)
    L = Learner(ro, max_is=MAX_IS, arrival=arrival, adam_total_steps=SCHEDULE)
    L.set_logp_old(torch.from_numpy(logp_old).cuda())
    return dict(c, run=_run_update, learner=L)


def _run_update(s):
    L = s["learner"]
    L.update()
    return [L.head_out, L.value, L.scalars, L.adv, L.ret, L.is_w] + L.opt_params


# ---- the least a pass has to move and compute -----------------------------------------------------------------

def _params(c):
    return sum(4 * c["H"] * ((c["D"] if l == 0 else c["H"]) + c["H"] + 2) for l in range(c["layers"])) + (c["act"] + 1) * (c["H"] + 1)


def _lstm_flops(c, rows, backward, dx):
    H = c["H"]
    d = [c["D"] if l == 0 else H for l in range(c["layers"])]
    f = sum(8 * H * (x + H) for x in d) + 2 * H * (c["act"] + 1)
    if backward:
        f += sum(8 * H * (x + H) for x in d) + 2 * H * (c["act"] + 1)                       # weight gradients
        f += sum(8 * H * H for _ in d) + 8 * H * sum(d[1:]) + 2 * H * (c["act"] + 1) + (8 * H * d[0] if dx else 0)
    return f * rows


def work(case):
    c, op = case, case["op"]
    if op == "targets":
        return {"bytes": 21 * c["S"] + 8 * c["N"], "flops": 8 * c["S"]}
    if op == "ingest":
        row = 4 * (c["D"] + max(c["act"], 1) + 3 + c["epochs"] + 2 * c["layers"] * c["H"]) + 1
        return {"bytes": c["S"] * (2 * row + 12) + 4 * c["N"], "flops": 0}
    if op == "pack":
        row = 4 * c["D"] + (2 if c["x_bf16"] else 4) * c["D"] + 8 * max(c["act"], 1) + 32 + 16
        return {"bytes": c["S"] * row + 16 * c["layers"] * c["H"] * (c["N"] + int(c["S"] * c["p_done"])), "flops": 0}
    if op == "loss":
        return {"bytes": c["M"] * ((12 * c["act"] if c["dist"] == 1 else 8 * c["act"] + 4) + 24), "flops": c["M"] * (20 * c["act"] + 20)}
    if op == "adam":
        return {"bytes": 28 * _params(c), "flops": 14 * _params(c)}
    if op == "lstm":
        p, M = 4 * _params(c), c["M"]
        b = M * c["D"] * (2 if c["x_bf16"] else 4) + p + 4 * M * (c["act"] + 1)
        if c["backward"]:
            b += p + 4 * M * (c["act"] + 1) + (4 * M * c["D"] if c["dx"] else 0)
        return {"bytes": b, "flops": _lstm_flops(c, M, c["backward"], c["dx"])}
    rows = c["S"] * c["epochs"]
    row = 4 * (c["D"] + max(c["act"], 1) + 3 + c["epochs"] + 2 * c["layers"] * c["H"]) + 1
    return {"bytes": c["S"] * row + rows * 4 * c["D"] + c["epochs"] * c["B"] * 28 * _params(c), "flops": _lstm_flops(c, rows, True, False)}


# ---- tolerances -----------------------------------------------------------------------------------------------

# About four times the largest difference from the 64-bit results below, over the listed cases and drawn ones
# (relative 2-norm, largest element).  A whole update ends in optimiser steps whose size does not depend on the
# gradient's, so what a gradient of rounding size decides shows in its outputs.
def tolerance(case):
    op = case["op"]
    if op in ("ingest", "pack"):
        return "exact"                              # integers and moved values
    if op == "lstm":
        return {"rel": 1.5e-2, "max": 0.2} if case["compute"] else {"rel": 1e-5, "max": 1e-4}
    if op == "update":
        return {"rel": 3e-2, "max": 0.3} if case["bf16"] else {"rel": 1e-4, "max": 1e-2}
    return {"adam": {"rel": 2e-7, "max": 4e-6}, "loss": {"rel": 5e-6, "max": 1e-4}, "targets": {"rel": 1e-6, "max": 1e-5}}[op]


# ---- the same in 64 bits --------------------------------------------------------------------------------------

def exact(case, seed):
    f = {"targets": _exact_targets, "ingest": _exact_ingest, "pack": _exact_pack, "loss": _exact_loss, "adam": _exact_adam,
         "lstm": _exact_lstm, "update": _exact_update}[case["op"]]
    return f(case, seed)


def _scan(delta, slope):
    """x[k] = delta[k] + slope[k] * x[k + 1], x beyond the end 0, by doubling."""
    b, a, d = delta.clone(), slope.clone(), 1
    while d < len(b):
        b[:-d] += a[:-d] * b[d:].clone()
        a[:-d] *= a[d:].clone()
        a[-d:] = 0.0
        d *= 2
    return b


def _gae64(rewards, values, dones, last_values, env_off):
    r, v, off = rewards.double(), values.double(), env_off.long()
    end = off[1:][off[1:] > off[:-1]] - 1              # last step of every non-empty stretch
    nxt = torch.cat([v[1:], v[:1]])
    nxt[end] = last_values.double()[off[1:] > off[:-1]]
    alive = 1.0 - dones.double()
    gamma, lam = float(np.float32(GAMMA)), float(np.float32(LAM))
    slope = gamma * lam * alive
    slope[end] = 0.0
    adv = _scan(r + gamma * alive * nxt - v, slope)
    return adv, adv + v


def _is64(env_off, S, N):
    L = (env_off[1:] - env_off[:-1]).long()
    w = torch.clamp((S / N) / L.double(), max=MAX_IS)
    return torch.repeat_interleave(w, L)


def _exact_targets(c, seed):
    i = _targets_inputs(c, seed)
    adv, ret = _gae64(i["rewards"], i["values"], i["dones"], i["last_values"], i["env_off"])
    return adv, ret, _is64(i["env_off"], c["S"], c["N"])


def _exact_ingest(c, seed):
    i = _ingest_inputs(c, seed)
    env = i["env"].cpu().numpy()
    order = np.argsort(env, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(env, minlength=c["N"]))])
    o = torch.from_numpy(order).cuda()
    return [torch.from_numpy(off.astype(np.int32)).cuda(), o.to(torch.int32), _zeros(4, dtype=torch.int32)] + [f[o] for f in i["fields"]]


def _pack64(dones, env_off, started, key, B, b):
    """Index arrays of minibatch b: sequences cut at stretch starts and after episode ends, in order of (key, id),
    laid end to end, the b-th of B equal shares packed longest first."""
    dones, env_off = dones.cpu().numpy(), env_off.cpu().numpy().astype(np.int64)
    S = len(dones)
    M = S // B
    ends = np.nonzero(dones)[0] + 1
    first = np.unique(np.concatenate([env_off[:-1], ends[ends < S]]))
    first = first[first < S]
    length = np.diff(np.concatenate([first, [S]]))
    fresh = np.isin(first, ends)
    s = started.cpu().numpy()
    opening = {}
    for e in range(len(s)):
        if env_off[e + 1] > env_off[e]:
            opening[int(env_off[e])] = bool(s[e])
    fresh |= np.array([opening.get(int(k), False) for k in first])
    order = np.lexsort((np.arange(len(first)), key.cpu().numpy().view(np.uint32)[first]))
    at = np.concatenate([[0], np.cumsum(length[order])])
    pieces = []
    for j, q in enumerate(order):
        lo, hi = max(at[j], b * M), min(at[j + 1], (b + 1) * M)
        if lo < hi:
            pieces.append((first[q] + lo - at[j], hi - lo, fresh[q] and lo == at[j]))
    start, ln, fr = (np.array(x) for x in zip(*pieces))
    o = np.argsort(-ln, kind="stable")
    start, ln, fr = start[o], ln[o], fr[o]
    bs, t_off = _layout(ln)
    gather = np.concatenate([start[:n] + t for t, n in enumerate(bs)])
    return dict(K=len(first), start=start, ln=ln, fresh=fr, bs=bs, t_off=t_off, gather=gather, M=M)


def _padded(values, n, fill, dtype):
    out = np.full(n, fill, dtype)
    out[:len(values)] = values
    return torch.from_numpy(out).cuda()


def _exact_pack(c, seed):
    i = _pack_inputs(c, seed)
    out = []
    for b in range(c["B"]):
        p = _pack64(i["dones"], i["env_off"], i["started"], i["seq_key"], c["B"], b)
        M, n, T = p["M"], len(p["ln"]), len(p["bs"])
        g = torch.from_numpy(p["gather"]).cuda()
        keep = torch.from_numpy((~p["fresh"]).astype(np.float32)).cuda().view(1, -1, 1)
        states = []
        for t in (i["rnn_h"], i["rnn_c"]):
            full = _zeros(c["layers"], M, c["H"])
            full[:, :n] = t[:, torch.from_numpy(p["start"]).cuda()] * keep
            states.append(full)
        obs = i["obs"][g]
        out += [torch.tensor([n, T, p["K"], 0], dtype=torch.int32, device="cuda"), _padded(p["start"], M, 0, np.int32),
                _padded(p["ln"], M, 0, np.int32), _padded(p["fresh"], M, 0, np.uint8), _padded(p["bs"], M, 0, np.int32),
                _padded(p["t_off"], M + 1, M, np.int32), g.to(torch.int32), obs.bfloat16() if c["x_bf16"] else obs, i["actions"][g],
                i["logp_old"][g], i["adv"][g], i["ret"][g], i["is_weight"][g]] + states
    return out


def _logp(u, actions, log_std):
    if log_std is None:
        return torch.log_softmax(u, 1).gather(1, actions.long().view(-1, 1)).squeeze(1)
    z = (actions.double() - u) * torch.exp(-log_std)
    return (-0.5 * z * z - log_std - 0.5 * math.log(2 * math.pi)).sum(1)


def _ppo64(u, value, log_std, actions, logp_old, adv, ret, weight):
    """The total loss and its six scalars."""
    logp = _logp(u, actions, log_std)
    if log_std is None:
        lp = torch.log_softmax(u, 1)
        entropy = -(lp.exp() * lp).sum(1)
    else:
        entropy = (log_std + 0.5 * math.log(2 * math.pi * math.e)).sum().expand(len(u))
    rho = torch.exp(logp - logp_old.double())
    clip = float(np.float32(CLIP))
    a, w = adv.double(), weight.double()
    policy = (w * -torch.minimum(rho * a, torch.clamp(rho, 1 - clip, 1 + clip) * a)).mean()
    vloss = (w * 0.5 * (value - ret.double()) ** 2).mean()
    ent = (w * entropy).mean()
    total = policy + float(np.float32(VALUE_COEF)) * vloss - float(np.float32(ENTROPY_COEF)) * ent
    kl, frac = (logp_old.double() - logp).mean(), ((rho - 1).abs() > clip).double().mean()
    return total, torch.stack([x.detach() for x in (total, policy, vloss, ent, kl, frac)])


def _exact_loss(c, seed):
    i = _loss_inputs(c, seed)
    u, v = i["u"].double().requires_grad_(), i["value"].double().requires_grad_()
    ls = i["log_std"].double().requires_grad_() if c["dist"] == 1 else None
    total, scalars = _ppo64(u, v, ls, i["actions"], i["logp_old"], i["adv"], i["ret"], i["weight"])
    total.backward()
    return [scalars, u.grad, v.grad] + ([ls.grad] if ls is not None else [])


def _adam64(p, g, m, v, k, scale=1.0):
    lr0, b1, b2, eps = (float(np.float32(x)) for x in (LR0, BETA1, BETA2, EPS))
    g = g.double() * scale
    m = b1 * m.double() + (1 - b1) * g
    v = b2 * v.double() + (1 - b2) * g * g
    lr = lr0 * (1 + math.cos(math.pi * min(k, SCHEDULE) / SCHEDULE)) / 2
    return p.double() - lr * (m / (1 - b1 ** (k + 1))) / (torch.sqrt(v / (1 - b2 ** (k + 1))) + eps), m, v


def _exact_adam(c, seed):
    i = _adam_inputs(c, seed)
    norm = torch.sqrt(sum((g.double() ** 2).sum() for g in i["grads"]))
    scale = min(1.0, MAX_NORM / (float(norm) + 1e-6))
    new = [_adam64(p, g, m, v, 0, scale) for p, g, m, v in zip(i["params"], i["grads"], i["m"], i["v"])]
    return [n[0] for n in new] + [n[1] for n in new] + [n[2] for n in new] + [norm.view(1)]


def _net64(x, bs, h0, c0, weights, layers):
    """Head outputs and values of the packed rows; weights: flat list of float64 tensors."""
    for l in range(layers):
        W_ih, W_hh, b_ih, b_hh = weights[4 * l:4 * l + 4]
        z_in = x @ W_ih.t() + (b_ih + b_hh)
        W_t = W_hh.t().contiguous()
        h, cell, row, out = h0[l].double(), c0[l].double(), 0, []
        for n in bs.tolist():
            i, f, g, o = (z_in[row:row + n] + h[:n] @ W_t).chunk(4, 1)
            cell = torch.sigmoid(f) * cell[:n] + torch.sigmoid(i) * torch.tanh(g)
            h = torch.sigmoid(o) * torch.tanh(cell)
            out.append(h)
            row += n
        x = torch.cat(out)
    W_a, b_a, w_v, b_v = weights[4 * layers:]
    return x @ W_a.t() + b_a, x @ w_v + b_v


def _exact_lstm(c, seed):
    i = _lstm_inputs(c, seed)
    x = i["x"].double()
    w = [t.double() for t in i["weights"]]
    if not c["backward"]:
        with torch.no_grad():
            return list(_net64(x, i["bs"], i["h0"], i["c0"], w, c["layers"]))
    for t in w + [x]:
        t.requires_grad_()
    u, v = _net64(x, i["bs"], i["h0"], i["c0"], w, c["layers"])
    ((u * i["d_u"].double()).sum() + (v * i["d_v"].double()).sum()).backward()
    return [u.detach(), v.detach()] + [t.grad for t in w] + ([x.grad] if c["dx"] else [])


def _exact_update(c, seed):
    _, ro, _, logp_old = _update_inputs(c, seed)
    dev = {k: torch.from_numpy(np.ascontiguousarray(ro[k].view(np.int32) if ro[k].dtype == np.uint32 else ro[k])).cuda()
           for k in ("rewards", "values", "dones", "last_values", "env_off", "env_started_episode", "obs", "actions", "seq_key", "rnn_h", "rnn_c")}
    logp_old = torch.from_numpy(logp_old).cuda()
    adv, ret = _gae64(dev["rewards"], dev["values"], dev["dones"], dev["last_values"], dev["env_off"])
    isw = _is64(dev["env_off"], c["S"], c["N"])
    flat = [lw[n] for lw in ro["weights"]["layers"] for n in ("W_ih", "W_hh", "b_ih", "b_hh")]
    flat += [ro["weights"][n] for n in ("W_a", "b_a", "w_v", "b_v")] + ([ro["weights"]["log_std"]] if c["dist"] == 1 else [])
    p = [torch.from_numpy(np.asarray(a, np.float32)).cuda().double() for a in flat]
    m, v = [torch.zeros_like(t) for t in p], [torch.zeros_like(t) for t in p]
    k, n_w = 0, 4 * c["layers"] + 4
    for e in range(c["epochs"]):
        for b in range(c["B"]):
            q = _pack64(dev["dones"], dev["env_off"], dev["env_started_episode"], dev["seq_key"][e], c["B"], b)
            g = torch.from_numpy(q["gather"]).cuda()
            keep = torch.from_numpy((~q["fresh"]).astype(np.float32)).cuda().view(1, -1, 1)
            at = torch.from_numpy(q["start"]).cuda()
            p = [t.detach().requires_grad_() for t in p]
            u, val = _net64(dev["obs"][g].double(), q["bs"], dev["rnn_h"][:, at] * keep, dev["rnn_c"][:, at] * keep, p[:n_w], c["layers"])
            total, scalars = _ppo64(u, val, p[n_w] if c["dist"] == 1 else None, dev["actions"][g], logp_old[g], adv[g], ret[g], isw[g])
            total.backward()
            with torch.no_grad():
                new = [_adam64(a, a.grad, x, y, k) for a, x, y in zip(p, m, v)]
            p, m, v = ([n[j].detach() for n in new] for j in range(3))
            k += 1
    return [u.detach(), val.detach(), scalars, adv, ret, isw] + p
