"""Time loops whose groups fall from more than 512 alive pieces through 512, 256, 16 and 4: every form of a loop and every change of
form inside one launch, against plain torch in 64 bits on the packed rows."""
import numpy as np
import pytest
import torch

from tests.util import closer, l2_rel_err

pytestmark = pytest.mark.gpu


def reference(x, batch_sizes, W, layers, h0, c0, d_u, d_v):
    """Outputs, weight gradients and input gradient of the packed rows, in float64."""
    t64 = lambda a: a.double().requires_grad_()
    w, rows = [t64(t) for t in W], t64(x)
    seq = rows
    for l in range(layers):
        W_ih, W_hh, b_ih, b_hh = w[4 * l:4 * l + 4]
        z = seq @ W_ih.t() + (b_ih + b_hh)
        h, c, out, at = h0[l].double(), c0[l].double(), [], 0
        for n in batch_sizes:
            i, f, g, o = (z[at:at + n] + h[:n] @ W_hh.t()).chunk(4, 1)
            c = torch.sigmoid(f) * c[:n] + torch.sigmoid(i) * torch.tanh(g)
            h = torch.sigmoid(o) * torch.tanh(c)
            out.append(h)
            at += n
        seq = torch.cat(out)
    u, v = seq @ w[4 * layers].t() + w[4 * layers + 1], seq @ w[4 * layers + 2] + w[4 * layers + 3]
    ((u * d_u.double()).sum() + (v * d_v.double()).sum()).backward()
    return [u.detach(), v.detach()], [t.grad for t in w], rows.grad


def run(ver, batch_sizes, layers, compute, H, D=36, A=4):
    g = torch.Generator(device="cuda").manual_seed(H + layers)
    normal = lambda *shape, scale=1.0: torch.randn(*shape, generator=g, device="cuda").mul_(scale)
    T, n_seq, M = len(batch_sizes), batch_sizes[0], sum(batch_sizes)
    x = normal(M, D)
    W = []
    for l in range(layers):
        d = D if l == 0 else H
        W += [normal(4 * H, d, scale=d ** -0.5), normal(4 * H, H, scale=H ** -0.5), normal(4 * H, scale=0.1), normal(4 * H, scale=0.1)]
    W += [normal(A, H, scale=H ** -0.5), normal(A, scale=0.1), normal(H, scale=H ** -0.5), normal(1, scale=0.1)]
    h0, c0 = normal(layers, n_seq, H, scale=0.5), normal(layers, n_seq, H, scale=0.5)
    d_u, d_v = normal(M, A, scale=1.0 / M), normal(M, scale=1.0 / M)
    i32 = dict(dtype=torch.int32, device="cuda")
    info, bs, t_off = torch.tensor([n_seq, T, M, 0], **i32), torch.zeros(M, **i32), torch.full((M + 1,), M, **i32)
    bs[:T] = torch.tensor(batch_sizes, **i32)
    t_off[:T] = torch.tensor([0] + list(np.cumsum(batch_sizes)[:-1]), **i32)
    cfg = ver.lstm_cfg(layers, D, H, A, compute, 0)
    ws = ver.workspace(ver.ver_lstm_workspace_bytes(cfg, M))
    ws.fill_(-1)
    nan = lambda t: torch.full_like(t, float("nan"))
    u, v, grads, dx = nan(d_u), nan(d_v), [nan(t) for t in W], nan(x)
    ver.ver_lstm_fwd(cfg, x, M, info, bs, t_off, h0, c0, n_seq, W, u, v, ws)
    ver.ver_lstm_bwd(cfg, x, M, info, bs, t_off, h0, c0, n_seq, W, d_u, d_v, grads, dx, ws)
    torch.cuda.synchronize()
    assert ws[0].item() == 0, "device-side wait timed out"
    (r_u, r_v), r_grads, r_dx = reference(x, batch_sizes, W, layers, h0, c0, d_u, d_v)
    close, host = closer(compute), lambda t: t.double().cpu().numpy()
    close(host(u), host(r_u), "head_out")
    close(host(v), host(r_v), "value")
    if compute:   # (the bar of tests/util.py for what comes out of back-propagation through time in bf16, in the 2-norm)
        for got, ref in zip(grads + [dx], r_grads + [r_dx]):
            assert l2_rel_err(host(got), host(ref)) <= 7e-3
    else:
        for k, (got, ref) in enumerate(zip(grads + [dx], r_grads + [r_dx])):
            close(host(got), host(ref), f"gradient {k}")


def falls(batch_sizes, groups, line):
    """First timestep with at most `line` pieces in the largest of `groups` groups that the pieces are dealt to."""
    return next((t for t, n in enumerate(batch_sizes) if (n + groups - 1) // groups <= line), len(batch_sizes))


# 525 pieces per group, 513, 512, ...; the last has long stretches of more than 16 pieces (the backward loop asks for 24 timesteps)
ONE = [4200, 4104, 4096, 2000, 700, 260, 140, 129, 128, 96, 40, 24, 8, 8, 3]


@pytest.mark.parametrize("compute,hidden", [(0, 64), (0, 256), (0, 320), (0, 448), (0, 512), (1, 64), (1, 320), (1, 512), (1, 576), (1, 1024)])
def test_one_layer_falls_through_all_forms(ver, compute, hidden):
    t_many, t_few, t_quad = (falls(ONE, 8, n) for n in (512, 16, 4))
    assert 0 < t_many < t_few < t_quad < len(ONE)
    run(ver, ONE, 1, compute, hidden)


@pytest.mark.parametrize("compute,hidden", [(0, 256), (0, 512), (1, 64), (1, 512), (1, 576), (1, 1024)])
def test_two_layers_fall_through_all_forms(ver, compute, hidden):
    """The cuts give the last group most pieces, far above 512; in each direction enough timesteps for the forms of a shared launch."""
    fall = [2400, 2300, 1600] + [900] * 4 + [500] * 10 + [140] * 10 + [100] * 30 + [20] * 3 + [9, 5, 2, 1]
    assert fall[0] > 3 * 512
    run(ver, fall, 2, compute, hidden)


@pytest.mark.parametrize("pieces,steps", [(51, 7), (51, 8), (51, 15), (51, 16), (51, 23), (51, 24), (51, 47), (51, 48), (75, 48), (99, 48), (147, 24), (195, 48)])
@pytest.mark.parametrize("compute,hidden", [(0, 256), (0, 448), (1, 64), (1, 192), (1, 512), (1, 1024)])
def test_lines_of_shared_launches(ver, compute, hidden, pieces, steps):
    """17, 25, 33, 49 and 65 pieces per group: both sides of the least numbers of timesteps forward (24) and backward (24, 48)."""
    run(ver, [pieces] * steps, 2, compute, hidden)


@pytest.mark.parametrize("pieces,steps", [(136, 23), (136, 24), (200, 24), (256, 24), (264, 24)])
@pytest.mark.parametrize("compute,hidden", [(0, 320), (0, 384), (1, 128), (1, 192)])
def test_lines_of_one_layer(ver, compute, hidden, pieces, steps):
    run(ver, [pieces] * steps, 1, compute, hidden)
