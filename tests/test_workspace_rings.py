"""The workspace of the LSTM holds the exchange ring of the loops beyond 16 pieces (lstm_many.h) only where a kernel of the width and
direction runs them, and no more of its rows than the minibatch can fill.  CPU only (the query touches no device)."""
import pytest

from paper_2210_05064_amd import binding as ver

SLOTS = 8 * 4   # groups x slots of the ring
ROUNDING = 4096   # of the arrays' beginnings


def ws(compute, hidden, layers, rows):
    return ver.ver_lstm_workspace_bytes(ver.lstm_cfg(layers, 32, hidden, 4, compute, 0), rows)


# bytes of everything else, as before there was such a ring
@pytest.mark.parametrize("compute,hidden,layers,rows,others,fwd_rows,bwd_rows", [
    (0, 64, 1, 59, 1003520, 0, 0), (0, 64, 2, 1024, 8409856, 0, 0), (0, 128, 1, 8192, 73882368, 0, 0),   # fp32 up to 128 units: neither direction
    (0, 256, 2, 1024, 38275840, 512, 0),                                                                # fp32 up to 256: forward
    (0, 512, 1, 300, 23805184, 304, 0),                                                                 # too few rows for 24 timesteps of 17 pieces
    (1, 512, 2, 8192, 429462272, 512, 0), (1, 256, 1, 2000, 38784768, 512, 0),                          # bf16 256 and 512: forward
    (1, 64, 1, 59, 609280, 64, 0), (1, 64, 2, 300, 2358272, 304, 0)])
def test_ring_only_where_it_is_used(compute, hidden, layers, rows, others, fwd_rows, bwd_rows):
    ring = SLOTS * hidden * (2 if compute else 4) * max(fwd_rows, 4 * bwd_rows)
    assert others <= ws(compute, hidden, layers, rows) <= others + ring + ROUNDING
