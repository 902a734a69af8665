"""GPU parity at the edges of the kernels' tiles and of their dispatch: shapes just below, at and
just above a tile's rows, columns and k groups, each checked against the CPU oracle (scores within
the bound of the data type, tokens bit for bit except where the oracle flags a near tie)."""
import numpy as np
import pytest

import oracle
from paper_2607_02119_amd import inputs
from tests._compare import TokenCheck, say, score_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2607_02119_amd import harness  # noqa: E402

GAP_TOL, TOPK_TOL, TOPP_TOL = 1e-3, 1e-4, 1e-5


def check_one_step(wl, t, score_tol):
    dw = harness.DeviceWorkload(wl)
    dw.load_hidden([t])
    dw.tokens.fill_(-1)
    dw.run_step(t, hidden_index=0)
    torch.cuda.synchronize()
    o = oracle.head_step(dw.host_head, inputs.make_batch(wl, t, dw.layout), seed=dw.seed,
                         gap_tol=GAP_TOL, topk_tol=TOPK_TOL, topp_tol=TOPP_TOL)
    tc = TokenCheck()
    tc.add(dw.tokens.cpu().numpy(), o["tokens"], o["flags"], where=f"t={t}")
    tc.assert_ok(wl.name)
    if wl.Rs:
        rows = [r for r, _ in dw.plan.sampled_rows()]
        err = score_rel_err(dw.scores.cpu().numpy(), rows, o["scores"],
                            oracle.stream_sizes(dw.host_head))
        say(f"  score rel err {err:.3e}")
        assert err <= score_tol
    assert dw.status() == 0


# fp32 head: row blocks of 16, 32 and 64 rows and row tiles beyond, 16-column
# (text: 32-column) workgroups, k16 groups dealt to four waves; H below one
# group, not a multiple of 16, and not a multiple of 4
F32 = [
    # H, V, pairs, solo, text, V_text
    (4, 1, 0, 1, 0, 0),
    (3, 5, 1, 0, 1, 1),
    (16, 16, 8, 0, 1, 32),
    (17, 17, 8, 1, 2, 33),
    (64, 31, 16, 0, 16, 64),
    (272, 40, 16, 1, 17, 31),
    (255, 33, 30, 4, 33, 65),
    (1028, 20, 32, 1, 65, 97),
]


@pytest.mark.parametrize("H,V,pairs,solo,text,V_text", F32)
def test_fp32_head_tiles(H, V, pairs, solo, text, V_text):
    wl = inputs.Workload(f"f32_{H}_{V}", H=H, K=2, V=V, n_pairs=pairs, n_solo=solo, n_text=text,
                         V_text=V_text, dtype="f32", top_k=3, steps=4, shuffle=True,
                         bias=H % 2 == 0)
    say(f"case {wl.name} R={wl.R}")
    check_one_step(wl, 2, 1e-5)
