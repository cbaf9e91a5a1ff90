"""The fetch of the entmax decode's candidates at the sizes where its forms meet: 4, 16 and 64 groups of 64 tokens to each of the
sixteen segments and a token more, peaked rows, rows of which every group passes with one candidate or many, page sizes whose
groups are shorter.

Results against the float64 oracle under the rules of tests/helpers.py."""
import math

import pytest
import torch

from oracle import entmaxkv_oracle as orc
from paper_2605_21649_amd import binding as ekv
from paper_2605_21649_amd import synth
from tests.helpers import DeviceState, unit_kv, check_decode_unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 0.1, 0.04, 0.01])
@pytest.mark.parametrize("tokens,page,dtype", [(4 * 1024, 16, "bf16"), (4 * 1024 + 1, 16, "f32"), (16 * 1024, 16, "bf16"), (16 * 1024 + 1, 32, "bf16"),
                                               (17 * 960 - 5, 12, "f32"), (64 * 1024, 16, "bf16"), (64 * 1024 + 1, 64, "bf16"), (65 * 960, 20, "bf16")])
def test_candidates_at_the_edges_of_a_segment(tokens, page, dtype, scale):
    w = synth.Workload("fetch", 1, 2, 1, 128, tokens, page, dtype, scale=scale / math.sqrt(128.0))
    inp = synth.make_inputs(w, 31 + tokens, device="cpu")
    st = DeviceState(w, inp)
    toks = torch.full((1, 2, 65536), -1, device="cuda", dtype=torch.int32)
    ekv.ekv_decode_full(st.cfg, st.inp["q"], st.cache(), st.out, st.tau, st.supp, st.workspace(ekv.EKV_OP_DECODE_FULL),
                        extras=ekv.decode_extras(support_tokens=toks))
    torch.cuda.synchronize()
    for hq in range(2):
        q, K, V = unit_kv(inp, w, 0, hq)
        ref = orc.entmax_attention(q, K, V, w.alpha, w.score_scale)
        check_decode_unit(w, st.out[0, hq].cpu().numpy(), float(st.tau[0, hq]), int(st.supp[0, hq]),
                          toks[0, hq].cpu().numpy(), ref, boundary_expected=True)
