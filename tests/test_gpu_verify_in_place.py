"""The verify step with its emitted tokens written over its input tokens (one array for both): the
same tokens, accepted lengths and log-probs, bit for bit, as with an array of their own, for few
sequences (every workgroup of the mass pass takes the decisions for itself and reads the drafts) and
for a batch that takes them in a launch of its own."""
import pytest
import torch

import workloads
from helpers import dev, model_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k", [(1, 1), (2, 7), (4, 15), (3, 18), (600, 2)])
def test_in_place(molt_lib, B, k):
    print(f"case B={B} k={k}", flush=True)
    w = workloads.TINY_FP32.scaled(batch=B, k=k, ctx_lo=1, ctx_hi=9)
    layout = workloads.make_kv_layout(w, 3)
    model = model_from(w, [workloads.make_layer_weights(w, 3, l) for l in range(w.n_layers)],
                       workloads.make_head_weights(w, 3), molt_lib)
    caches = [workloads.make_kv_cache(w, layout, 3, l) for l in range(w.n_layers)]
    kv = molt_lib.KVCache([dev(c[0]) for c in caches], [dev(c[1]) for c in caches],
                          dev(torch.from_numpy(layout.block_tables)), dev(torch.from_numpy(layout.context_lens)))
    reached = set()
    for seed in range(8):
        tokens = dev(torch.from_numpy(workloads.make_step_tokens(w, seed)))
        u = dev(workloads.make_uniforms(B, k, seed)) * 1e-3    # every draft that p allows is kept
        u[:, k] *= 1e3
        u[seed % B, seed % (k + 1)] = 0.999
        a = molt_lib.verify_step(model, kv, tokens, u)
        out = {"tokens": tokens, "n_accepted": torch.empty_like(a["n_accepted"]),
               "logprobs": torch.empty_like(a["logprobs"])}
        molt_lib.verify_step(model, kv, tokens, u, out=out)
        for key in ("tokens", "n_accepted"):
            assert torch.equal(a[key], out[key]), key
        assert torch.equal(torch.nan_to_num(a["logprobs"], nan=7.0), torch.nan_to_num(out["logprobs"], nan=7.0))
        reached.update(a["n_accepted"].tolist())
    print("accepted lengths", sorted(reached), flush=True)
    assert len(reached) > 1
