"""GPU tests: captured arrays of run-time compiled variants, however an expression reads them; tiles at the end of the keys and tiles of
which a wave sees nothing, whose transform the kernel leaves out."""
import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs, runner

pytestmark = pytest.mark.gpu

FORMS = {
    "indexed": "aux2[h * 64 + min(abs(i - j), 63)]",
    "pointer": "*(aux2 + h * 64 + min(abs(i - j), 63))",
    "long_index": "aux2[(long)h * 64 + min(abs(i - j), 63)]",
    "unsigned_index": "aux2[(unsigned)(h * 64 + min(abs(i - j), 63))]",
    "negative_index": "aux3[h * 64 + min(abs(i - j), 63) - 100]",
}


@pytest.mark.parametrize("Sq,Sk", [(333, 333), (100, 64), (64, 65), (500, 320)])
def test_array_forms(Sq, Sk):
    """The same bias read in every form gives the same bits, with and without the pre-pass over the tiles, within the tolerance of the oracle."""
    import torch
    dev = "cuda:0"
    B, H, D = 2, 4, 64
    w = inputs.causal_bf16(B=B, H=H, Hkv=2, S=Sq, Sk=Sk, D=D, causal=False, salt=21)
    ids_q, ids_k = (inputs.doc_ids(B, n, seed=78, lo=20, hi=90) for n in (Sq, Sk))
    ids_k[:, 0] = 0                                                            # no row of a document without keys
    ids_q = np.minimum(ids_q, ids_k.max(axis=1)[:, None])
    table = inputs.normal((H, 64), inputs.tensor_seed(9, 8), "bf16")
    flat = torch.from_numpy(table.astype(np.float32)).to(dev, torch.bfloat16).reshape(-1)
    arrays = [torch.from_numpy(ids_q).to(dev), torch.from_numpy(ids_k).to(dev), flat, flat[100:]]
    dw = runner.upload(w, out_dtype="f32")
    ref, ref_lse = ao.attention_custom(w.q, w.k, w.v, scale=w.scale,
                                       score_mod=lambda s, b, g, h, i, j: s + table.astype(np.float64)[h][np.minimum(np.abs(i - j), 63)],
                                       mask=lambda b, g, h, i, j: ids_q[b][:, None] != ids_k[b][None, :])
    first = None
    for name, form in FORMS.items():
        var = fb.CustomVariant(f"s + {form}", "aux0[b * Sq + i] != aux1[b * Sk + j]", D, aux=arrays)
        need = var.skip_workspace_size(dw.tq, dw.tk)
        for ws in (None, torch.empty(need, dtype=torch.uint8, device=dev)):
            dw.out.fill_(float("nan"))
            dw.lse.fill_(float("nan"))
            fb.check(var.forward(dw.tq, dw.tk, dw.tv, float(w.scale), dw.tout, dw.tlse, workspace=ws))
            torch.cuda.synchronize()
            got = dw.out.cpu().numpy().copy(), dw.lse.cpu().numpy()[..., 0].copy()
            if first is None:
                first = got
                dead = np.isneginf(ref_lse)
                assert np.array_equal(np.isneginf(got[1]), dead)
                assert float(np.max(np.abs(got[0] - ref))) <= 1e-2 and float(np.max(np.abs(got[1][~dead] - ref_lse[~dead]))) <= 1e-3
            assert np.array_equal(got[0], first[0]) and np.array_equal(got[1], first[1]), (name, ws is None)
        var.release()


@pytest.mark.parametrize("far", [-1e4, -1e9, -1e30, -2.2e38])
def test_rows_hidden_by_a_finite_score(far):
    """Rows whose scores are all far below zero by the same amount, and rows with one key that is not: the average of the values, and that key's."""
    import torch
    B, H, S, D = 1, 2, 160, 64
    w = inputs.causal_bf16(B=B, H=H, Hkv=H, S=S, D=D, causal=False, salt=22)
    hidden = np.ones((S, S), np.float32)
    hidden[:100, 3] = 0.0
    hidden[100:120, 130:] = 0.0
    table = torch.from_numpy(hidden).to("cuda:0", torch.bfloat16)
    dw = runner.upload(w, out_dtype="f32")
    var = fb.CustomVariant(f"0.0f * s + {far:.9e}f * (float)aux2[i * Sk + j]", None, D, aux=[None, None, table])
    fb.check(var.forward(dw.tq, dw.tk, dw.tv, float(w.scale), dw.tout, dw.tlse))
    torch.cuda.synchronize()
    ref, ref_lse = ao.attention_custom(w.q, w.k, w.v, scale=w.scale, score_mod=lambda s, b, g, h, i, j: np.float64(np.float32(far)) * hidden, mask=None)
    assert float(np.max(np.abs(dw.out.cpu().numpy() - ref))) <= 1e-2
    # lse: the product far * log2(e) and its way back are rounded to fp32
    assert float(np.max(np.abs(dw.lse.cpu().numpy()[..., 0] - ref_lse) / (1e-3 + 2.0 ** -22 * np.abs(ref_lse)))) <= 1.0
    var.release()


@pytest.mark.parametrize("B,H,S,D", [(64, 8, 300, 128), (64, 8, 500, 128), (33, 16, 770, 128), (64, 8, 250, 64), (72, 8, 129, 64)])
@pytest.mark.parametrize("hidden", ["documents", "columns"])
def test_pairs_of_tiles_with_a_map(hidden, B, H, S, D):
    """Launches whose workgroups take a long and a short q-tile, with the classes of the pre-pass: the bits of the call without them, and fp32 torch."""
    import torch
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(S)
    q, k, v = (torch.randn(B, 1, H, S, D, generator=gen, device=dev).to(torch.bfloat16) for _ in range(3))
    ids = torch.from_numpy(inputs.doc_ids(B, S, seed=5, lo=20, hi=90)).to(dev)
    mask, aux = ("aux0[b * Sq + i] != aux0[b * Sk + j]", [ids]) if hidden == "documents" else ("(j % 64) == 5", [])
    var = fb.CustomVariant(None, mask, D, aux=aux, base_mask=fb.FL_MASK_CAUSAL)
    t = [fb.tensor_desc(x) for x in (q, k, v)]
    got = []
    for ws in (None, torch.empty(var.skip_workspace_size(t[0], t[1]), dtype=torch.uint8, device=dev)):
        out, lse = torch.full_like(q, float("nan")), torch.full((B, 1, H, S, 1), float("nan"), device=dev)
        fb.check(var.forward(*t, D ** -0.5, fb.tensor_desc(out), fb.tensor_desc(lse), workspace=ws))
        torch.cuda.synchronize()
        got.append((out, lse))
    var.release()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    i = torch.arange(S, device=dev)
    for b in range(0, B, 9):
        off = (i[None, :] > i[:, None]) | ((ids[b][:, None] != ids[b][None, :]) if hidden == "documents" else (i[None, :] % 64 == 5))
        s = (torch.matmul(q[b, 0].float(), k[b, 0].float().transpose(-1, -2).contiguous()) * D ** -0.5).masked_fill(off, float("-inf"))
        ref = torch.matmul(torch.softmax(s, -1), v[b, 0].float())
        assert float((got[1][0][b, 0].float() - ref).abs().max()) <= 2e-2    # the output's own rounding to bf16, values up to 4
