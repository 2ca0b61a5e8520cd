"""What a keyset takes from a context's budget: the bytes that vlp.h states and
the server's admission counts, to the byte."""
import os
import re

import pytest

import synth

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_keyset_takes_the_stated_bytes():
    from paper_2506_12761_amd import serve, vlp
    text = open(os.path.join(ROOT, "include", "vlp.h")).read()
    text = text[text.index("Load a client's evaluation keys"):text.index("vlp_status vlp_keyset_load")]
    stated = sum(int(b.replace(",", "")) for b in re.findall(r"\(([\d,]+) B\)", text))
    assert stated == serve.KEYSET_BYTES
    bk, ksk = synth.uniform_keys(3)
    with vlp.Context(0) as ctx:
        empty = vlp.vlp_mem_info(ctx.ctx)[0]
    with vlp.Context(0, hbm_budget=empty + stated) as ctx:
        ks = ctx.load_keys(bk, ksk)
        assert vlp.vlp_mem_info(ctx.ctx)[0] == empty + stated
        ctx.drop_keys(ks)
        assert vlp.vlp_mem_info(ctx.ctx)[0] == empty
    with vlp.Context(0, hbm_budget=empty + stated - 1) as ctx:
        with pytest.raises(vlp.VlpError) as e:
            ctx.load_keys(bk, ksk)
        assert e.value.status == vlp.VLP_EBUDGET
        assert vlp.vlp_mem_info(ctx.ctx)[0] == empty
