"""Launch policy of the decode on the host: sizes and orders that the kernel's merge and its workgroups rely on.  No launch is made."""
import pytest

from tests.test_library_abi import fake_struct, kb

SPLITS_OF_THE_MERGE = 32  # rows of partial results that the merge of a query head holds


def most_splits(c, context):
    """The most splits a sequence may take, from the workspace: B * H_q * (splits + 4 correction parts) rows of 132 floats."""
    per_row, rest = divmod(kb.kvlinc_decode_workspace_bytes(c, context), c.B * c.H_q * 132 * 4)
    assert rest == 0
    return per_row - 4


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("corr", [True, False])
def test_no_sequence_takes_more_splits_than_the_merge_holds(bits, corr):
    off = {} if corr else dict(S=0, S16=0, P=0, Wq=0, Wk=0)
    for H_kv in (1, 2, 3, 4, 5, 6, 7, 8, 16, 32):
        for gq in range(1, 9):
            for B in list(range(1, 41)) + [64, 144, 257]:
                c = fake_struct(B=B, H_q=H_kv * gq, H_kv=H_kv, bits=bits, max_groups=1025, **off)
                for context in (1, 128, 700, 1281, 4096, 9000, 17000, 20000, 32768, 70000, 131072):
                    splits = most_splits(c, context)
                    assert 1 <= splits <= SPLITS_OF_THE_MERGE, (B, H_kv, gq, context, splits)
