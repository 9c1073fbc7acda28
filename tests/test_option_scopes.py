"""A call that needs another tolerance or split method for a while gives the
caller's back whichever way it returns: the handle's options are set by
mps_set_option and otherwise only through OptionScope (the autotuner, which sets
candidates in turn, restores them behind its loop)."""
import os
import re

from paper_1703_00387_amd import build as B


def test_options_change_only_in_scopes():
    found = []
    for f in sorted(os.listdir(B.CSRC)):
        if f == "tune.hip":
            continue
        text = open(os.path.join(B.CSRC, f)).read()
        body = re.sub(r"mps_status mps_set_option\(.*?^}", "", text, flags=re.M | re.S)
        found += [(f, m) for m in re.findall(r"h->(?:jac_\w+|split_method|warm_start) = [^=].*", body)]
    assert not found, found
