"""The build shows the compiler's warnings (no GPU)."""
import subprocess
import sys

from paper_2505_24504_amd import build

NOTICE = "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)\n"


def test_warnings_are_shown_beside_the_feature_notice(capsys):
    """The host pass's notice about the device feature comes with every file and is left out;
    a warning of the same file is not."""
    warning = "fv.hip:179:1: warning: failed to meet occupancy target [-Wpass-failed]\n"
    for text, shown in ((NOTICE * 5, ""), (NOTICE + warning + NOTICE, warning), ("", "")):
        p = subprocess.Popen([sys.executable, "-c", f"import sys; sys.stdout.write({text!r})"],
                             stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        build._wait(("fv.hip", p))
        assert capsys.readouterr().err == shown
