"""MI355X-native staged multi-tenant CNN inference (arXiv 2111.14255): Python side of libmtsched.so."""
import os as _os


def _runtime_environment():
    """Settings the HIP runtime reads when it initialises (the first HIP call of the process), so they are made on
    import of the package, before anything touches the GPU.

    GPU_MAX_HW_QUEUES: hardware queues the runtime shares among the HIP streams of the process.  Passes run on queues of
    the library's own; the streams of the probes and of the framework share these.  Raised to 8 if lower (HIP's default is
    4); a larger value already set is kept; MTSCHED_HW_QUEUES=<n> (1..32) forces a value, for measurements.
    HIP_FORCE_DEV_KERNARG: kernel arguments of HIP launches in device memory; in host memory every launch starts with a
    read over the host link (848 against 578 us for 98 launches).
    HSA_ENABLE_INTERRUPT=0: waits of the HIP runtime poll the signal instead of sleeping until the driver's interrupt wakes
    the thread (mt_run polls its own signals in any case).  The price is a busy host thread per waiting call; a value
    already set in the environment is kept.

    MTSCHED_KEEP_ENV=1 switches all of this off: the process environment is left as it is (for hosts that set these
    variables themselves, or that must not have a polling thread).  None of the settings has any effect when the HIP
    runtime was initialised before this package is imported."""
    if _os.environ.get("MTSCHED_KEEP_ENV", "") not in ("", "0"):
        return
    want = _os.environ.get("MTSCHED_HW_QUEUES")
    try:
        have = int(_os.environ.get("GPU_MAX_HW_QUEUES", "0") or 0)
    except ValueError:
        have = 0
    if want:
        _os.environ["GPU_MAX_HW_QUEUES"] = str(max(1, min(32, int(want))))
    elif have < 8:
        _os.environ["GPU_MAX_HW_QUEUES"] = "8"
    _os.environ.setdefault("HIP_FORCE_DEV_KERNARG", "1")
    _os.environ.setdefault("HSA_ENABLE_INTERRUPT", "0")


_runtime_environment()

from . import binding  # noqa: E402,F401
