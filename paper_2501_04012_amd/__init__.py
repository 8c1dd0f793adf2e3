"""MI355X-native denoising step and cache-hit resume loop of a latent video
diffusion transformer, behind a C-ABI library.  `synth` (seeded inputs) imports
without the native library; everything else needs it built."""
import importlib

_binding = None


def __getattr__(name):
    if name in ("synth", "binding", "build"):
        return importlib.import_module("." + name, __name__)
    # the binding loads the native library on first use, and raises if it is missing; asking the import system for it
    # on every call cost as much as the rest of a call's host work
    global _binding
    if _binding is None:
        _binding = importlib.import_module(".binding", __name__)
    return getattr(_binding, name)
