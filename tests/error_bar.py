"""A bar for attention outputs that holds at any context length."""
import numpy as np

# Largest difference over the row's root mean square (over its heads and dims).  The output of a row of n random tokens shrinks as
# 1 / sqrt(n), and so do the errors: rounding the output to bf16 is at most 2^-9 of a value, about 5 rms at the most; rounding every weight
# to bf16 adds independent errors of at most 2^-9 of a term each, whose sum is about 2^-9 / sqrt(3) of the rms and five times that at the
# most.  Together 1.5 % of the rms (measured: up to 1.8 %); the bar is four times that.  (The reference reads the stored e4m3 values, so an
# e4m3 cache has the same bar.)  A lost partial of 25 moves a row by about 20 % of its rms, an output of zeros by more than 100 %.
OF_RMS = 6e-2


def worst_of_rms(out, ref):
    """Largest difference of a row over the root mean square of its reference, over all rows."""
    ref = ref.reshape(len(ref), -1)
    rms = np.sqrt(np.mean(ref * ref, axis=1))
    return float(np.max(np.max(np.abs(out.reshape(ref.shape) - ref), axis=1) / rms))
