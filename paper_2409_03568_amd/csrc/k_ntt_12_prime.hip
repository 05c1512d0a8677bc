// Kernels of the NTT path for N = 2^12: encryption through prime-field transforms (see k_ntt_impl.hpp).
#include "k_ntt_impl.hpp"
CKKS_DEFINE_RING_PRIME(12)
