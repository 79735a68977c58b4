// Real Schur form A = Q T Q^T of the remark on real input in Sec. 2.2.1: the
// Francis double-shift instance of the chain QR (H and Z real n x n, ld n; T
// quasi-upper-triangular with standardised 2x2 blocks).
#include "qrchain.hpp"

namespace msqrt {

template <typename T>
bool rhseqr(hipStream_t st, int n, T* H, T* Z, HseqrWork& w, T hnorm) {
  return qr::schur_qr<qr::RealRoute<T>>(st, n, H, Z, w, hnorm);
}

template bool rhseqr<float>(hipStream_t, int, float*, float*, HseqrWork&, float);
template bool rhseqr<double>(hipStream_t, int, double*, double*, HseqrWork&, double);

}  // namespace msqrt
