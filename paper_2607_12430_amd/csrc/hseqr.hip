// Complex Schur form of an upper Hessenberg matrix (the Schur decomposition
// of Alg. 2): the single-shift instance of the chain QR, matrices in the
// stacked layout.
#include "qrchain.hpp"

namespace msqrt {

template <typename T>
bool hseqr(hipStream_t st, int n, T* H, T* Z, HseqrWork& w, T hnorm) {
  return qr::schur_qr<qr::CplxRoute<T>>(st, n, H, Z, w, hnorm);
}

template bool hseqr<float>(hipStream_t, int, float*, float*, HseqrWork&, float);
template bool hseqr<double>(hipStream_t, int, double*, double*, HseqrWork&, double);

}  // namespace msqrt
