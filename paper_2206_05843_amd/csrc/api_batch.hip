// Batched solves: many independent matrices analysed as one block-diagonal
// system (levels per matrix), solved in one persistent launch.
#include <algorithm>
#include <cstring>

#include "common.h"

namespace {

__global__ void k_fill_mat_of_row(const int64_t *__restrict__ row_off, int32_t nmat, int32_t *mat_of_row) {
  for (int32_t m = blockIdx.x; m < nmat; m += gridDim.x)
    for (int64_t r = row_off[m] + threadIdx.x; r < row_off[m + 1]; r += blockDim.x) mat_of_row[r] = m;
}

// Global row pointers of the block-diagonal union (local pointers of matrix m
// occupy n_m + 1 entries at row_off[m] + m of the concatenated array).
__global__ void k_global_rp(int64_t total, const int32_t *__restrict__ mat_of_row, const int64_t *__restrict__ row_off,
                            const int64_t *__restrict__ nnz_off, const int32_t *__restrict__ rp_cat, int32_t *grp,
                            int64_t total_nnz) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= total; r += (int64_t)gridDim.x * blockDim.x) {
    if (r == total) {
      grp[r] = (int32_t)total_nnz;
      continue;
    }
    const int32_t m = mat_of_row[r];
    grp[r] = (int32_t)(nnz_off[m] + rp_cat[row_off[m] + m + (r - row_off[m])]);
  }
}

// Entries of row r shifted to global column numbers.
__global__ void k_global_entries(int64_t total, const int32_t *__restrict__ mat_of_row,
                                 const int64_t *__restrict__ row_off, const int32_t *__restrict__ grp,
                                 const int32_t *__restrict__ ci_cat, const double *__restrict__ va_cat, int32_t *gci,
                                 double *gva) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < total; r += (int64_t)gridDim.x * blockDim.x) {
    const int32_t off = (int32_t)row_off[mat_of_row[r]];
    for (int32_t q = grp[r]; q < grp[r + 1]; ++q) {
      gci[q] = ci_cat[q] + off;
      gva[q] = va_cat[q];
    }
  }
}

__global__ void k_mat_max(int64_t total, const int32_t *__restrict__ mat_of_row, const int32_t *__restrict__ lev1,
                          int32_t *mx) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < total; r += (int64_t)gridDim.x * blockDim.x)
    atomicMax(mx + mat_of_row[r], lev1[r]);
}

__global__ void k_combined_keys(int64_t total, const int32_t *__restrict__ mat_of_row, const int32_t *__restrict__ lvl_off,
                                const int32_t *__restrict__ lev1, int32_t *keys) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < total; r += (int64_t)gridDim.x * blockDim.x)
    keys[r] = lvl_off[mat_of_row[r]] + lev1[r];
}

__global__ void k_offset_copy(const int32_t *__restrict__ src, int32_t n, int32_t off, int32_t *dst) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = src[i] - off;
}

int bit_width64(int64_t v) {
  int b = 0;
  while (v > 0) ++b, v >>= 1;
  return b;
}

// How a batch is solved: nc columns a group (groups may overlap: 13 columns are
// four groups of 4), workgroups of wg threads, whether each has a CU's whole LDS,
// and the matrices in the persistent queue, the longest chain first.
struct BatchForm {
  int32_t nc = 1, wg = 512;
  bool whole = false;
  std::vector<int32_t> queue;
  std::vector<char> queued;  // per matrix
};

// Estimated microseconds, by which a form is chosen. A matrix in the queue is one
// workgroup's chain of windows: by columns x rows a level takes 1 x 8 0.17, 1 x 40
// 0.3, 1 x 300 1.8, 1 x 1,000 5.8, 1 x 3,000 14.3, 4 x 8 0.26, 4 x 300 5.5, 4 x 1,000
// 20.7, 4 x 3,000 51 with 512 threads; 256 threads take about 1.4 times as long,
// 1,024 0.85 times.
// Workgroups that share a CU share its rate of items (columns x rows), not the
// latency of the levels.
constexpr double kLevelUs = 0.12, kItemUs = 0.005;
double wg_factor(int32_t wg) { return wg <= 256 ? 1.4 : wg >= 1024 ? 0.85 : 1.0; }
double chain_us(int64_t rows, int32_t nlev, int32_t nc, int32_t wg) {
  return wg_factor(wg) * (kLevelUs * nlev + kItemUs * (double)(rows * nc));
}
// A level on the whole device: in LDS windows of nc columns spread over workgroups
// (1 column x 500 rows 1.1, 1 x 1,000 2.3; 16 columns in groups of one x 500 2.1, x
// 1,000 6.1), or as a launch of its own (4.2 and its data; 40 levels x 3,000 rows
// x 4 columns 167 against 1,390 in windows of four).
double window_level_us(int64_t rows, int32_t nrhs, int32_t nc) {
  return 0.4 + 0.0013 * (double)rows * (nc + 0.2 * nrhs);
}
double launch_level_us(int64_t rows, int32_t nrhs) { return 4.2 + 1.4e-5 * (double)rows * nrhs; }
bool level_in_windows(const Plan &P, int32_t l, int32_t nrhs, int32_t nc) {
  const int64_t rows = P.h_level_ptr[(size_t)l + 1] - P.h_level_ptr[(size_t)l];
  return level_fits_window(P, l, nc) && window_level_us(rows, nrhs, nc) <= launch_level_us(rows, nrhs);
}

// The form with nc columns a group, and its estimated time: the queue lasts as
// long as its longest chain, or as all its levels over the workgroups in flight and
// all its items over the CUs, and the matrices outside it follow one after another. Outside are those with a level too
// wide for an LDS window and, longest chain first, as many more as shorten the
// whole: one matrix of 40 levels of 3,000 rows, 4 columns, takes 2,057 us in the
// queue and 167 outside, 64 of them 2,663 and 10,257. Only matrices of 100 rows a
// level and more are worth a look.
double batch_form(const sptrsv_ctx *h, int32_t nrhs, int32_t nc, int32_t wg, int32_t cus, BatchForm &f) {
  const Plan &P = h->bat;
  const int32_t nm = h->b_nmat, groups = (nrhs + nc - 1) / nc;
  f.nc = nc;
  f.whole = (int64_t)nm * groups <= cus;
  f.wg = f.whole ? 1024 : wg;
  f.queued.assign((size_t)nm, 1);
  f.queue.clear();
  const int32_t most = f.whole ? cus : std::max(1, batch_resident_blocks(wg, batch_lds(wg)));
  std::vector<double> in((size_t)nm), out((size_t)nm, -1.0);  // out < 0: stays in the queue
  double outside = 0.0;
  int64_t levels = 0, rows_in = 0;  // of the queue
  for (int32_t m = 0; m < nm; ++m) {
    const bool fits = thin_window_bytes(h->b_widest[(size_t)m], 0, 1, nc, kWidths) <= thin_win_bytes();
    const int32_t nl = h->b_nlev[(size_t)m];
    in[(size_t)m] = chain_us(h->b_n[(size_t)m], nl, nc, f.wg);
    if (!fits || h->b_n[(size_t)m] >= (int64_t)100 * nl) {
      out[(size_t)m] = 5.0;
      for (int64_t l = h->b_lvl_off[(size_t)m]; l < h->b_lvl_off[(size_t)m + 1]; ++l) {
        const int64_t rows = P.h_level_ptr[(size_t)l + 1] - P.h_level_ptr[(size_t)l];
        out[(size_t)m] += level_in_windows(P, (int32_t)l, nrhs, nc) ? window_level_us(rows, nrhs, nc)
                                                                    : launch_level_us(rows, nrhs);
      }
    }
    if (!fits) {
      f.queued[(size_t)m] = 0;
      outside += out[(size_t)m];
    } else {
      f.queue.push_back(m);
      levels += nl;
      rows_in += h->b_n[(size_t)m];
    }
  }
  std::stable_sort(f.queue.begin(), f.queue.end(),
                   [&](int32_t a, int32_t b) { return in[(size_t)a] > in[(size_t)b]; });
  // widest level of the queue from its j-th matrix on, which decides how many workgroups share a CU
  std::vector<int64_t> widest(f.queue.size() + 1, 0);
  for (size_t j = f.queue.size(); j-- > 0;) widest[j] = std::max(widest[j + 1], h->b_widest[(size_t)f.queue[j]]);
  auto total = [&](size_t j) {  // the first j of the queue outside; 12: copies of b and x
    const int64_t need = thin_window_bytes(widest[j], 0, 1, nc, kWidths) + thin_ctl_bytes();
    const int64_t fit = (int64_t)cus * std::max<int64_t>(1, (thin_win_bytes() + thin_ctl_bytes()) / need);
    const double longest = j < f.queue.size() ? in[(size_t)f.queue[j]] : 0.0;
    const double slots = (double)std::min<int64_t>(most, fit);
    const double all = wg_factor(f.wg) * kLevelUs * (double)levels * groups / slots +
                       (f.whole ? wg_factor(f.wg) : 1.0) * kItemUs * (double)rows_in * nc * groups / cus;
    return outside + (outside > 0.0 ? 12.0 : 0.0) + std::max(longest, all);
  };
  double us = total(0);
  size_t leave = 0;
  const double outside0 = outside;
  for (size_t j = 0; j < f.queue.size() && out[(size_t)f.queue[j]] >= 0.0; ++j) {
    outside += out[(size_t)f.queue[j]];
    levels -= h->b_nlev[(size_t)f.queue[j]];
    rows_in -= h->b_n[(size_t)f.queue[j]];
    const double t = total(j + 1);
    if (t < (outside0 == 0.0 && leave == 0 ? 0.8 : 1.0) * us) {
      us = t;
      leave = j + 1;
    }
  }
  for (size_t j = 0; j < leave; ++j) f.queued[(size_t)f.queue[j]] = 0;
  f.queue.erase(f.queue.begin(), f.queue.begin() + (ptrdiff_t)leave);
  return us;
}

// The best of 1 and 4 columns a group or, where no CU is shared, 8 and all. Few
// tasks take one column each: the chains run side by side on CUs that would be idle
// (16 matrices of 40 levels of 600 rows, 16 columns: 145 us against 541 in groups of
// 4 and 1,307 with all columns of a matrix in one workgroup). With many deep ones 4
// columns are best, as most levels (a few rows wide) then fit one wave (512 matrices
// of 1,000 to 50,000 rows x 16 columns: 3.91 ms in groups of 4 with 256 threads,
// 4.15 in groups of 8 with 512, 6.3 in groups of 2); where a workgroup has a CU to
// itself and there are several for each CU, more (512 matrices of 600 levels of 8
// rows, 16 columns, 1,024 threads: 1,220 us in groups of 4, 731 in one).
// What stays slower than one task a matrix with all its columns and narrower
// records: one column, a few matrices, levels of 600 to 1,500 rows, 1,024 threads
// (16 matrices of 40 levels of 600 rows: 135 us against 111).
BatchForm best_form(const sptrsv_ctx *h, int32_t nrhs, int32_t wg, int32_t cus) {
  BatchForm best;
  double best_us = 0.0;
  int32_t last = 0;
  for (int32_t nc : {1, 4, 8, nrhs}) {
    if (nc > nrhs || nc == last) continue;
    last = nc;
    BatchForm f;
    const double us = batch_form(h, nrhs, nc, wg, cus, f);
    if (nc > 4 && !f.whole && wg < 1024) continue;
    if (best_us == 0.0 || us < best_us) {
      best_us = us;
      best = std::move(f);
    }
  }
  return best;
}

// Per-matrix LDS windows for nrhs (cached). The matrices of the queue have windows
// as large as lets several workgroups share a CU (batch_lds), or as the widest
// queued level needs; with no more tasks than CUs they take a whole CU's LDS (and
// 1,024 threads). The others are solved level by level: narrow levels in thin runs,
// the others one device-wide launch each, as a single plan's mode-0 schedule.
sptrsv_status_t batch_windows(sptrsv_ctx *h, int32_t nrhs, int32_t wg, hipStream_t s) {
  if (h->b_win_nrhs == nrhs && h->b_win_wg == wg) return SPTRSV_OK;
  Plan &P = h->bat;
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const BatchForm form = best_form(h, nrhs, wg, std::max(cus, 1));
  const int32_t nc = form.nc;
  const std::vector<char> &fits = form.queued;
  P.h_win.clear();
  h->b_h_mwin.assign((size_t)h->b_nmat + 1, 0);
  h->b_wide.clear();
  std::vector<uint8_t> flag((size_t)h->b_nmat, 0);
  int64_t cap = form.whole ? thin_win_bytes() : batch_lds(wg) - thin_ctl_bytes();
  for (int32_t m = 0; m < h->b_nmat; ++m) {
    flag[(size_t)m] = fits[(size_t)m] ? 0 : 1;
    if (fits[(size_t)m]) cap = std::max(cap, thin_window_bytes(h->b_widest[(size_t)m], 0, 1, nc, kWidths));
  }
  h->b_ncol = nc;
  h->b_wg = form.wg;
  h->b_lds = (int32_t)cap + thin_ctl_bytes();
  for (int32_t m = 0; m < h->b_nmat; ++m) {
    h->b_h_mwin[(size_t)m] = (int32_t)P.h_win.size();
    if (fits[(size_t)m])
      cut_windows(P, (int32_t)h->b_lvl_off[(size_t)m], (int32_t)h->b_lvl_off[(size_t)m + 1], nc, form.wg, cap, true,
                  P.h_win);
  }
  h->b_h_mwin[(size_t)h->b_nmat] = (int32_t)P.h_win.size();
  for (int32_t m = 0; m < h->b_nmat; ++m) {
    if (fits[(size_t)m]) continue;
    BatchWide bw;
    bw.m = m;
    const int32_t l0 = (int32_t)h->b_lvl_off[(size_t)m], l1 = (int32_t)h->b_lvl_off[(size_t)m + 1];
    for (int32_t l = l0; l < l1; ++l) {
      const bool thin = level_in_windows(P, l, nrhs, nc);
      if (!bw.runs.empty() && thin && bw.runs.back().thin && bw.runs.back().l1 == l)
        bw.runs.back().l1 = l + 1;
      else
        bw.runs.push_back(Run{l, l + 1, thin});
    }
    for (Run &r : bw.runs)
      if (r.thin) {
        r.wi = (int32_t)P.h_win.size();
        r.nw = cut_windows(P, r.l0, r.l1, nc, form.wg, thin_win_bytes(), true, P.h_win);
      }
    h->b_wide.push_back(std::move(bw));
  }
  const std::vector<int32_t> &q = form.queue;
  h->b_nq = (int32_t)q.size();
  HIPCHK(h, h->b_order.reserve(std::max<size_t>(q.size(), 1)));
  if (!q.empty()) HIPCHK(h, hipMemcpy(h->b_order.p, q.data(), sizeof(int32_t) * q.size(), hipMemcpyHostToDevice));
  HIPCHK(h, h->b_wide_flag.reserve((size_t)h->b_nmat));
  HIPCHK(h, hipMemcpy(h->b_wide_flag.p, flag.data(), (size_t)h->b_nmat, hipMemcpyHostToDevice));
  h->b_win_nrhs = -1;  // until the images are built
  STCHK(build_images(h, P, nc, s));
  HIPCHK(h, h->b_mwin.alloc((size_t)h->b_nmat + 1));
  HIPCHK(h, hipMemcpy(h->b_mwin.p, h->b_h_mwin.data(), sizeof(int32_t) * ((size_t)h->b_nmat + 1),
                      hipMemcpyHostToDevice));
  h->b_win_nrhs = nrhs;
  h->b_win_wg = wg;
  return SPTRSV_OK;
}

// The matrices taken out of the persistent launch, level by level.
sptrsv_status_t batch_wide_solves(sptrsv_ctx *h, int32_t nrhs, hipStream_t s) {
  Plan &P = h->bat;
  const sptrsv_schedule_t d = default_schedule();
  for (const BatchWide &bw : h->b_wide)
    for (const Run &r : bw.runs) {
      if (r.thin) {
        const int32_t p0 = P.h_level_ptr[(size_t)r.l0];
        if (thin_piped(r.nw, kWaitTicks))
          HIPCHK(h, launch_fill_pending(p0, P.h_level_ptr[(size_t)r.l1] - p0, nrhs, nullptr, P.xp.p, s));
        HIPCHK(h, launch_thin_run(h->b_wg, P.win.p + r.wi, r.nw, nrhs, thin_args(P), h->d_err.p, s, nullptr, 0.f,
                                  h->b_ncol, kWaitTicks));
      } else
        HIPCHK(h, launch_wide_level(d.wide_threads, 1, P.h_level_ptr[(size_t)r.l0], P.h_level_ptr[(size_t)r.l1], nrhs,
                                    P.srp.p, P.sci.p, P.sva.p, P.sdg.p, P.ell_c.p, P.ell_v.p, P.bp.p, P.xp.p,
                                    h->d_err.p, s));
    }
  return SPTRSV_OK;
}

}  // namespace

extern "C" {

sptrsv_status_t sptrsv_batch_analyze(sptrsv_handle_t h, int32_t nmat, const int32_t *h_n, const int64_t *h_row_off,
                                     const int64_t *h_nnz_off, const int32_t *d_row_ptr_cat, const int32_t *d_col_cat,
                                     const double *d_val_cat, hipStream_t s) {
  if (!h || nmat < 1 || !h_n || !h_row_off || !h_nnz_off || !d_row_ptr_cat || !d_col_cat || !d_val_cat)
    return SPTRSV_ERR_ARG;
  h->last_error.clear();
  h->b_ready = false;
  h->b_win_nrhs = -1;
  // host bookkeeping: offsets must describe back-to-back matrices
  std::vector<int64_t> row_off((size_t)nmat + 1), nnz_off((size_t)nmat + 1);
  int64_t acc = 0;
  for (int32_t m = 0; m < nmat; ++m) {
    if (h_n[m] < 1 || h_row_off[m] != acc) return set_err(h, SPTRSV_ERR_ARG, "batch: bad size/offset of matrix %d", m);
    row_off[(size_t)m] = acc;
    acc += h_n[m];
  }
  row_off[(size_t)nmat] = acc;
  const int64_t total = acc;
  if (total >= (int64_t)1 << 31) return set_err(h, SPTRSV_ERR_OVERFLOW, "batch: too many rows");
  for (int32_t m = 0; m < nmat; ++m) nnz_off[(size_t)m] = h_nnz_off[m];
  int32_t last_nnz = 0;
  HIPCHK(h, hipMemcpyAsync(&last_nnz, d_row_ptr_cat + (row_off[(size_t)nmat - 1] + nmat - 1 + h_n[nmat - 1]),
                           sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipStreamSynchronize(s));
  const int64_t total_nnz = nnz_off[(size_t)nmat - 1] + last_nnz;
  nnz_off[(size_t)nmat] = total_nnz;
  for (int32_t m = 0; m < nmat; ++m)
    if (nnz_off[(size_t)m] < 0 || nnz_off[(size_t)m + 1] < nnz_off[(size_t)m])
      return set_err(h, SPTRSV_ERR_ARG, "batch: bad nonzero offset of matrix %d", m);
  if (total_nnz >= (int64_t)1 << 31) return set_err(h, SPTRSV_ERR_OVERFLOW, "batch: too many nonzeros");
  h->b_nmat = nmat;
  h->b_n.assign(h_n, h_n + nmat);
  h->b_row_off = row_off;
  DArr<int64_t> d_nnz_off;
  HIPCHK(h, h->b_row_off_d.alloc((size_t)nmat + 1));
  HIPCHK(h, d_nnz_off.alloc((size_t)nmat + 1));
  HIPCHK(h, hipMemcpy(h->b_row_off_d.p, row_off.data(), sizeof(int64_t) * ((size_t)nmat + 1), hipMemcpyHostToDevice));
  HIPCHK(h, hipMemcpy(d_nnz_off.p, nnz_off.data(), sizeof(int64_t) * ((size_t)nmat + 1), hipMemcpyHostToDevice));
  // block-diagonal union in global numbering
  HIPCHK(h, h->b_mat_of_row.alloc((size_t)total));
  HIPCHK(h, h->b_rp.alloc((size_t)total + 1));
  HIPCHK(h, h->b_ci.alloc((size_t)total_nnz));
  HIPCHK(h, h->b_va.alloc((size_t)total_nnz));
  hipLaunchKernelGGL(k_fill_mat_of_row, dim3(std::min(nmat, 4096)), dim3(256), 0, s, h->b_row_off_d.p, nmat,
                     h->b_mat_of_row.p);
  hipLaunchKernelGGL(k_global_rp, dim3(grid_for(total + 1, 256, 8192)), dim3(256), 0, s, total, h->b_mat_of_row.p,
                     h->b_row_off_d.p, d_nnz_off.p, d_row_ptr_cat, h->b_rp.p, total_nnz);
  HIPCHK(h, hipGetLastError());
  int32_t *aux = h->d_aux.p;
  HIPCHK(h, hipMemsetAsync(aux + 1, 0, sizeof(int32_t), s));
  // each matrix's local pointers must be well formed before entries are read
  HIPCHK(h, launch_validate((int32_t)total, (int32_t)total_nnz, h->b_rp.p, d_col_cat, d_val_cat, aux + 1, s));
  int32_t bits = 0;
  HIPCHK(h, hipMemcpyAsync(&bits, aux + 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipStreamSynchronize(s));
  if (bits & (EB_ARG | EB_NOT_LOWER))  // malformed pointers, or a negative local column
    return set_err(h, status_from_bits(bits & (EB_ARG | EB_NOT_LOWER)), "batch: malformed matrix (bits 0x%x)", bits);
  hipLaunchKernelGGL(k_global_entries, dim3(grid_for(total, 256, 8192)), dim3(256), 0, s, total, h->b_mat_of_row.p,
                     h->b_row_off_d.p, h->b_rp.p, d_col_cat, d_val_cat, h->b_ci.p, h->b_va.p);
  HIPCHK(h, hipGetLastError());
  HIPCHK(h, hipMemsetAsync(aux + 1, 0, sizeof(int32_t), s));
  HIPCHK(h, launch_validate((int32_t)total, (int32_t)total_nnz, h->b_rp.p, h->b_ci.p, h->b_va.p, aux + 1, s));
  HIPCHK(h, hipMemcpyAsync(&bits, aux + 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipStreamSynchronize(s));
  if (bits) return set_err(h, status_from_bits(bits), "batch: invalid matrix (bits 0x%x)", bits);
  // levels of every row (longest path; matrices are independent)
  const int32_t n = (int32_t)total;
  Plan &P = h->bat;
  P = Plan{};
  P.sched = default_schedule();
  P.n = n;
  P.nnz = total_nnz;
  DArr<int32_t> lev1, keys, ktmp, vtmp, hist, mx, lvl_off_d;
  DArr<long long> cnt, ex, hist64;
  HIPCHK(h, lev1.alloc(n));
  HIPCHK(h, keys.alloc(n));
  HIPCHK(h, ktmp.alloc(n));
  HIPCHK(h, vtmp.alloc(n));
  HIPCHK(h, cnt.alloc(n));
  HIPCHK(h, ex.alloc(n));
  HIPCHK(h, mx.alloc(nmat));
  HIPCHK(h, lvl_off_d.alloc(nmat));
  const size_t hn = radix_hist_elems(n);
  HIPCHK(h, hist.alloc(hn));
  HIPCHK(h, hist64.alloc(hn));
  const size_t scr = std::max(scan_scratch_elems((int64_t)hn), scan_scratch_elems(n)) + 16;
  if (h->scan_tmp.n < scr) HIPCHK(h, h->scan_tmp.alloc(scr));
  HIPCHK(h, hipMemsetAsync(aux, 0, 8 * sizeof(int32_t), s));
  HIPCHK(h, hipMemsetAsync(lev1.p, 0, sizeof(int32_t) * (size_t)n, s));
  HIPCHK(h, hipMemsetAsync(mx.p, 0, sizeof(int32_t) * (size_t)nmat, s));
  HIPCHK(h, launch_levels(n, h->b_rp.p, h->b_ci.p, lev1.p, reinterpret_cast<unsigned *>(aux), aux + 1, s));
  hipLaunchKernelGGL(k_mat_max, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, (int64_t)n, h->b_mat_of_row.p, lev1.p,
                     mx.p);
  HIPCHK(h, hipGetLastError());
  h->b_nlev.assign((size_t)nmat, 0);
  HIPCHK(h, hipMemcpyAsync(h->b_nlev.data(), mx.p, sizeof(int32_t) * (size_t)nmat, hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipMemcpyAsync(&bits, aux + 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipStreamSynchronize(s));
  if (bits) return set_err(h, status_from_bits(bits), "batch: level construction failed (bits 0x%x)", bits);
  h->b_lvl_off.assign((size_t)nmat + 1, 0);
  std::vector<int32_t> lvl_off32((size_t)nmat);
  for (int32_t m = 0; m < nmat; ++m) {
    lvl_off32[(size_t)m] = (int32_t)h->b_lvl_off[(size_t)m];
    h->b_lvl_off[(size_t)m + 1] = h->b_lvl_off[(size_t)m] + h->b_nlev[(size_t)m];
  }
  const int32_t nlev = (int32_t)h->b_lvl_off[(size_t)nmat];
  P.nlev = nlev;
  HIPCHK(h, hipMemcpy(lvl_off_d.p, lvl_off32.data(), sizeof(int32_t) * (size_t)nmat, hipMemcpyHostToDevice));
  // positions grouped by matrix, then level, rows ascending (stable sort)
  hipLaunchKernelGGL(k_combined_keys, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, (int64_t)n, h->b_mat_of_row.p,
                     lvl_off_d.p, lev1.p, keys.p);
  HIPCHK(h, hipGetLastError());
  HIPCHK(h, P.level_ptr.alloc((size_t)nlev + 1));
  HIPCHK(h, P.perm.alloc(n));
  HIPCHK(h, P.iperm.alloc(n));
  HIPCHK(h, P.row_level.alloc(n));
  HIPCHK(h, launch_iota(P.perm.p, n, s));
  HIPCHK(h, launch_radix_by_key(keys.p, P.perm.p, ktmp.p, vtmp.p, n, bit_width64(nlev), hist.p, hist64.p,
                                h->scan_tmp.p, s));
  HIPCHK(h, launch_level_ptr_from_sorted(keys.p, n, P.level_ptr.p, nlev, s));
  HIPCHK(h, launch_invert_perm(P.perm.p, n, P.iperm.p, s));
  HIPCHK(h, launch_sub1(lev1.p, n, P.row_level.p, s));
  // level-ordered copy, overflow prefix, statistics
  HIPCHK(h, P.srp.alloc((size_t)n + 1));
  HIPCHK(h, launch_count_off(P.perm.p, h->b_rp.p, n, cnt.p, s));
  HIPCHK(h, launch_scan_i64(cnt.p, ex.p, n, h->scan_tmp.p, s));
  HIPCHK(h, launch_ptr_from_scan(ex.p, cnt.p, n, P.srp.p, aux + 1, s));
  const int64_t noff = total_nnz - n;
  HIPCHK(h, P.sci.alloc((size_t)std::max<int64_t>(noff, 1)));
  HIPCHK(h, P.sva.alloc((size_t)std::max<int64_t>(noff, 1)));
  HIPCHK(h, P.sdg.alloc(n));
  HIPCHK(h, launch_fill_solve(n, P.perm.p, P.iperm.p, h->b_rp.p, h->b_ci.p, h->b_va.p, P.srp.p, P.sci.p, P.sva.p,
                              P.sdg.p, s));
  HIPCHK(h, P.ell_c.alloc(n));
  HIPCHK(h, P.ell_v.alloc((size_t)2 * n));
  HIPCHK(h, launch_fill_ell(n, P.srp.p, P.sci.p, P.sva.p, P.ell_c.p, P.ell_v.p, s));
  HIPCHK(h, P.tp.alloc(kThinCtlWords));
  HIPCHK(h, hipMemsetAsync(P.tp.p, 0, kThinCtlWords * sizeof(unsigned), s));
  HIPCHK(h, P.lv_rows.alloc(nlev));
  HIPCHK(h, P.lv_nnz.alloc(nlev));
  HIPCHK(h, P.lv_cost.alloc(nlev));
  HIPCHK(h, launch_level_stats(nlev, P.level_ptr.p, P.srp.p, P.lv_rows.p, P.lv_nnz.p, P.lv_cost.p,
                               reinterpret_cast<long long *>(aux + 4), s));
  P.h_level_ptr.resize((size_t)nlev + 1);
  HIPCHK(h, hipMemcpyAsync(P.h_level_ptr.data(), P.level_ptr.p, sizeof(int32_t) * ((size_t)nlev + 1),
                           hipMemcpyDeviceToHost, s));
  P.h_lv_nnz.resize((size_t)nlev);
  HIPCHK(h, hipMemcpyAsync(P.h_lv_nnz.data(), P.lv_nnz.p, sizeof(int64_t) * (size_t)nlev, hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipMemcpyAsync(&bits, aux + 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(h, hipStreamSynchronize(s));
  if (bits) return set_err(h, status_from_bits(bits), "batch: plan construction failed (bits 0x%x)", bits);
  STCHK(build_extra_hist(h, P, s));
  h->b_widest.assign((size_t)nmat, 0);
  for (int32_t m = 0; m < nmat; ++m)
    for (int64_t l = h->b_lvl_off[(size_t)m]; l < h->b_lvl_off[(size_t)m + 1]; ++l)
      h->b_widest[(size_t)m] =
          std::max<int64_t>(h->b_widest[(size_t)m], P.h_level_ptr[(size_t)l + 1] - P.h_level_ptr[(size_t)l]);
  HIPCHK(h, h->b_q.alloc(2));
  HIPCHK(h, hipMemset(h->b_q.p, 0, 2 * sizeof(unsigned)));
  P.ready = true;
  h->b_ready = true;
  return SPTRSV_OK;
}

sptrsv_status_t sptrsv_batch_solve(sptrsv_handle_t h, int32_t nrhs, const double *d_b_cat, double *d_x_cat,
                                   hipStream_t s) {
  if (!h) return SPTRSV_ERR_ARG;
  if (!h->b_ready) return set_err(h, SPTRSV_ERR_STATE, "batch: not analysed");
  if (nrhs < 1 || !d_b_cat || !d_x_cat) return set_err(h, SPTRSV_ERR_ARG, "batch solve args");
  Plan &P = h->bat;
  const size_t len = sizeof(double) * (size_t)P.n * (size_t)nrhs;
  const char *b0 = reinterpret_cast<const char *>(d_b_cat), *x0 = reinterpret_cast<const char *>(d_x_cat);
  if (b0 < x0 + len && x0 < b0 + len) return set_err(h, SPTRSV_ERR_ARG, "b and x overlap");
  STCHK(ensure_work(h, P, nrhs));
  const int32_t wg = effective_sched(P, nrhs).wg_threads;
  STCHK(batch_windows(h, nrhs, wg, s));
  if (h->b_nq > 0) {
    const int32_t tasks = h->b_nq * ((nrhs + h->b_ncol - 1) / h->b_ncol);
    const int32_t grid = std::min(tasks, batch_resident_blocks(h->b_wg, h->b_lds));
    ThinArgs ta = thin_args(P);
    ta.rio = RowsIO{d_b_cat, d_x_cat, P.perm.p, nullptr, nullptr, nullptr, 1, 1};
    ta.lds = h->b_lds;
    HIPCHK(h, launch_batch_run(h->b_wg, h->b_nq, grid, h->b_order.p, h->b_mwin.p, P.win.p, nrhs, h->b_ncol,
                               h->b_row_off_d.p, ta, h->b_q.p, h->d_err.p, s));
  }
  if (!h->b_wide.empty()) {
    HIPCHK(h, launch_batch_gather(P.n, nrhs, d_b_cat, h->b_mat_of_row.p, h->b_row_off_d.p, P.iperm.p,
                                  h->b_wide_flag.p, P.bp.p, s));
    STCHK(batch_wide_solves(h, nrhs, s));
    HIPCHK(h, launch_batch_scatter(P.n, nrhs, P.xp.p, h->b_mat_of_row.p, h->b_row_off_d.p, P.iperm.p,
                                   h->b_wide_flag.p, d_x_cat, s));
  }
  return SPTRSV_OK;
}

sptrsv_status_t sptrsv_batch_solve_looped(sptrsv_handle_t h, int32_t nrhs, const double *d_b_cat, double *d_x_cat,
                                          hipStream_t s) {
  if (!h) return SPTRSV_ERR_ARG;
  if (!h->b_ready) return set_err(h, SPTRSV_ERR_STATE, "batch: not analysed");
  if (nrhs < 1 || !d_b_cat || !d_x_cat) return set_err(h, SPTRSV_ERR_ARG, "batch solve args");
  Plan &P = h->bat;
  STCHK(ensure_work(h, P, nrhs));
  const int32_t wg = effective_sched(P, nrhs).wg_threads;
  STCHK(batch_windows(h, nrhs, wg, s));
  HIPCHK(h, launch_batch_gather(P.n, nrhs, d_b_cat, h->b_mat_of_row.p, h->b_row_off_d.p, P.iperm.p, nullptr, P.bp.p,
                                s));
  HIPCHK(h, launch_fill_pending(0, P.n, nrhs, nullptr, P.xp.p, s));
  for (int32_t m = 0; m < h->b_nmat; ++m) {
    const int32_t wi = h->b_h_mwin[(size_t)m], nw = h->b_h_mwin[(size_t)m + 1] - wi - 1;
    if (nw >= 1)
      HIPCHK(h, launch_thin_run(h->b_wg, P.win.p + wi, nw, nrhs, thin_args(P), h->d_err.p, s, nullptr, 0.f,
                                h->b_ncol, kWaitTicks));
  }
  STCHK(batch_wide_solves(h, nrhs, s));
  HIPCHK(h, launch_batch_scatter(P.n, nrhs, P.xp.p, h->b_mat_of_row.p, h->b_row_off_d.p, P.iperm.p, nullptr, d_x_cat,
                                 s));
  return SPTRSV_OK;
}

sptrsv_status_t sptrsv_batch_levels(sptrsv_handle_t h, int32_t i, int32_t *nlev, int32_t *d_level_ptr,
                                    int32_t *d_level_rows, hipStream_t s) {
  if (!h) return SPTRSV_ERR_ARG;
  if (!h->b_ready) return set_err(h, SPTRSV_ERR_STATE, "batch: not analysed");
  if (i < 0 || i >= h->b_nmat) return set_err(h, SPTRSV_ERR_ARG, "batch: matrix %d out of range", i);
  const int32_t nl = h->b_nlev[(size_t)i];
  if (nlev) *nlev = nl;
  const int32_t l0 = (int32_t)h->b_lvl_off[(size_t)i];
  const int32_t p0 = (int32_t)h->b_row_off[(size_t)i], n = h->b_n[(size_t)i];
  if (d_level_ptr)
    hipLaunchKernelGGL(k_offset_copy, dim3(grid_for(nl + 1, 256, 1024)), dim3(256), 0, s, h->bat.level_ptr.p + l0,
                       nl + 1, p0, d_level_ptr);
  if (d_level_rows)
    hipLaunchKernelGGL(k_offset_copy, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, h->bat.perm.p + p0, n, p0,
                       d_level_rows);
  HIPCHK(h, hipGetLastError());
  HIPCHK(h, hipStreamSynchronize(s));
  return SPTRSV_OK;
}

}  // extern "C"
