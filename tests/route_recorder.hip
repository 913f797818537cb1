// Stand-ins for the library's launchers that write down what they are asked for instead of launching it: linked with the host side of
// the C ABI they show, without a GPU, which kernels a call takes and with what.  One line a launch, "launcher key=value ...".
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>

#include "../paper_2401_04658_amd/csrc/la2_internal.h"

namespace {
std::string lines;
hipError_t note(const char* format, ...) {
  char line[1024];
  va_list a;
  va_start(a, format);
  vsnprintf(line, sizeof(line), format, a);
  va_end(a);
  lines += line;
  lines += '\n';
  return hipSuccess;
}
const char* text(const la2::ScanParams& p) {
  static char line[768];
  snprintf(line, sizeof(line),
           "batch=%d heads=%d n=%d nchunks=%d chunk_tokens=%d nscan=%d keep=%d plain=%d split=%d prefix=%d ragged=%d packed=%d pairs=%d "
           "states=%p init=%p fin=%p acc=%p rstd=%p w=%p",
           p.batch, p.heads, p.n, p.nchunks, p.chunk_tokens, p.nscan, p.keep, p.plain, p.value_split, p.self_prefix, p.ragged_state,
           p.cu_seqlens != nullptr, p.wg_map != nullptr ? p.wg_pairs : 0, (void*)p.states, (void*)p.init[0], (void*)p.fin[0],
           (void*)p.acc_states, (void*)p.rstd, p.w[0]);
  return line;
}
}  // namespace

extern "C" int routes_take(char* out, int size) {
  const int n = (int)lines.size();
  if (n < size) memcpy(out, lines.c_str(), (size_t)n + 1);
  lines.clear();
  return n < size ? n : -1;
}

namespace la2 {
int block_size_bf16(int) { return 64; }
int block_size_f32(int) { return 32; }
bool stream_state(int64_t, int) { return false; }
hipError_t launch_scan_bf16(int, int d, bool rev, const ScanParams& p, hipStream_t) { return note("scan_bf16 d=%d rev=%d %s", d, rev, text(p)); }
hipError_t launch_chunk_states_bf16(int, int d, bool rev, const ScanParams& p, hipStream_t) {
  return note("chunk_states_bf16 d=%d rev=%d %s", d, rev, text(p));
}
hipError_t launch_scan_wide(int, int d, bool rev, bool state_only, const ScanParams& p, hipStream_t) {
  return note("%s d=%d rev=%d %s", state_only ? "chunk_states_wide" : "scan_wide", d, rev, text(p));
}
hipError_t launch_bwd_scans_bf16(int, int d, const ScanParams& q, const ScanParams& r, hipStream_t) {
  (void)note("bwd_scans_bf16 d=%d rev=1 %s", d, text(r));
  return note("+dq d=%d rev=0 %s", d, text(q));
}
hipError_t launch_bwd_scans_wide(int, int d, const ScanParams& q, const ScanParams& r, hipStream_t) {
  (void)note("bwd_scans_wide d=%d rev=1 %s", d, text(r));
  return note("+dq d=%d rev=0 %s", d, text(q));
}
hipError_t launch_chunk_state_pair_bf16(int, int d, const ScanParams& f, const ScanParams& r, hipStream_t) {
  (void)note("chunk_state_pair_bf16 d=%d rev=0 %s", d, text(f));
  return note("+rev d=%d rev=1 %s", d, text(r));
}
hipError_t launch_left_product_bf16(int d, bool rev, const ScanParams& p, hipStream_t) { return note("left_product d=%d rev=%d %s", d, rev, text(p)); }
hipError_t launch_scan_f32(int d, bool rev, const ScanParams& p, hipStream_t) { return note("scan_f32 d=%d rev=%d %s", d, rev, text(p)); }
hipError_t launch_chunk_states_f32(int d, bool rev, const ScanParams& p, hipStream_t) { return note("chunk_states_f32 d=%d rev=%d %s", d, rev, text(p)); }
hipError_t launch_chunk_state_pair_f32(int d, const ScanParams& f, const ScanParams& r, hipStream_t) {
  (void)note("chunk_state_pair_f32 d=%d rev=0 %s", d, text(f));
  return note("+rev d=%d rev=1 %s", d, text(r));
}
hipError_t launch_varlen_map(const ScanParams& p, int4*, int32_t*, int64_t, hipStream_t) { return note("varlen_map %s", text(p)); }
hipError_t launch_state_scan(int d, bool rev, const ScanParams& p, hipStream_t) { return note("state_scan d=%d rev=%d %s", d, rev, text(p)); }
hipError_t launch_recur(int d, int, int batch, int n, const RecurParams& p, hipStream_t) {
  return note("recur d=%d batch=%d nscan=%d t0=%d t1=%d", d, batch, n, p.t0, p.t1);
}
hipError_t launch_tail_bf16(int, int d, int batch, const RecurParams& p, hipStream_t) { return note("tail d=%d batch=%d t0=%d t1=%d", d, batch, p.t0, p.t1); }
hipError_t launch_short_scans(int, int d, const ShortParams& p, hipStream_t) {
  return note("short d=%d batch=%d heads=%d n=%d nscan=%d fin=%p", d, p.batch, p.heads, p.n, p.nscan, (void*)p.fin);
}
hipError_t launch_norm_bwd_rows(int d, int, const NormBwdParams&, hipStream_t) { return note("norm_bwd_rows d=%d", d); }
hipError_t launch_norm_fwd_rows(int d, int, const NormBwdParams&, float, hipStream_t) { return note("norm_fwd_rows d=%d", d); }
hipError_t launch_state_copy(float*, const float*, int64_t, hipStream_t) { return note("state_copy"); }
hipError_t launch_decode(int, int, int d, int, const void*, const void*, const void*, const float*, float*, void*, bool, float, hipStream_t) {
  return note("decode d=%d", d);
}
}  // namespace la2
