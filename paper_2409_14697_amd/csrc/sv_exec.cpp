// Plan execution: upload of the plan's device image, then one launch per pass
// (the dense and sweep passes through run_op_sweep).
#include "sv_host.h"

namespace sv {

sv_status build_fragments(const PackedPlan& pk, unsigned char* dev, hipStream_t s) {
  if (!pk.n_mx) return SV_OK;
  SV_LAUNCH(launch_stage_frags((PassStageDev*)(dev + pk.off_stage), (const uint32_t*)(dev + pk.off_list), pk.n_mx,
                               dev + pk.off_pool, dev + pk.off_frags, s),
            s);
  return SV_OK;
}

sv_status execute_plan(sv_state* s, const sv_plan* p) {
  PackedPlan pk;
  if (sv_status st = pack_plan(p, &pk)) return st;
  void* dev = nullptr;
  if (!pk.host.empty()) {
    sv_status st = upload(s, pk.host.data(), pk.host.size(), pk.dev_bytes, &dev);
    if (st != SV_OK) return st;
  }
  unsigned char* db = (unsigned char*)dev;
  if (sv_status st = build_fragments(pk, db, s->stream)) return st;
  // complex64 states: FP64 renormalisation after every `renorm` dense ops
  const int renorm = s->dt == SV_C64 ? p->opts.renorm_interval : 0;
  int since = 0;
  for (size_t i = 0; i < p->passes.size(); ++i) {
    const Pass& ps = p->passes[i];
    if (ps.kind == PASS_SWEEP) {
      sv_status st = run_op_sweep(s, ps.phys, nullptr);
      if (st != SV_OK) return st;
    } else if (ps.kind == PASS_DENSE) {
      sv_status st = run_op_sweep(s, ps.phys, db + pk.dense_off[i], p->opts.fp32_mfma != 0);
      if (st != SV_OK) return st;
      if (renorm > 0 && ++since >= renorm) {
        if (sv_status r = renormalize(s)) return r;
        since = 0;
      }
    } else if (ps.kind == PASS_MATRIX && s->dt == SV_C128) {
      SV_LAUNCH(launch_matrix_pass(ps.mx_k, s->ptr, s->n, ps.n_local, (const PassDescDev*)(db + pk.off_desc),
                                   pk.desc_index[i], (int)ps.stages.size(), (const PassStageDev*)(db + pk.off_stage),
                                   db + pk.off_pool, s->stream),
                s->stream);
    } else {
      SV_LAUNCH(launch_pass(s->dt, s->ptr, s->n, ps.n_local, (const PassDescDev*)(db + pk.off_desc),
                            pk.desc_index[i], (const PassStageDev*)(db + pk.off_stage),
                            (const PassItemDev*)(db + pk.off_items), db + pk.off_pool, db + pk.off_frags,
                            pk.pass_lp[i] != 0, pk.pass_mx[i], s->stream),
                s->stream);
    }
    if (ps.kind == PASS_MATRIX && renorm > 0 && (since += ps.n_ops) >= renorm) {
      if (sv_status r = renormalize(s)) return r;
      since = 0;
    }
  }
  if (renorm > 0 && since > 0) return renormalize(s);
  return SV_OK;
}

}  // namespace sv
