#define APT_MFMA_DT 1
#define APT_MFMA_DEAL false
#include "apt_mfma.inc"
