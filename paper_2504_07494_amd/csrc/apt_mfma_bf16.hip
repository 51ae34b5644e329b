#define APT_MFMA_DT 2
#define APT_MFMA_DEAL false
#include "apt_mfma.inc"
